// Log-sum-exp combine of the split partials, the tree-mask builder and the
// page-gather test hook.
#include "owl_device.h"

namespace owl {

// ---------------------------------------------------------------------------
// Combine.  A partial of split s is the triple (m_s, l_s, O_s) with
// O_s = sum_k 2^(x_k - m_s) v_k and l_s = sum_k 2^(x_k - m_s) over the split's
// visible keys (x = score * log2 e; m_s is the reference the split happened to
// use, not necessarily its max).  With M = max_s m_s:
//     out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s.
// For fp32 inputs the partials are the raw accumulator fragments, float4
// [slot][u][lane] = channels 16*u + 4*quad .. +3 of row lane%16.  For 16-bit
// inputs (HALF) a row of a partial is stored normalised, O_s / (l_s s_s) with s_s
// its largest magnitude, as fp16: uint4 [slot][u/2][lane] holds the lane's four
// channels of tiles u and u + 1; the weight of split s is then 2^(m_s - M) w_s, w_s = l_s s_s.
//
// Two ways to spread the work, chosen by the launch:
//   few sequences  One workgroup per (sequence, KV head, 16-row tile, pair of channel tiles); its WAVES
//                  wavefronts (4, or 8 when there are more than 32 partials; 16 gained nothing) take every
//                  WAVES-th partial, reduce their share against their own running maximum, and are
//                  merged through LDS with the same formula.
//   batches        (BY_CHANNEL) a sequence has few partials but there are many rows: one workgroup per
//                  (sequence, KV head, 16-row tile), a wavefront per pair of channel tiles, each merging
//                  all partials by itself: a quarter of the workgroups, no LDS, no barrier.
// ---------------------------------------------------------------------------
typedef _Float16 c_f16x2 __attribute__((ext_vector_type(2)));

struct RowStats {                                    // of a row of a partial, as the split-KV pass leaves them (kPartMl)
    float m, l, w;
};

// acc += c * (the four values of one channel tile), each product and sum in fp32.
__device__ __forceinline__ void add_scaled(float4 &acc, float c, uint32_t lo, uint32_t hi)
{
    const c_f16x2 a = __builtin_bit_cast(c_f16x2, lo), b = __builtin_bit_cast(c_f16x2, hi);
    acc.x = __builtin_fmaf((float)a[0], c, acc.x);
    acc.y = __builtin_fmaf((float)a[1], c, acc.y);
    acc.z = __builtin_fmaf((float)b[0], c, acc.z);
    acc.w = __builtin_fmaf((float)b[1], c, acc.w);
}
__device__ __forceinline__ void add_scaled(float4 &acc, float c, float4 x)
{
    acc.x = __builtin_fmaf(x.x, c, acc.x);
    acc.y = __builtin_fmaf(x.y, c, acc.y);
    acc.z = __builtin_fmaf(x.z, c, acc.z);
    acc.w = __builtin_fmaf(x.w, c, acc.w);
}
__device__ __forceinline__ void scale(float4 &acc, float a)
{
    acc.x *= a; acc.y *= a; acc.z *= a; acc.w *= a;
}

// This kernel is a chain: arguments, partials, merge, store.  Beside the round trips the number of instructions between them
// counts (executed by a wavefront: 633 with 32 partials a row and 1024 with 128, now 403 and 666): addresses advance by a constant
// instead of a product for each partial, a row's three statistics come in one load, the greatest reference of the partials
// in flight is found first (one rescale for all of them instead of one each), the halves enter the sums as they are
// (v_fma_mix), four wavefronts share the end, and what a batch needs to find its partials (LATE) is a kernel of its own.
// us per call, 8 heads, bf16: 24 rows, 5K / 32K tokens 11.65 -> 11.2 / 27.7 -> 27.25, 240 rows, 5K 16.85 -> 16.5, 320 rows, 1 head,
// 128K 34.7 -> 34.0, four sequences of 900-9K, 48 rows 19.85 -> 19.35.
template <int D, bool HALF, int WAVES, bool BY_CHANNEL, bool LATE>
__global__ void __launch_bounds__(64 * WAVES) combine_kernel(const KParams p)
{
    constexpr int NT = D / 16, UPW = 2;              // channel tiles per wavefront
    constexpr int NUG = NT / UPW;
    static_assert(!BY_CHANNEL || WAVES == NUG, "one wavefront per pair of channel tiles");
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // KV heads vary fastest, as in the split-KV pass: with eight heads the partials of a head were written on XCD (head mod 8) and
    // are found in its L2 (row tiles fastest: 240 rows, four sequences 6.6 -> 5.4 us, 320 rows, 128K 7.5 -> 6.8; lone 240 rows, 5K
    // whole call 19.4 -> 18.5).
    const int tg = BY_CHANNEL ? blockIdx.y : blockIdx.y / NUG;
    const int u0 = (BY_CHANNEL ? w : (int)(blockIdx.y % NUG)) * UPW;
    const int g = blockIdx.x, b = blockIdx.z;
    const int j = lane & 15, qd = lane >> 4;
    constexpr int kStride = BY_CHANNEL ? 1 : WAVES;  // this wavefront's partials: first, first + kStride, ...
    const int first = BY_CHANNEL ? 0 : w;

    // The merge is a chain, the loads are not: the partials of kInFlight splits are requested together, so that a wavefront
    // pays the memory latency once per batch rather than once per split (up to 32 splits: once).
    constexpr int kInFlight = 8;
    constexpr uint32_t kMlBytes = kPartMl * sizeof(float), kTileBytes = HALF ? 512 : 1024, kPartBytes = NT * kTileBytes;
    RowStats st[kInFlight];
    uint4 raw[kInFlight][HALF ? 1 : UPW];                    // fp16 or fp32 values as they are stored
    const uint32_t ml_lane = j * sizeof(RowStats), po_lane = lane * 16 + u0 * kTileBytes;
    const char *ml = nullptr, *po = nullptr;                 // of this wavefront's next partial (wave-uniform)
    int at = 0;                                              // its number in the sequence
    auto start = [&](int s_first, int s0) {
        const uint32_t slot = ((uint32_t)g * (uint32_t)p.n_slots + (uint32_t)(s_first + s0)) * (uint32_t)p.RT + (uint32_t)tg;
        ml = reinterpret_cast<const char *>(p.part_ml) + (size_t)slot * kMlBytes;
        po = static_cast<const char *>(p.part_o) + (size_t)slot * kPartBytes;
        at = s0;
    };
    const uint32_t step = (uint32_t)kStride * (uint32_t)p.RT;
    const uint64_t ml_step = (uint64_t)step * kMlBytes, po_step = (uint64_t)step * kPartBytes;
    auto load = [&](int limit) {                             // past the end: re-read the last one, not merged
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            st[k] = *reinterpret_cast<const RowStats *>(ml + ml_lane);
            static_assert(UPW == 2, "one 16-byte piece per lane holds a pair of channel tiles");
#pragma unroll
            for (int u = 0; u < (HALF ? 1 : UPW); ++u) raw[k][u] = *reinterpret_cast<const uint4 *>(po + po_lane + u * kTileBytes);
            const bool more = at + kStride < limit;
            at += kStride;
            ml += more ? ml_step : 0;
            po += more ? po_step : 0;
        }
    };

    // The partials of this row tile: `ns` slots from s_first on (wave-uniform).  Where they begin depends on
    // the lengths only in a batch; otherwise the first ones are requested before the length is known.
    int limit = LATE ? 0 : (p.dealt ? p.rule.max_workers : p.max_splits), ns = 0;
    if constexpr (!LATE) {
        start(p.dealt ? 0 : b * p.max_splits, min(first, limit - 1));
        load(limit);
    }
    // Row r of the tile belongs to node r / G, which the product with the reciprocal gives exactly (see the split-KV pass).
    const int row = tg * kRowTile + j;
    const int i = (int)(((float)row + 0.5f) * __builtin_amdgcn_rcpf((float)p.G)), hh = row - i * p.G;
    const int64_t o = (((int64_t)b * p.N + i) * p.Hq + g * p.G + hh) * D + 4 * qd + 16 * u0;
    // (entries out of range are reported from here as well: every sequence has its workgroups in this grid, while the
    // split-KV pass of a batch never gets to one that is left without drafts)
    int Nb, L;
    if constexpr (LATE) {
        const BatchUnits u = batch_units(p);
        const SeqSize size = size_of(p, u, b);
        Nb = size.drafts;
        L = size.len;
        if (Nb > 0 && L + Nb > 0) {
            const Deal deal = deal_units(p, u.total);
            const int before = units_before(p, u, b), w0 = deal_worker(deal, before);
            limit = ns = deal_worker(deal, before + stages_of(L + Nb) - 1) - w0 + 1;
            start(w0 + b, min(first, limit - 1));
            load(limit);
        }
    } else {
        Nb = load_n_draft(p.n_draft_seq, b, p.N, p.dev_status);
        L = load_ctx_len(p.ctx_lens, b, p.max_ctx_len, p.dev_status);
        const int T_b = Nb == 0 ? 0 : L + Nb;                 // a sequence without drafts wrote no partials
        if (T_b > 0 && !p.dealt) {
            ns = min((T_b + p.C - 1) / p.C, p.max_splits);
        } else if (T_b == p.max_ctx_len + p.N) {
            ns = p.full_pieces;
        } else if (T_b > 0) {
            ns = deal_worker(deal_units(p, seq_units(p, T_b)), stages_of(T_b) - 1) + 1;
        }
    }

    float mw = -INFINITY, lw = 0.f;
    float4 acc[UPW];
#pragma unroll
    for (int u = 0; u < UPW; ++u) acc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = first; s0 < ns;) {
        float top = mw;
#pragma unroll
        for (int k = 0; k < kInFlight; ++k)
            if (s0 + kStride * k < ns) top = fmaxf(top, st[k].m);    // uniform over the wavefront
        if (s0 != first) {
            const float a = __builtin_amdgcn_exp2f(mw - top);
            lw *= a;
#pragma unroll
            for (int u = 0; u < UPW; ++u) scale(acc[u], a);
        }
        mw = top;
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            if (s0 + kStride * k < ns) {
                const float c = __builtin_amdgcn_exp2f(st[k].m - top);
                lw = __builtin_fmaf(st[k].l, c, lw);
                if constexpr (HALF) {
                    const float co = c * st[k].w;                    // the stored rows are O / w, w = l s
                    add_scaled(acc[0], co, raw[k][0].x, raw[k][0].y);
                    add_scaled(acc[1], co, raw[k][0].z, raw[k][0].w);
                } else {
#pragma unroll
                    for (int u = 0; u < UPW; ++u) add_scaled(acc[u], c, __builtin_bit_cast(float4, raw[k][u]));
                }
            }
        }
        s0 += kStride * kInFlight;
        if (s0 < ns) load(limit);
    }
    if constexpr (BY_CHANNEL) {
        if (row >= p.R) return;
        const float inv = i < Nb ? 1.0f / lw : 0.f;                  // rows of absent nodes come out as zeros
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            scale(acc[u], inv);
            store_out4(p.out, o + 16 * u, i < Nb ? acc[u] : make_float4(0.f, 0.f, 0.f, 0.f), p.out_dtype);
        }
    } else {
        // The first four wavefronts finish two of a lane's eight channels each.
        static_assert(WAVES >= 4 && UPW == 2, "four wavefronts, two channels of one tile each");
        __shared__ float4 s_acc[WAVES][UPW][64];
        __shared__ float2 s_ml[WAVES][64];
#pragma unroll
        for (int u = 0; u < UPW; ++u) s_acc[w][u][lane] = acc[u];
        s_ml[w][lane] = make_float2(mw, lw);
        __syncthreads();
        if (w >= 4 || row >= p.R) return;
        const int u = w >> 1, half = w & 1;
        float2 ml_of[WAVES];
        float M = -INFINITY, lsum = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            ml_of[k] = s_ml[k][lane];
            M = fmaxf(M, ml_of[k].x);
        }
        float2 tot = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const float wk = __builtin_amdgcn_exp2f(ml_of[k].x - M);        // 0 for a wavefront without partials
            lsum = __builtin_fmaf(ml_of[k].y, wk, lsum);
            const float2 y = reinterpret_cast<const float2 *>(&s_acc[k][u][lane])[half];
            tot.x = __builtin_fmaf(y.x, wk, tot.x);
            tot.y = __builtin_fmaf(y.y, wk, tot.y);
        }
        const float inv = 1.0f / lsum;
        store_out2(p.out, o + 16 * u + 2 * half, i < Nb ? make_float2(tot.x * inv, tot.y * inv) : make_float2(0.f, 0.f), p.out_dtype);
    }
}

template <int D, int WAVES, bool BY_CHANNEL, bool LATE>
static void launch_combine_as(const KParams &p, bool half_partials, dim3 grid, hipStream_t s)
{
    const dim3 block(64 * WAVES);
    if (half_partials) hipLaunchKernelGGL((combine_kernel<D, true, WAVES, BY_CHANNEL, LATE>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((combine_kernel<D, false, WAVES, BY_CHANNEL, LATE>), grid, block, 0, s, p);
}

template <int D, bool LATE>
static void launch_combine_d(const KParams &p, bool half_partials, hipStream_t s)
{
    // Partials per sequence on average, if all sequences are alike.
    const int per_seq = p.dealt ? (p.rule.max_workers + p.B - 1) / p.B : p.max_splits;
    if (p.B > 1 && per_seq <= 8) {
        launch_combine_as<D, D / 32, true, LATE>(p, half_partials, dim3(p.Hkv, p.RT, p.B), s);
        return;
    }
    const dim3 grid(p.Hkv, p.RT * (D / 32), p.B);
    // a wavefront merges its splits as a chain, 8 loads in flight: beyond 32 splits more wavefronts share them
    if (per_seq > 32) launch_combine_as<D, 8, false, LATE>(p, half_partials, grid, s);
    else launch_combine_as<D, 4, false, LATE>(p, half_partials, grid, s);
}

hipError_t launch_combine(const KParams &p, int D, bool half_partials, hipStream_t s)
{
    const bool late = p.dealt && p.B > 1;                    // where a sequence's partials begin depends on the lengths
    if (D == 128) late ? launch_combine_d<128, true>(p, half_partials, s) : launch_combine_d<128, false>(p, half_partials, s);
    else late ? launch_combine_d<64, true>(p, half_partials, s) : launch_combine_d<64, false>(p, half_partials, s);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tree mask: one wavefront per sequence, lane i = node i.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) tree_mask_kernel(const int32_t *parent, int N, uint64_t *anc,
                                                       int32_t *depth, uint32_t *status)
{
    const int b = blockIdx.x, i = threadIdx.x;
    const uint64_t set = ancestor_sets(parent[(int64_t)b * N + min(i, N - 1)], i, N, status);
    if (i < N) {
        anc[(int64_t)b * N + i] = set;
        if (depth) depth[(int64_t)b * N + i] = __popcll(set);
    }
}

hipError_t launch_tree_mask(const int32_t *parent, int B, int N, uint64_t *anc, int32_t *depth,
                            uint32_t *status, hipStream_t s)
{
    hipLaunchKernelGGL(tree_mask_kernel, dim3(B), dim3(64), 0, s, parent, N, anc, depth, status);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gather: dst[t][g][:] = cache row of logical position first + t, 16 bytes per
// thread.  Same page walk as the split-KV pass.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) gather_kernel(const unsigned char *cache,
                                                     const int32_t *page_table, int seq,
                                                     int max_pages, int64_t n_pool_pages, int Hkv,
                                                     int row_bytes, int es, int64_t stride_page,
                                                     int64_t stride_head, int64_t stride_token,
                                                     int64_t first, int64_t n, unsigned char *dst,
                                                     uint32_t *status)
{
    const int ppr = row_bytes / 16;
    const int64_t total = n * Hkv * ppr;
    for (int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x; id < total;
         id += (int64_t)gridDim.x * 256) {
        const int piece = (int)(id % ppr);
        const int g = (int)((id / ppr) % Hkv);
        const int64_t t = id / ((int64_t)ppr * Hkv);
        const int64_t pos = first + t;
        const int64_t pg = load_page(page_table, seq, max_pages, n_pool_pages, (int)(pos / kPage), status);
        const int64_t off = (pg * stride_page + g * stride_head + (pos % kPage) * stride_token) * es;
        *reinterpret_cast<uint4 *>(dst + (t * Hkv + g) * row_bytes + piece * 16) =
            *reinterpret_cast<const uint4 *>(cache + off + piece * 16);
    }
}

hipError_t launch_gather(const owl_verify_desc &d, const void *cache, const int32_t *page_table,
                         int seq, int64_t first, int64_t n, void *dst, uint32_t *status,
                         hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const int es = d.qkv_dtype == OWL_F32 ? 4 : 2;
    const int row_bytes = d.head_dim * es;
    const int64_t total = n * d.n_kv_heads * (row_bytes / 16);
    int blocks = (int)((total + 255) / 256);
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(gather_kernel, dim3(blocks), dim3(256), 0, s,
                       static_cast<const unsigned char *>(cache), page_table, seq,
                       d.max_pages_per_seq, d.n_pool_pages, d.n_kv_heads, row_bytes, es,
                       d.kv_stride_page, d.kv_stride_head, d.kv_stride_token, first, n,
                       static_cast<unsigned char *>(dst), status);
    return hipGetLastError();
}

// Makes the runtime resolve the combine kernels now, so that their first launch may happen
// inside a stream capture.
template <int D, bool HALF, bool LATE>
static hipError_t load_combine()
{
    const void *fns[] = {
        reinterpret_cast<const void *>(&combine_kernel<D, HALF, 4, false, LATE>),
        reinterpret_cast<const void *>(&combine_kernel<D, HALF, 8, false, LATE>),
        reinterpret_cast<const void *>(&combine_kernel<D, HALF, D / 32, true, LATE>),
    };
    hipFuncAttributes a;
    hipError_t e = hipSuccess;
    for (const void *f : fns)
        if (e == hipSuccess) e = hipFuncGetAttributes(&a, f);
    return e;
}

hipError_t load_aux_kernels()
{
    hipError_t (*const loads[])() = {
        &load_combine<128, true, false>, &load_combine<128, true, true>, &load_combine<128, false, false>, &load_combine<128, false, true>,
        &load_combine<64, true, false>, &load_combine<64, true, true>, &load_combine<64, false, false>, &load_combine<64, false, true>,
    };
    hipError_t e = hipSuccess;
    for (auto load : loads)
        if (e == hipSuccess) e = load();
    return e;
}

}  // namespace owl
