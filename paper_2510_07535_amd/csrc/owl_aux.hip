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
// channels of tiles u and u + 1; the weight of split s is then 2^(m_s - M) l_s s_s.
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

__device__ __forceinline__ float2 unpack_half2(uint32_t w)
{
    const c_f16x2 h = __builtin_bit_cast(c_f16x2, w);
    return make_float2((float)h[0], (float)h[1]);
}

template <int D, bool HALF, int WAVES, bool BY_CHANNEL>
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

    // The merge is a chain (each partial rescales the running sums), the loads are not: the
    // partials of kInFlight splits are requested together, so that a wavefront pays the
    // memory latency once per batch rather than once per split (up to 32 splits: once).
    constexpr int kInFlight = 8;
    float ms[kInFlight], ls[kInFlight], ss[kInFlight];
    uint4 raw[kInFlight][HALF ? 1 : UPW];                    // fp16 or fp32 values as they are stored
    auto load = [&](int s_first, int s0, int limit) {        // past the end: re-read the last one, not merged
        const size_t slot0 = ((size_t)g * p.n_slots + s_first) * p.RT + tg;
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            const size_t slot = slot0 + (size_t)min(s0 + kStride * k, limit - 1) * p.RT;
            ms[k] = p.part_ml[slot * kPartMl + j];
            ls[k] = p.part_ml[slot * kPartMl + 16 + j];
            ss[k] = HALF ? p.part_ml[slot * kPartMl + 32 + j] : 1.f;
            const uint4 *po = static_cast<const uint4 *>(p.part_o) + slot * (size_t)(NT / (HALF ? 2 : 1) * 64) + lane;
            static_assert(UPW == 2, "one 16-byte piece per lane holds a pair of channel tiles");
            if constexpr (HALF) raw[k][0] = po[(u0 / 2) * 64];
            else
#pragma unroll
                for (int u = 0; u < UPW; ++u) raw[k][u] = po[(u0 + u) * 64];
        }
    };

    // The partials of this row tile: `ns` slots from s_first on (wave-uniform).  Where they begin depends on
    // the lengths only in a batch; otherwise the first ones are requested before the length is known.
    const bool late = p.dealt && p.B > 1;
    int s_first = p.dealt ? 0 : b * p.max_splits, limit = p.dealt ? p.rule.max_workers : p.max_splits, ns = 0;
    if (!late) load(s_first, first, limit);
    // (entries out of range are reported from here as well: every sequence has its workgroups in this grid, while the
    // split-KV pass of a batch never gets to one that is left without drafts)
    int Nb, L;
    if (late) {
        const BatchUnits u = batch_units(p);
        const SeqSize size = size_of(p, u, b);
        Nb = size.drafts;
        L = size.len;
        if (Nb > 0 && L + Nb > 0) {
            const Deal deal = deal_units(p, u.total);
            const int before = units_before(p, u, b), w0 = deal_worker(deal, before);
            s_first = w0 + b;
            limit = ns = deal_worker(deal, before + stages_of(L + Nb) - 1) - w0 + 1;
            load(s_first, first, limit);
        }
    } else {
        Nb = load_n_draft(p.n_draft_seq, b, p.N, p.dev_status);
        L = load_ctx_len(p.ctx_lens, b, p.max_ctx_len, p.dev_status);
        const int T_b = Nb == 0 ? 0 : L + Nb;                 // a sequence without drafts wrote no partials
        if (T_b > 0 && !p.dealt) {
            ns = min((T_b + p.C - 1) / p.C, p.max_splits);
        } else if (T_b > 0) {
            const Deal deal = T_b == p.max_ctx_len + p.N ? p.full : deal_units(p, seq_units(p, T_b));
            ns = deal_worker(deal, stages_of(T_b) - 1) + 1;
        }
    }

    float mw = -INFINITY, lw = 0.f;
    float4 acc[UPW];
#pragma unroll
    for (int u = 0; u < UPW; ++u) acc[u] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int s0 = first; s0 < ns;) {
#pragma unroll
        for (int k = 0; k < kInFlight; ++k) {
            if (s0 + kStride * k < ns) {                     // uniform over the wavefront
                const float mn = fmaxf(mw, ms[k]);
                const float a = __builtin_amdgcn_exp2f(mw - mn);     // 0 on the first round (mw = -inf)
                const float c = __builtin_amdgcn_exp2f(ms[k] - mn);
                mw = mn;
                lw = lw * a + ls[k] * c;
                const float co = HALF ? c * (ls[k] * ss[k]) : c;     // the stored rows are O / (l s)
#pragma unroll
                for (int u = 0; u < UPW; ++u) {
                    float4 x;
                    if constexpr (HALF) {
                        const float2 lo = unpack_half2(u ? raw[k][0].z : raw[k][0].x), hi = unpack_half2(u ? raw[k][0].w : raw[k][0].y);
                        x = make_float4(lo.x, lo.y, hi.x, hi.y);
                    } else {
                        x = __builtin_bit_cast(float4, raw[k][u]);
                    }
                    acc[u].x = acc[u].x * a + x.x * co; acc[u].y = acc[u].y * a + x.y * co;
                    acc[u].z = acc[u].z * a + x.z * co; acc[u].w = acc[u].w * a + x.w * co;
                }
            }
        }
        s0 += kStride * kInFlight;
        if (s0 < ns) load(s_first, s0, limit);
    }
    float lsum = lw;
    float4 tot[UPW];
    if constexpr (BY_CHANNEL) {
#pragma unroll
        for (int u = 0; u < UPW; ++u) tot[u] = acc[u];
    } else {
        __shared__ float4 s_acc[WAVES][UPW][64];
        __shared__ float s_m[WAVES][64], s_l[WAVES][64];
#pragma unroll
        for (int u = 0; u < UPW; ++u) s_acc[w][u][lane] = acc[u];
        s_m[w][lane] = mw;
        s_l[w][lane] = lw;
        __syncthreads();
        if (w != 0) return;
        float M = s_m[0][lane];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) M = fmaxf(M, s_m[k][lane]);
        lsum = 0.f;
#pragma unroll
        for (int u = 0; u < UPW; ++u) tot[u] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const float wk = s_m[k][lane] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(s_m[k][lane] - M);
            lsum += wk * s_l[k][lane];
#pragma unroll
            for (int u = 0; u < UPW; ++u) {
                const float4 y = s_acc[k][u][lane];
                tot[u].x += wk * y.x; tot[u].y += wk * y.y; tot[u].z += wk * y.z; tot[u].w += wk * y.w;
            }
        }
    }
    const int row = tg * kRowTile + j;
    if (row >= p.R) return;
    const int i = row / p.G, hh = row % p.G;
    const float inv = i < Nb ? 1.0f / lsum : 0.f;                   // rows of absent nodes come out as zeros
    const int64_t o = (((int64_t)b * p.N + i) * p.Hq + g * p.G + hh) * D + 4 * qd;
#pragma unroll
    for (int u = 0; u < UPW; ++u)
        store_out4(p.out, o + 16 * (u0 + u),
                   i < Nb ? make_float4(tot[u].x * inv, tot[u].y * inv, tot[u].z * inv, tot[u].w * inv)
                          : make_float4(0.f, 0.f, 0.f, 0.f),
                   p.out_dtype);
}

template <int D, int WAVES, bool BY_CHANNEL>
static void launch_combine_as(const KParams &p, bool half_partials, dim3 grid, hipStream_t s)
{
    const dim3 block(64 * WAVES);
    if (half_partials) hipLaunchKernelGGL((combine_kernel<D, true, WAVES, BY_CHANNEL>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((combine_kernel<D, false, WAVES, BY_CHANNEL>), grid, block, 0, s, p);
}

template <int D>
static void launch_combine_d(const KParams &p, bool half_partials, hipStream_t s)
{
    // Partials per sequence on average, if all sequences are alike.
    const int per_seq = p.dealt ? (p.rule.max_workers + p.B - 1) / p.B : p.max_splits;
    if (p.B > 1 && per_seq <= 8) {
        launch_combine_as<D, D / 32, true>(p, half_partials, dim3(p.Hkv, p.RT, p.B), s);
        return;
    }
    const dim3 grid(p.Hkv, p.RT * (D / 32), p.B);
    // a wavefront merges its splits as a chain, 8 loads in flight: beyond 32 splits more wavefronts share them
    if (per_seq > 32) launch_combine_as<D, 8, false>(p, half_partials, grid, s);
    else launch_combine_as<D, 4, false>(p, half_partials, grid, s);
}

hipError_t launch_combine(const KParams &p, int D, bool half_partials, hipStream_t s)
{
    if (D == 128) launch_combine_d<128>(p, half_partials, s);
    else launch_combine_d<64>(p, half_partials, s);
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
hipError_t load_aux_kernels()
{
    hipFuncAttributes a;
    hipError_t e = hipSuccess;
    const void *fns[] = {
        reinterpret_cast<const void *>(&combine_kernel<128, true, 4, false>), reinterpret_cast<const void *>(&combine_kernel<128, true, 8, false>),
        reinterpret_cast<const void *>(&combine_kernel<128, true, 4, true>),
        reinterpret_cast<const void *>(&combine_kernel<128, false, 4, false>), reinterpret_cast<const void *>(&combine_kernel<128, false, 8, false>),
        reinterpret_cast<const void *>(&combine_kernel<128, false, 4, true>),
        reinterpret_cast<const void *>(&combine_kernel<64, true, 4, false>), reinterpret_cast<const void *>(&combine_kernel<64, true, 8, false>),
        reinterpret_cast<const void *>(&combine_kernel<64, true, 2, true>),
        reinterpret_cast<const void *>(&combine_kernel<64, false, 4, false>), reinterpret_cast<const void *>(&combine_kernel<64, false, 8, false>),
        reinterpret_cast<const void *>(&combine_kernel<64, false, 2, true>),
    };
    for (const void *f : fns)
        if (e == hipSuccess) e = hipFuncGetAttributes(&a, f);
    return e;
}

}  // namespace owl
