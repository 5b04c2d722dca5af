// Device-side helpers used by more than one kernel.
#pragma once

#include "owl_internal.h"

namespace owl {

__device__ __forceinline__ void flag_status(uint32_t *st, uint32_t bit)
{
    if (st) atomicOr(st, bit);
}

// Four consecutive output channels, starting at element index `e` of the output array, in the
// output type: fp32 as it is, 16-bit types rounded to nearest even from the fp32 value.
__device__ __forceinline__ void store_out4(void *out, int64_t e, float4 v, int out_dtype)
{
    typedef float o_f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 o_bf16x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 o_f16x2 __attribute__((ext_vector_type(2)));
    if (out_dtype == OWL_F32) {
        *reinterpret_cast<float4 *>(static_cast<float *>(out) + e) = v;
        return;
    }
    const o_f32x2 lo = {v.x, v.y}, hi = {v.z, v.w};
    uint2 w;
    if (out_dtype == OWL_BF16) {
        w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, o_bf16x2));
        w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, o_bf16x2));
    } else {
        w.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, o_f16x2));
        w.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, o_f16x2));
    }
    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(out) + e) = w;
}

// Two channels, likewise.
__device__ __forceinline__ void store_out2(void *out, int64_t e, float2 v, int out_dtype)
{
    typedef float o_f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 o_bf16x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 o_f16x2 __attribute__((ext_vector_type(2)));
    if (out_dtype == OWL_F32) {
        *reinterpret_cast<float2 *>(static_cast<float *>(out) + e) = v;
        return;
    }
    const o_f32x2 x = {v.x, v.y};
    *reinterpret_cast<uint32_t *>(static_cast<uint16_t *>(out) + e) =
        out_dtype == OWL_BF16 ? __builtin_bit_cast(uint32_t, __builtin_convertvector(x, o_bf16x2))
                              : __builtin_bit_cast(uint32_t, __builtin_convertvector(x, o_f16x2));
}

// Asks for every line of the launch's arguments at once and waits for them.  They are cold in each launch, and left to
// itself the compiler loads them in several rounds, close to their uses, each a memory round trip of its own.  It pays where
// most of them are needed before the first load (split-KV pass: 56 rows, 8 heads, 600 / 2000 tokens 9.85 -> 9.78,
// 11.44 -> 11.33 us; a decoding iteration of one sequence of 1000 tokens, four layers, with it in its small steps 58.5 -> 57.8).
// The combine asks for a lone sequence's partials with a few of them, and waiting for the rest first cost every call 0.2-0.35 us
// (320 rows, 1 head, 10K tokens 14.03 -> 14.39, 56 rows, 8 heads, 2000 tokens 11.33 -> 11.68); the drafter kernels gain nothing.
template <typename Kernel> struct ArgBytes;
template <typename... A> struct ArgBytes<void(A...)> {      // of a kernel's type: its arguments one after the other, each aligned
    static constexpr int end_of()
    {
        size_t at = 0;
        ((at = (at + alignof(A) - 1) / alignof(A) * alignof(A) + sizeof(A)), ...);
        return (int)at;
    }
    static constexpr int value = end_of();
};
template <typename Kernel>
__device__ __forceinline__ void fetch_args()
{
    constexpr int bytes = ArgBytes<Kernel>::value;
    typedef const __attribute__((address_space(4))) int32_t *Line;
    const Line at = (Line)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int n = (bytes + 63) / 64;
    static_assert(n <= 4, "four lines of arguments");
    const int32_t a = at[0], b = at[n > 1 ? 16 : 0], c = at[n > 2 ? 32 : 0], d = at[n > 3 ? 48 : 0];
    asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d));
}

// Reads through the scalar cache; for arrays no kernel of the launch writes, uniform index.
__device__ __forceinline__ int load_uniform(const int32_t *a, int i)
{
    return ((const __attribute__((address_space(4))) int32_t *)reinterpret_cast<uintptr_t>(a))[i];
}

// Prefix length of sequence b, forced into [0, max_ctx_len].
__device__ __forceinline__ int load_ctx_len(const int32_t *ctx_lens, int b, int max_ctx_len,
                                            uint32_t *st)
{
    int L = load_uniform(ctx_lens, b);
    if (L < 0 || L > max_ctx_len) {
        flag_status(st, OWL_DEV_BAD_CTX_LEN);
        L = L < 0 ? 0 : max_ctx_len;
    }
    return L;
}

// Number of drafted tokens of sequence b: N unless a per-sequence array is given,
// whose entries are forced into [0, N].
__device__ __forceinline__ int load_n_draft(const int32_t *n_draft_seq, int b, int N, uint32_t *st)
{
    if (!n_draft_seq) return N;
    int n = load_uniform(n_draft_seq, b);
    if (n < 0 || n > N) {
        flag_status(st, OWL_DEV_BAD_NDRAFT);
        n = n < 0 ? 0 : N;
    }
    return n;
}

__device__ __forceinline__ Deal deal_units(const KParams &p, int units) { return deal_units(p.rule, units); }
__device__ __forceinline__ int seq_units(const KParams &p, int tokens) { return seq_units(p.rule, tokens); }

// Inclusive sum over the lanes of the wavefront, without LDS: within rows of 16 lanes by shifts of 1, 2, 4 and 8, then the
// last lane of a row to the next one, then lane 31 to the upper half.  (By shuffles through LDS, six
// round trips, and with each sequence's size read once more behind it, a batch took 0.5-1 us longer in both kernels: 16 rows,
// 24 sequences of 400-2K, head_dim 64, 19.7 -> 19.1 us; 64 rows, 100 of 100-1K 71.8 -> 68.6; 320 rows, 8 of 500-3K 43.0 -> 41.4.)
__device__ __forceinline__ int lane_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// The same steps for the greatest of the lanes' numbers, none below -1.
__device__ __forceinline__ int wave_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xc, 0xf, false));
    return __builtin_amdgcn_readlane(v, 63);
}

// The same steps for a sum of floats, which lane 63 ends up with and every lane gets.
__device__ __forceinline__ float wave_sum(float v)
{
#define OWL_DPP_ADD(ctrl, rows)                                                                                              \
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xf, false))
    OWL_DPP_ADD(0x111, 0xf);
    OWL_DPP_ADD(0x112, 0xf);
    OWL_DPP_ADD(0x114, 0xf);
    OWL_DPP_ADD(0x118, 0xf);
    OWL_DPP_ADD(0x142, 0xa);
    OWL_DPP_ADD(0x143, 0xc);
#undef OWL_DPP_ADD
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Length and draft count of a sequence, forced into range (and flagged).
struct SeqSize {
    int len, drafts;
};

// The units of a batch: lane l of the calling wavefront keeps sequence l's size and the running sum through it;
// sequences from 64 on are read again when they are asked for.
struct BatchUnits {
    int scan, total;
    SeqSize size;
};

// Sequences b0 .. b0 + 63, one a lane: their sizes and the running sum of their units.
__device__ __forceinline__ int chunk_scan(const KParams &p, int b0, SeqSize *size)
{
    const int b = b0 + (threadIdx.x & 63);
    int L = 0, n = 0;
    if (b < p.B) {
        const int len = p.ctx_lens[b], drafts = p.n_draft_seq ? p.n_draft_seq[b] : p.N;
        L = len < 0 ? 0 : min(len, p.max_ctx_len);
        n = drafts < 0 ? 0 : min(drafts, p.N);
        if (L != len) flag_status(p.dev_status, OWL_DEV_BAD_CTX_LEN);
        if (n != drafts) flag_status(p.dev_status, OWL_DEV_BAD_NDRAFT);
    }
    if (size) *size = SeqSize{L, n};
    return lane_scan(n == 0 ? 0 : seq_units(p, L + n));
}

__device__ __forceinline__ BatchUnits batch_units(const KParams &p)
{
    BatchUnits u;
    u.scan = chunk_scan(p, 0, &u.size);
    u.total = __builtin_amdgcn_readlane(u.scan, 63);
    for (int b0 = 64; b0 < p.B; b0 += 64) u.total += __builtin_amdgcn_readlane(chunk_scan(p, b0, nullptr), 63);
    return u;
}

// Size of sequence b, which lane b holds if b < 64: no second round trip for it.  Wave-uniform.
__device__ __forceinline__ SeqSize size_of(const KParams &p, const BatchUnits &u, int b)
{
    if (b < 64) return SeqSize{__builtin_amdgcn_readlane(u.size.len, b), __builtin_amdgcn_readlane(u.size.drafts, b)};
    return SeqSize{load_ctx_len(p.ctx_lens, b, p.max_ctx_len, nullptr), load_n_draft(p.n_draft_seq, b, p.N, nullptr)};
}

// Sequence that unit x falls into (0 <= x < total) and the units before it.  Wave-uniform.
__device__ __forceinline__ void find_unit(const KParams &p, const BatchUnits &u, int x, int *b_out, int *before_out)
{
    int base = 0, scan = u.scan;
    for (int b0 = 0;;) {
        const unsigned long long hit = __ballot(x < base + scan);
        if (hit || b0 + 64 >= p.B) {
            const int l = hit ? (int)__ffsll((long long)hit) - 1 : 63;
            *b_out = min(b0 + l, p.B - 1);
            *before_out = base + (l > 0 ? __builtin_amdgcn_readlane(scan, max(l - 1, 0)) : 0);
            return;
        }
        base += __builtin_amdgcn_readlane(scan, 63);
        b0 += 64;
        scan = chunk_scan(p, b0, nullptr);
    }
}

// Units before sequence b.  Wave-uniform.
__device__ __forceinline__ int units_before(const KParams &p, const BatchUnits &u, int b)
{
    int base = 0, scan = u.scan;
    for (int b0 = 0; b >= b0 + 64;) {
        base += __builtin_amdgcn_readlane(scan, 63);
        b0 += 64;
        scan = chunk_scan(p, b0, nullptr);
    }
    const int l = b & 63;
    return base + (l > 0 ? __builtin_amdgcn_readlane(scan, max(l - 1, 0)) : 0);
}

// Physical page of logical page lp of sequence b; an id outside the pool (or a
// logical page beyond the table) is replaced by page 0 and flagged.
__device__ __forceinline__ int load_page(const int32_t *page_table, int b, int max_pages,
                                         int64_t n_pool_pages, int lp, uint32_t *st)
{
    int pg;
    if (page_table) {
        if (lp >= max_pages) {
            flag_status(st, OWL_DEV_BAD_PAGE);
            return 0;
        }
        pg = page_table[(int64_t)b * max_pages + lp];
    } else {
        pg = lp;
    }
    if (pg < 0 || pg >= n_pool_pages) {
        flag_status(st, OWL_DEV_BAD_PAGE);
        pg = 0;
    }
    return pg;
}

// Ancestor-or-self sets (Sec. 3.2.2: a token placed after a tree path sees that path): one
// wavefront, lane i = node i < n <= 64, `parent` its entry of the parent array; the other lanes'
// results mean nothing.  A parent that is not in {-1} u [0, i) makes its node a root and is
// flagged.  Every round adds the set of the node the lane has reached and jumps to where that
// one has reached, so a chain of 64 takes six rounds.  (A walk from parent to parent, 90 ns a
// step, held up the workers that have the drafts of a chain of 60 for 5.3 us: 240 rows, 8 heads,
// 7K tokens, bf16, 23.5 -> 21.3 us, head_dim 64 19.6 -> 16.4; trees six deep within 1 %.)
__device__ __forceinline__ uint64_t ancestor_sets(int parent, int i, int n, uint32_t *st)
{
    if (i < n && (parent < -1 || parent >= i)) {
        flag_status(st, OWL_DEV_BAD_PARENT);
        parent = -1;
    }
    int up = i < n ? parent : -1;
    uint64_t set = (uint64_t)1 << i;
#pragma unroll 1                                     // (unrolled, it costs the fp32 kernel registers and 5 % of its time)
    for (int round = 0; round < 6 && __ballot(up >= 0); ++round) {       // (short paths need fewer)
        const int from = up < 0 ? i : up;
        const uint32_t lo = __shfl((uint32_t)set, from), hi = __shfl((uint32_t)(set >> 32), from);
        const int next = __shfl(up, from);
        set |= ((uint64_t)hi << 32) | lo;            // (a lane that has reached its root adds its own set)
        up = next;
    }
    return set;
}

// max over the four lanes {l, l^16, l^32, l^48}.  permlane32_swap(a, b) trades
// a's upper 32 lanes against b's lower 32; permlane16_swap trades a's odd
// 16-lane rows against b's even rows; fed with two copies of x, the two
// results together hold x and its partner for every lane.
__device__ __forceinline__ float quad_column_max(float v)
{
    const uint32_t x = __builtin_bit_cast(uint32_t, v);
    auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const float a = fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
    const uint32_t y = __builtin_bit_cast(uint32_t, a);
    auto r2 = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return fmaxf(__builtin_bit_cast(float, (uint32_t)r2[0]), __builtin_bit_cast(float, (uint32_t)r2[1]));
}

}  // namespace owl
