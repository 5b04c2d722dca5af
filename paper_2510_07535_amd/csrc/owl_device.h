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

// Cached rows of sequence b that the pass has to scan: 0 for a sequence without drafts.
__device__ __forceinline__ int seq_tokens(const KParams &p, int b)
{
    int L = p.ctx_lens[b];
    L = L < 0 ? 0 : (L > p.max_ctx_len ? p.max_ctx_len : L);        // flagged where the sequence is processed
    int n = p.n_draft_seq ? p.n_draft_seq[b] : p.N;
    n = n < 0 ? 0 : (n > p.N ? p.N : n);
    return n == 0 ? 0 : L + n;
}

// ---------------------------------------------------------------------------
// How the K/V of a launch is dealt out when the caller leaves the split size to
// the library.  A KV head (and row group) has `workers` workgroups, all resident
// at once, one per compute unit; the sequences' stages of 64 tokens are laid end
// to end and every worker takes an equal run of them, crossing from one sequence
// into the next where its share asks for it.  Each run is cut at the sequence
// boundaries into pieces, one partial per piece.  So every compute unit gets the
// same work whatever the lengths are, and pays for set-up and epilogue once or
// twice instead of once per split.  (Equal splits in 4-5 rounds of workgroups, the
// alternative, left 9 % of the compute units idle in the last round and 9 % of
// the time in set-up and epilogues on 16 sequences of 8K-64K tokens.)
//
// A sequence counts `seq_extra` units beyond its stages, at its end: what the masked
// steps over its drafts and the set-up of the following piece cost.
// ---------------------------------------------------------------------------
// a / b for 0 <= a, 0 < b and quotients below 2^20: a multiplication and a correction instead of the
// thirty dependent instructions of an integer division (four of them cost a workgroup half a microsecond).
__device__ __forceinline__ int quotient(int a, int b)
{
    int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
    int r = a - q * b;
    if (r < 0) --q, r += b;
    if (r >= b) ++q;
    return __builtin_amdgcn_readfirstlane(q);
}

__device__ __forceinline__ Deal deal_units(const KParams &p, int units)
{
    // more than one round only where a share would outgrow the page list in LDS
    int n = p.round_workers;
    if (units > n * kMaxPieceUnits) n *= quotient(units + n * kMaxPieceUnits - 1, n * kMaxPieceUnits);
    n = min(n, p.max_workers);
    if (units < n * p.min_units) n = max(1, quotient(units, p.min_units));
    const int q = quotient(units, n);
    return Deal{n, q, units - q * n};
}
__device__ __forceinline__ int deal_begin(const Deal &d, int worker) { return worker * d.q + min(worker, d.r); }
__device__ __forceinline__ int deal_worker(const Deal &d, int unit)
{
    const int cut = d.r * (d.q + 1);
    return unit < cut ? quotient(unit, d.q + 1) : d.r + quotient(unit - cut, d.q);
}

__device__ __forceinline__ int stages_of(int tokens) { return (tokens + kSplitQuantum - 1) / kSplitQuantum; }
__device__ __forceinline__ int seq_units(const KParams &p, int tokens)
{
    return tokens == 0 ? 0 : stages_of(tokens) + p.seq_extra;
}

// Inclusive sum over the lanes of the wavefront.
__device__ __forceinline__ int lane_scan(int v)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(v, off);
        if (lane >= off) v += up;
    }
    return v;
}

// The units of a batch: lane l of the calling wavefront keeps the running sum through sequence l;
// sequences from 64 on are read again when they are asked for.
struct BatchUnits {
    int scan, total;
};

__device__ __forceinline__ int chunk_scan(const KParams &p, int b0)
{
    const int b = b0 + (threadIdx.x & 63);
    return lane_scan(b < p.B ? seq_units(p, seq_tokens(p, b)) : 0);
}

__device__ __forceinline__ BatchUnits batch_units(const KParams &p)
{
    BatchUnits u;
    u.scan = chunk_scan(p, 0);
    u.total = __builtin_amdgcn_readlane(u.scan, 63);
    for (int b0 = 64; b0 < p.B; b0 += 64) u.total += __builtin_amdgcn_readlane(chunk_scan(p, b0), 63);
    return u;
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
        scan = chunk_scan(p, b0);
    }
}

// Units before sequence b.  Wave-uniform.
__device__ __forceinline__ int units_before(const KParams &p, const BatchUnits &u, int b)
{
    int base = 0, scan = u.scan;
    for (int b0 = 0; b >= b0 + 64;) {
        base += __builtin_amdgcn_readlane(scan, 63);
        b0 += 64;
        scan = chunk_scan(p, b0);
    }
    const int l = b & 63;
    return base + (l > 0 ? __builtin_amdgcn_readlane(scan, max(l - 1, 0)) : 0);
}

// The last words of a batch's workspace say what equal splits of the planned size would make of it
// (int32): [0] that size C, [1] the number of (sequence, split) pairs, [2 + b] the pairs of the
// sequences before b (b = 0 .. B).  For inspection; no kernel reads it.  One wavefront.
__device__ __forceinline__ void write_batch_info(const KParams &p)
{
    const int lane = threadIdx.x & 63;
    int base = 0;
    for (int b0 = 0; b0 < p.B; b0 += 64) {
        const bool live = b0 + lane < p.B;
        const int n = live ? (seq_tokens(p, b0 + lane) + p.C - 1) / p.C : 0;
        const int scan = lane_scan(n);
        if (live) p.batch_info[2 + b0 + lane] = base + scan - n;
        base += __builtin_amdgcn_readlane(scan, 63);
    }
    if (lane == 0) {
        p.batch_info[2 + p.B] = base;
        p.batch_info[0] = p.C;
        p.batch_info[1] = base;
    }
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

// Ancestor-or-self set of node i (Sec. 3.2.2: a token placed after a tree path
// sees that path).  `parent` is a copy of the sequence's parent array in LDS or
// registers-backed memory; a parent that is not in {-1} u [0, j) ends the walk
// as if it were a root and is flagged.  The walk visits strictly decreasing
// indices, so it ends after at most i + 1 steps.
__device__ __forceinline__ uint64_t ancestor_set(const int32_t *parent, int i, int *depth_out,
                                                 uint32_t *st)
{
    uint64_t set = 0;
    int depth = 0;
    int jn = i;
    while (jn >= 0) {
        set |= (uint64_t)1 << jn;
        ++depth;
        int pj = parent[jn];
        if (pj < -1 || pj >= jn) {
            flag_status(st, OWL_DEV_BAD_PARENT);
            pj = -1;
        }
        jn = pj;
    }
    if (depth_out) *depth_out = depth;
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
