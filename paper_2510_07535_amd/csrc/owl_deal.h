// How the K/V of a launch is dealt out when the caller leaves the split size to the library: the
// arithmetic that the kernels and the host share (integers only, the same results on both).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace owl {

constexpr int kPage = 16;                 // tokens per cache page
constexpr int kSplitQuantum = 64;         // split_tokens is a multiple of every stage size
// The page list of one piece of work sits in LDS (12 KB beside the 128 KB ring); one worker's share of
// a launch whose work is dealt out evenly never exceeds it (see deal_units).
constexpr int kMaxPiecePages = 3072;
constexpr int kMaxPieceUnits = kMaxPiecePages * kPage / kSplitQuantum - 1;

// `units` stages of work dealt out evenly: the first r workers take q + 1 of them, the others q.
struct Deal {
    int32_t workers, q, r;
};

// What the plan fixes about the dealing of a launch.
struct DealRule {
    int32_t min_units;    // least units (stages of 64 tokens) worth a worker
    int32_t round_workers;// workers per (KV head, row group) that run at the same time
    int32_t max_workers;  // workers per (KV head, row group) of the launched grid
    int32_t merge;        // kMergeUnits where the merge limits the workers (most_workers), else 0
    int32_t seq_extra;    // units a sequence counts beyond its stages (set-up, masked steps)
};

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
// a / b for 0 <= a, 0 < b and quotients below 2^20.  In a kernel (a, b uniform over the wavefront): a multiplication and a
// correction instead of the thirty dependent instructions of an integer division (four of them cost a workgroup half a
// microsecond).
__host__ __device__ inline int quotient(int a, int b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
    int r = a - q * b;
    if (r < 0) --q, r += b;
    if (r >= b) ++q;
    return __builtin_amdgcn_readfirstlane(q);
#else
    return a / b;
#endif
}

// Largest integer whose square is at most x, 0 <= x < 2^30 (uniform over the wavefront).
__host__ __device__ inline int root_of(int x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    int r = __builtin_amdgcn_readfirstlane((int)__builtin_amdgcn_sqrtf((float)x));       // off by one at most
#else
    int r = (int)__builtin_sqrt((double)x);
#endif
    if (r * r > x) --r;
    if ((r + 1) * (r + 1) <= x) ++r;
    return r;
}

// One more worker shortens the longest share, one more partial lengthens the merge, which is a chain.  With few rows
// (up to four row tiles, 16-bit) a lone sequence of U units takes about 0.9 us U / n + 0.03 us n beyond its fixed part
// with n workers per KV head, least near n = sqrt(24 U) .. sqrt(32 U); up to 64 partials are one round of loads and free.
// Measured with 24, us, against one share per compute unit and against splits of at least 256 tokens: 1 KV head, 4 rows,
// bf16, 10K / 20K / 41K tokens 12.5 / 14.2 / 16.1, 14.2 / 17.2 / 18.4, 13.0 / 14.7 / 17.8; 2 heads, 10K 12.9, 14.4, 13.3;
// 16 to 40 in its place: within 2 %.  More rows (1 head, 240 rows, 40K: 21.1 -> 22.1 us) and fp32 (1 head, 5K: 13.0 -> 15.1 us)
// pay more for a stage and are left alone.
constexpr int kMergeUnits = 24, kMergeFree = 64;

__host__ __device__ inline int most_workers(const DealRule &p, int units)
{
    int n = p.round_workers;
    if (p.merge > 0 && n > kMergeFree && units > kMergeFree) n = min(n, max(kMergeFree, root_of(units * p.merge)));
    // more than one round only where a share would outgrow the page list in LDS
    if (units > n * kMaxPieceUnits) n *= quotient(units + n * kMaxPieceUnits - 1, n * kMaxPieceUnits);
    if (units < n * p.min_units) n = max(1, quotient(units, p.min_units));
    return n;
}

__host__ __device__ inline Deal deal_units(const DealRule &p, int units)
{
    int n = min(most_workers(p, units), p.max_workers);
    if (p.merge > 0 && units > n) {                  // no more than the longest share makes necessary: the rest only adds
        const int longest = quotient(units + n - 1, n);      // partials (4 heads, 4 rows, 5K: 64 -> 40 workers, 13.0 -> 12.4 us);
        const int enough = quotient(units + longest - 1, longest);
        if (16 * (n - enough) > n) n = enough;       // one or two fewer are not worth other shares (8 heads, 32K: 32 and 31 alike)
    }
    const int q = quotient(units, n);
    return Deal{n, q, units - q * n};
}
__host__ __device__ inline int deal_begin(const Deal &d, int worker) { return worker * d.q + min(worker, d.r); }
__host__ __device__ inline int deal_worker(const Deal &d, int unit)
{
    const int cut = d.r * (d.q + 1);
    return unit < cut ? quotient(unit, d.q + 1) : d.r + quotient(unit - cut, d.q);
}

__host__ __device__ inline int stages_of(int tokens) { return (tokens + kSplitQuantum - 1) / kSplitQuantum; }
__host__ __device__ inline int seq_units(const DealRule &p, int tokens)
{
    return tokens == 0 ? 0 : stages_of(tokens) + p.seq_extra;
}

}  // namespace owl
