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

__host__ __device__ inline Deal deal_units(const DealRule &p, int units)
{
    // more than one round only where a share would outgrow the page list in LDS
    int n = p.round_workers;
    if (units > n * kMaxPieceUnits) n *= quotient(units + n * kMaxPieceUnits - 1, n * kMaxPieceUnits);
    n = min(n, p.max_workers);
    if (units < n * p.min_units) n = max(1, quotient(units, p.min_units));
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
