// Split-KV pass of the verify-step attention for gfx950 (MI355X).
//
// One workgroup (8 wavefronts, two per SIMD) owns one (KV head, row group, share of
// the K/V): a share is one split of one sequence, or an even run of the whole
// batch's stages that may cross from one sequence into the next (deal_units), and is
// worked through piece by piece, one piece per sequence.  A piece streams its part of
// the paged K/V cache through LDS exactly once and holds, in MFMA accumulators, the un-normalised outputs of
// ALL query rows that share this KV head: rows = (draft node i, query head
// within the group), R = (Hq/Hkv) * N of them, cut into 16-row tiles that are
// dealt out to the wavefronts.  That packing is what makes the cost of
// verifying N drafted tokens "hidden" behind the scan of the context (Sec. 1 /
// Sec. 2 of the paper): the cache is read once whatever N is.
//
// Data movement: K/V go from HBM straight into LDS with 128-bit
// global_load_lds (no VGPR staging), one 16-token page of one tensor per
// wavefront and stage, 64 tokens per stage, in a ring of up to 4 stages (K
// stages in the lower half of the ring, V stages behind them) that is kept
// full ahead of the compute; readiness is tracked with vmcnt and one barrier
// per stage.
//
// Three loops share the ring: the pipelined fast loop (unmasked steps, up to
// two tiles per wave: matrix, vector and LDS work of neighbouring steps woven
// into one instruction stream), the plain fast loop (three tiles per wave, and
// the layout with two key groups: scores -> softmax -> V^T P per step, the two
// waves of a SIMD overlapping each other), and the careful loop (masked or
// ragged steps, exact online softmax; also the fallback when a frozen softmax
// reference overflowed).
//
// Tile algebra (all MFMA tiles are 16x16, wave64):
//   S^T[key][row] = K[key][:] . Q[row][:]        A = K fragment, B = Q fragment
//   O^T[d][row]  += V^T[d][key] * P^T[key][row]  A = V^T fragment, B = P fragment
// With keys along M, a lane owns ONE query row (column lane%16) and the keys of
// a tile sit in its registers, so the fp32 S^T accumulators turn into the bf16
// P^T operand in place.  K/Q take channels 32*kk + 8*quad + e (the order of the
// contraction index is free as long as both operands agree).  V^T fragments
// come from ds_read_b64_tr_b16, the transposing LDS read: in a block of 16
// lanes, lane i receives element i%4 of the 8 bytes addressed by lanes
// 4e + i/4 (e = 0..3); with lane 4e+c pointing at channels 4c..4c+3 of key e,
// lane i ends up with channel i of four keys.  The row sum l rides along as
// one more channel tile whose V^T operand is all ones, so it is summed from the
// very P values (after rounding to bf16) that weigh V.
//
// Visibility (Sec. 3.2.2, Decode Stage): every row sees the whole prefix; among
// the drafts, row (i, .) sees node j iff j is on i's root path, i included.
// Only 32-key steps that reach past the prefix take the masked ("careful") path.
#include <hip/hip_ext.h>

#include <type_traits>

#include "owl_device.h"

namespace owl {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

constexpr int kThreads = 512;        // 8 wavefronts
constexpr int kWaves = kThreads / 64;
constexpr float kMInit = -1.0e30f;   // "no key seen yet"; finite so that m - m is 0
constexpr float kGuardRoom = 11.0f;  // fp16: how far a score may lie above a guarded reference (2^16 is the limit)

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <typename T>
__device__ __forceinline__ f32x4 mfma16(const uint4 &a, const uint4 &b, const f32x4 &c)
{
    if constexpr (std::is_same<T, __bf16>::value)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

template <typename T>
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    f32x2 v = {lo, hi};
    if constexpr (std::is_same<T, __bf16>::value)
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    else
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

template <typename T>
__device__ __forceinline__ uint32_t ones2()
{
    return std::is_same<T, __bf16>::value ? 0x3F803F80u : 0x3C003C00u;
}

// 16 bytes per lane from global memory straight into LDS: lane l's data lands
// at lds_addr + 16*l.  lds_addr must be uniform over the wavefront.  K and V are
// read exactly once, so their transfers are marked non-temporal (`nt`): the lines are
// not kept in L2 or the memory-side cache, which leaves those to the queries, the
// page lists and the partials, and makes the 32K chain step 10 % shorter (the
// 128K tree step 2.5 %); the scope bits of the instruction make no difference.
#define OWL_DMA_POLICY " nt"
template <bool kOnce>
__device__ __forceinline__ void dma16(const void *gptr, uint32_t lds_addr)
{
    if constexpr (kOnce)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" OWL_DMA_POLICY "\n"
                     :
                     : "s"(lds_addr), "v"(gptr)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off\n"
                     :
                     : "s"(lds_addr), "v"(gptr)
                     : "memory", "m0");
}

// The same with a wave-uniform 64-bit base and a 32-bit per-lane byte offset.
__device__ __forceinline__ void dma16s(uint64_t sbase, uint32_t voff, uint32_t lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" OWL_DMA_POLICY "\n"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(sbase)
                 : "memory", "m0");
}

// Wait until at most N of this wavefront's vector-memory loads are in flight.
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Transposing 64-bit LDS read (see the file comment for the lane mapping).
__device__ __forceinline__ uint2 lds_read_tr16(const unsigned char *p)
{
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (s16x4 __attribute__((address_space(3))) *)(p));
    return __builtin_bit_cast(uint2, v);
}

// f(integral_constant<int, B>) ... f(integral_constant<int, E-1>), unrolled at compile time.
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(f);
    }
}

// Geometry of one instantiation.
template <typename T, int D, int TPW, int WR, int WK>
struct Geo {
    static constexpr bool kF32 = std::is_same<T, float>::value;
    static constexpr int ES = sizeof(T);
    static constexpr int KSTEPS = 2;                    // 32-key steps per stage
    static constexpr int SK = 32 * KSTEPS;              // keys per stage: 4 pages x 2 tensors = 8 waves
    static constexpr int ROWB = D * ES;                 // bytes of one key row
    static constexpr int PPR = ROWB / 16;               // 16-byte pieces per row
    static constexpr int RPI = 1024 / ROWB;             // key rows per DMA instruction
    static constexpr int LPS = kPage / RPI;             // DMA instructions per wave and stage
    static constexpr int NT = D / 16;                   // channel tiles of O^T
    static constexpr int STAGE = SK * ROWB;             // bytes per tensor per stage
    static constexpr int NS = (8 * STAGE <= 131072) ? 4 : ((6 * STAGE <= 131072) ? 3 : 2);
    static constexpr int VREG = NS * STAGE;             // LDS ring: K stages at [0, VREG), V stages behind them
    static constexpr int QREGS = kF32 ? D / 4 : D / 32; // Q fragment slots per tile
    static constexpr int KSWZ = (PPR - 1) & 15;         // K rows: piece ^= key & KSWZ
    static constexpr int VSWM = PPR >= 16 ? 7 : PPR / 2 - 1;   // V rows: piece ^= (key & VSWM) << 1
    static constexpr size_t PAGES = (size_t)NS * 2 * STAGE;           // behind the ring: page list, ancestor sets, parents, votes
    static constexpr size_t ANC = PAGES + kMaxPiecePages * 4, PARENT = ANC + 64 * 8, ANY = PARENT + 64 * 4;
    static constexpr size_t LDS = ANY + 2 * kWaves * 4;
    static_assert(WR * WK == kWaves && (WK == 1 || WK == 2), "eight wavefronts per workgroup");
    static_assert(NS * LPS < 64, "loads in flight must fit vmcnt");
    static_assert((WK - 1) * WR * TPW * (NT * 1024 + 512) <= NS * 2 * STAGE,
                  "cross-wave merge buffer must fit in the stage ring");
};

// One piece of work: the stages of sequence b between two token positions.
struct Piece {
    int b, L, Nb;                                    // sequence, its prefix length and number of drafts
    int pos0, pos1;                                  // [pos0, pos1) of its L + Nb cached rows, pos0 a multiple of 64
    size_t slot;                                     // where the partials of row tile 0 go
};

// This lane's number in its wavefront.  Formed anew in each piece (kAnew) it is not kept across the pieces of a share, where
// the loops of some kernels leave no register for it: in the three-tile kernel it went to scratch memory, and every reload
// between the requests of the first stages waited for all of them (128K hybrid, 320 rows 167.5 us against 172.3 with the
// number kept, 8 sequences of 500-3K 39.0 against 47.7; fp32, head_dim 128, 512 tokens 13.6 against 16.3).  With one tile of 16
// bits and two key groups there is room, and what follows from the number is then not derived again in the loop (320 rows, 1 head,
// 10K tokens, in row groups 14.39 us anew, 14.22 kept; 160 rows 12.98 and 12.82).  With one tile and the pipelined loop keeping it loses in
// batches, more the more pieces a share has (96 rows, 8 sequences of 1K-6.4K 18.5 us anew, 19.3 kept; 116 rows, 8 of 1.2K-2.5K 24.4
// and 25.0; fp16, 100 rows, 16 of 700-2K 21.5 and 21.7).  Two tiles: within 1 % either way.
template <bool kAnew>
__device__ __forceinline__ int lane_number()
{
    if constexpr (!kAnew) return threadIdx.x & 63;
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// Page-table entries first + tid and first + kThreads + tid of the window of sequence b that begins at pos0 (no branch: an
// entry past the table re-reads its last one and is not used).
struct PagePair {
    int page[2];
};

__device__ __forceinline__ PagePair load_pages(const KParams &p, int tid, int b, int pos0, int first)
{
    PagePair pg;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const int lp = pos0 / kPage + first + tid + r * kThreads;
        pg.page[r] = p.page_table ? p.page_table[(int64_t)b * p.max_pages + min(lp, p.max_pages - 1)] : lp;
    }
    return pg;
}

// What was asked for before the length that decides about the window was known: the parents of the sequence, and the first
// entries of the page list from token pos0 on (pos0 < 0: none).  They wait in registers for the set-up of the piece, which
// asks for the rest meanwhile; the three-tile kernel, which has none to spare across its loops, puts them in LDS at once
// (`kept` entries, as far as this wavefront's own go all of them pages of the pool).
struct Ahead {
    int pos0, kept;
    bool parents;
    PagePair pages;
    int parent;
};

// The kernel's arguments for one piece.  In fp16, whose second (guarded) loop takes more scalar registers, they are read
// again from the kernel-argument segment: kept across the pieces they made 36-79 scalar registers spill (3-16 so) and
// cost a call of 3K-7K tokens 0.2-0.4 us of 11-13 (head_dim 64, 8 KV heads, 4 rows, 3K: 11.5 -> 11.1 us).  The bf16
// kernels spill 21-58 and lose by reading again (16 sequences of 8K-64K, 104 rows: 452 -> 457 us).
template <typename T>
__device__ __forceinline__ const KParams &piece_args(const KParams &launch_args)
{
    if constexpr (std::is_same<T, _Float16>::value) {
        typedef const __attribute__((address_space(4))) KParams KernelArgs;
        KernelArgs *args = (KernelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(args));
        return *(const KParams *)args;
    } else {
        return launch_args;
    }
}

// Whether `v` holds in any thread of the workgroup; `words`: kWaves words of LDS that nothing else uses for the piece.
__device__ __forceinline__ bool workgroup_any(bool v, int wave, int lane, int32_t *words)
{
    const int any = __builtin_amdgcn_ballot_w64(v) != 0;
    if (lane == 0) words[wave] = any;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) all |= words[w];
    return __builtin_amdgcn_readfirstlane(all) != 0;
}

template <typename T, int D, int TPW, int WR, int WK, typename Stamp>
__device__ __forceinline__ void run_piece(const KParams &launch_args, unsigned char *smem, int wave, int g, int rg, const Piece &pc,
                                          const Ahead &ahead, Stamp &&stamp)
{
    using GEO = Geo<T, D, TPW, WR, WK>;
    constexpr bool kF32 = GEO::kF32;
    constexpr int ES = GEO::ES, KSTEPS = GEO::KSTEPS, SK = GEO::SK, ROWB = GEO::ROWB;
    constexpr int PPR = GEO::PPR, NT = GEO::NT, STAGE = GEO::STAGE, NS = GEO::NS;
    constexpr int RPI = GEO::RPI, LPS = GEO::LPS, QREGS = GEO::QREGS;
    constexpr int KSWZ = GEO::KSWZ, VSWM = GEO::VSWM, VREG = GEO::VREG;
    constexpr int KQ = kF32 ? 1 : QREGS;             // K/Q fragment slots of the 16-bit paths

    int32_t *s_pages = reinterpret_cast<int32_t *>(smem + GEO::PAGES);
    uint64_t *s_anc = reinterpret_cast<uint64_t *>(smem + GEO::ANC);
    int32_t *s_parent = reinterpret_cast<int32_t *>(smem + GEO::PARENT);
    int32_t *s_any = reinterpret_cast<int32_t *>(smem + GEO::ANY);
    const uint32_t lds0 =
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;

    // What follows from the thread's number and the KV head is derived once per piece: kept across the
    // pieces of a share (as the compiler would by itself) it does not fit the registers of the loops.
    const KParams &p = piece_args<T>(launch_args);
    asm volatile("" : "+s"(g), "+s"(rg), "+s"(wave));
    const int lane = lane_number<(TPW > 1) || WK == 1>(), tid = wave * 64 + lane;
    const int wr = wave % WR, wk = wave / WR;
    const int j = lane & 15, qd = lane >> 4;

    const int b = pc.b, L = pc.L, Nb = pc.Nb, pos0 = pc.pos0, pos1 = pc.pos1, Ttot = L + Nb;
    const int nstages = (pos1 - pos0 + SK - 1) / SK;
    const bool has_drafts = pos1 > L;               // uniform over the workgroup

    // ---- set-up: page list, parents and query rows are requested together, one memory round trip ----
    const int npg = (pos1 - pos0 + kPage - 1) / kPage;
    constexpr bool kKeptEarly = TPW == 3;
    const bool have = ahead.pos0 == pos0 && (!kKeptEarly || npg <= ahead.kept);      // uniform over the wavefront
    PagePair pages{};
    if (!have) pages = load_pages(p, tid, b, pos0, 0);
    else if (!kKeptEarly) pages = ahead.pages;
    int parent = kKeptEarly ? 0 : ahead.parent;
    if (has_drafts && !ahead.parents) parent = p.parent[(int64_t)b * p.N + min(tid, p.N - 1)];
    // ---- this wave's query rows: tiles wr, wr + WR, ... of the row group ----
    // Row `row` belongs to node row / G; the quotient is exact: rows stay below 2^12, where the error of
    // the product is far below the half that is added.
    int heads = p.G;
    asm volatile("" : "+s"(heads));
    const float inv_g = __builtin_amdgcn_rcpf((float)heads);
    auto node_of = [&](int row) -> int { return (int)(((float)row + 0.5f) * inv_g); };
    const unsigned char *q_head = static_cast<const unsigned char *>(p.q) + ((int64_t)b * p.N * p.Hq + (int64_t)g * p.G) * D * ES;
    auto row_offset = [&](int row) -> int64_t { return ((int64_t)node_of(row) * (p.Hq - p.G) + row) * ROWB; };
    uint4 qf[TPW][KQ];
    float qs[TPW][kF32 ? QREGS : 1];
    int irow[TPW];
    int my_nt = 0;
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        const int tg = rg * p.group_tiles + t * WR + wr;
        const bool tile_ok = t * WR + wr < p.group_tiles && tg < p.RT;
        my_nt += tile_ok ? 1 : 0;
        const int row = tg * kRowTile + j, i = node_of(row);
        irow[t] = tile_ok && row < p.R && i < Nb ? i : -1;
        if constexpr (kF32) {
            const float4 *qp = reinterpret_cast<const float4 *>(q_head + row_offset(min(row, p.R - 1)));
#pragma unroll
            for (int c = 0; c < QREGS / 4; ++c) {            // (the channels that a quad of lanes takes, see careful_step)
                const float4 x = qp[4 * c + qd];
                const bool on = irow[t] >= 0;
                qs[t][4 * c] = on ? x.x : 0.f;
                qs[t][4 * c + 1] = on ? x.y : 0.f;
                qs[t][4 * c + 2] = on ? x.z : 0.f;
                qs[t][4 * c + 3] = on ? x.w : 0.f;
            }
        }
    }

    auto keep_pages = [&](const PagePair &from, int first) {
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const int idx = first + tid + r * kThreads;
            int pg = from.page[r];
            if (idx >= npg) continue;
            if (pg < 0 || pg >= p.n_pool_pages || (p.page_table && pos0 / kPage + idx >= p.max_pages)) {
                flag_status(p.dev_status, OWL_DEV_BAD_PAGE);
                pg = 0;
            }
            s_pages[idx] = pg;
        }
    };
    if (!kKeptEarly || !have) keep_pages(pages, 0);
    for (int first = 2 * kThreads; first < npg; first += 2 * kThreads)           // more than 16K tokens in one piece
        keep_pages(load_pages(p, tid, b, pos0, first), first);
    if (has_drafts && !(kKeptEarly && ahead.parents) && tid < p.N) s_parent[tid] = parent;
    if (std::is_same<T, _Float16>::value && tid < 2) s_any[tid] = 0;
    __syncthreads();
    stamp(1);

    // ---- stage issue ----
    // Wave w brings one 16-token page of one tensor per stage: tensor w/4 (K, V),
    // page 4*s + w%4 of the split.  Lane l of DMA instruction `it` carries piece
    // l % PPR of slot it*RPI + l / PPR.  The 16-byte pieces of a row are stored
    // XOR-permuted by the slot number (K: piece ^ slot, V: piece ^ 2*(slot%8)) so
    // that the fragment reads below are bank-conflict free; the permutation is
    // applied to the global address, the LDS side of the transfer is always
    // lane-linear.  Slots past the end of the split (ragged last stage only)
    // re-read the last valid row: finite data whose scores are masked out later.
    const int ld_tensor = wave >> 2, ld_page = wave & 3;
    const unsigned char *ld_base = static_cast<const unsigned char *>(ld_tensor ? p.v : p.k);
    const int last_pgx = (pos1 - 1 - pos0) >> 4, last_slot = (pos1 - 1) & (kPage - 1);
    const int ld_piece = lane % PPR, ld_row = lane / PPR;
    const int64_t head_off = (int64_t)g * p.stride_head * ES;
    const int64_t tok_bytes = p.stride_token * ES;
    // (Held in their registers: fp16's arguments are in memory, and left to the compiler every stage of its loops loaded the
    // stride again, every masked step the scale, and waited for it, and with it for all LDS reads under way.)
    int64_t page_bytes = p.stride_page * ES;
    float c_log2 = p.c_log2;
    if constexpr (std::is_same<T, _Float16>::value) asm volatile("" : "+s"(page_bytes), "+s"(c_log2));

    // A whole page (every stage but the split's last page) needs no clamping:
    // the lane's byte offsets inside the page are fixed, only the page base
    // (wave-uniform, kept in scalar registers) changes from stage to stage.
    constexpr bool kKeepLdOff = TPW <= 2;            // three tiles per wave: no registers to spare, recompute
    auto ld_off_of = [&](int it) -> uint32_t {
        const int row = it * RPI + ld_row;
        const int swz = ld_tensor ? ((row & VSWM) << 1) : (row & KSWZ);
        return (uint32_t)(row * tok_bytes) + (uint32_t)((ld_piece ^ swz) << 4);
    };
    uint32_t ld_off[LPS];
#pragma unroll
    for (int it = 0; it < LPS; ++it) ld_off[it] = kKeepLdOff ? ld_off_of(it) : 0u;
    const bool ld_off_ok = tok_bytes * kPage < ((int64_t)1 << 31);
    const uint32_t ld_lds = lds0 + ld_tensor * VREG + ld_page * kPage * ROWB;

    // page id of this wave's page of stage s (to be handed to issue_stage; reading it
    // ahead of the stage barrier takes the LDS round trip off the issue path)
    auto stage_page = [&](int s) -> int { return s_pages[min(s * (SK / kPage) + ld_page, last_pgx)]; };
    auto issue_stage_pg = [&](int s, int pg_lane) {
        const int buf = s % NS;
        const int pgx_raw = s * (SK / kPage) + ld_page;
        const uint32_t lds_dst = ld_lds + buf * STAGE;
        if (pgx_raw < last_pgx && ld_off_ok) {           // uniform over the wave
            const int64_t pg = __builtin_amdgcn_readfirstlane(pg_lane);
            const uint64_t sb = (uint64_t)(uintptr_t)ld_base + (uint64_t)(pg * page_bytes + head_off);
            const uint64_t sbase = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(sb >> 32)) << 32) |
                                   (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sb);
#pragma unroll
            for (int it = 0; it < LPS; ++it)
                dma16s(sbase, kKeepLdOff ? ld_off[it] : ld_off_of(it),
                       __builtin_amdgcn_readfirstlane(lds_dst + it * RPI * ROWB));
            return;
        }
        const int slot_max = pgx_raw >= last_pgx ? last_slot : kPage - 1;
        const int64_t base = (int64_t)pg_lane * page_bytes + head_off;
#pragma unroll
        for (int it = 0; it < LPS; ++it) {
            const int row = it * RPI + ld_row;
            const int64_t off = base + min(row, slot_max) * tok_bytes;
            const int swz = ld_tensor ? ((row & VSWM) << 1) : (row & KSWZ);
            dma16<true>(ld_base + off + ((ld_piece ^ swz) << 4),
                  __builtin_amdgcn_readfirstlane(lds_dst + it * RPI * ROWB));
        }
    };
    auto issue_stage = [&](int s) { issue_stage_pg(s, stage_page(s)); };

    // The query rows travel like K pages: by DMA, 16 bytes a lane, rows contiguous, into the last TPW ring
    // slots (one tile of every wavefront each), before the stages that belong there are requested; from
    // there each wavefront picks its own fragments.  (Loaded straight into registers they took 2 us for
    // 20 row tiles, as 64-byte pieces of 16 rows per instruction, and the compiler, which does not see the
    // ring's transfers in the wait counter, drained the whole ring before it used them.)
    constexpr int kQSlot0 = NS - TPW;                // first ring slot the queries occupy
    auto q_lds = [&](int t) -> uint32_t {            // offset of this wavefront's tile t in the ring
        return (uint32_t)((kQSlot0 + t) * STAGE + (wave & 3) * (kPage * ROWB) + (wave >> 2) * VREG);
    };
    // Every worker of a head reads the same rows, so they stay in the caches, except where one worker takes the whole
    // sequence (non-temporal against cached, us: 24 rows, 8 heads, 5K tokens 14.0 -> 13.2, 320 rows, 1 head, 10K 15.3 -> 14.3,
    // 104 rows, 8 heads, 64K 55.0 -> 54.0; but 512 sequences of 125-500 tokens, 104 rows, 440 -> 448).  With three tiles a
    // wavefront, whose registers are all taken, both the choice and the cached form cost more (320 rows, 64 sequences of
    // 250-1000 tokens: 125.5 us, 131.4 with the choice, 128.4 cached; one of 128K 170-173 in every form).
    auto issue_queries = [&]() {
        const bool once = TPW == 3 || (pos0 == 0 && pos1 == Ttot);
        if constexpr (!kF32) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                const int row0 = (rg * p.group_tiles + t * WR + wr) * kRowTile;
#pragma unroll
                for (int it = 0; it < LPS; ++it) {
                    const int slot = it * RPI + ld_row;
                    const unsigned char *src = q_head + row_offset(min(row0 + slot, p.R - 1)) + ((ld_piece ^ (slot & KSWZ)) << 4);
                    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + q_lds(t) + it * RPI * ROWB);
                    if (once) dma16<true>(src, dst);
                    else dma16<false>(src, dst);
                }
            }
        }
    };
    auto take_queries = [&]() {
        if constexpr (!kF32) {
#pragma unroll
            for (int t = 0; t < TPW; ++t)
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    const uint4 x = *reinterpret_cast<const uint4 *>(smem + q_lds(t) + j * ROWB + (((4 * kk + qd) ^ (j & KSWZ)) << 4));
                    qf[t][kk] = irow[t] >= 0 ? x : make_uint4(0, 0, 0, 0);
                }
        }
    };
    static_assert(kF32 || (TPW < NS && 4 * kPage * ROWB == STAGE), "the queries leave at least one ring slot to the first stage");

    f32x4 O[TPW][NT + 1];
    float m[TPW];
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
        m[t] = kMInit;
#pragma unroll
        for (int u = 0; u <= NT; ++u) O[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    // ---- lane-constant parts of the fragment addresses (16-bit types) ----
    // K fragment (kt, kk): 16 bytes at key kt*16 + j, piece (4*kk + quad) ^ (j & KSWZ).
    // V^T fragment (u, h): transposing read; lane 4e + c of block `quad` points at
    // key 16*h + 4*quad + e, channels 16*u + 4*c .. +3.
    const int v_e = j >> 2, v_c = j & 3;
    const int v_key0 = 4 * qd + v_e;
    const int v_swz = (v_key0 & VSWM) << 1;
    const int v_lane_off = v_key0 * ROWB + (v_c & 1) * 8;

    // ---- K fragments of one 32-key step ----
    auto load_k_frags = [&](const unsigned char *Kb, uint4 (&kf)[2][KQ]) {
        if constexpr (!kF32) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                const int key = kt * 16 + j;
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk)
                    kf[kt][kk] = *reinterpret_cast<const uint4 *>(
                        Kb + key * ROWB + (((4 * kk + qd) ^ (key & KSWZ)) << 4));
            }
        }
    };
    // ---- V^T fragment of channel tile u for the 32 keys of a step ----
    auto load_v_frag = [&](const unsigned char *Vb, int u) -> uint4 {
        const unsigned char *a = Vb + v_lane_off + ((((2 * u) ^ v_swz) | (v_c >> 1)) << 4);
        const uint2 lo = lds_read_tr16(a);
        const uint2 hi = lds_read_tr16(a + 16 * ROWB);
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };

    // ---- fast step: no mask, fixed reference m, accumulators touched by MFMA only ----
    // fp16 storage: a frozen reference that overflows shows in the row sums.  The loops look for it at a few stages (see
    // `watched`) and give way to the plain loop with a guarded reference (see fast_sx).
    constexpr bool kGuard = std::is_same<T, _Float16>::value;
    constexpr bool kExactRedo = kGuard && TPW == 1 && WK == 2;       // see the passes
    // p = 2^(x - m) is exact in relative terms whatever m is; with m frozen at
    // the first step's row maximum, p overflows only if a later score exceeds
    // it by more than ~100 (log2 units), which the row sum exposes afterwards.
    // A step is cut in two: scores + softmax -> P (fast_sx), and O += V^T P with
    // the V^T fragments already in registers (fast_pv), so that the stage loop
    // can put a barrier between them.
    auto fast_sx = [&](const unsigned char *Kb, const unsigned char *Vb, uint4 (&pf)[TPW], uint4 (&vf)[NT],
                       auto ntag, auto gtag, [[maybe_unused]] float room) {
        constexpr int NA = decltype(ntag)::value;    // tiles this wave really owns
        constexpr bool kGuarded = decltype(gtag)::value;
        // One tile a wavefront: half of the V^T fragments are asked for behind the scores, so that they arrive while P is
        // formed; the fence keeps the compiler from gathering all of them behind P, which only the exponentials may pass.  us, all
        // behind P -> half before it: 408 rows, 1 head, 52K / 70K tokens 27.7 -> 27.0 / 33.2 -> 32.3, 496 rows, 60K 30.2 -> 29.5, 240 rows,
        // 8 heads, 5K 17.1 -> 16.9; up to 64 rows and 8 heads within 0.2 %.  (All of them before it: 33.2 -> 33.1, and 64 rows 0.5 %
        // longer.  fp16 with the frozen reference: 7K 20.5 -> 20.4.)
        constexpr bool kEarlyV = TPW == 1 && !kGuarded;
        if constexpr (!kF32 && NA > 0) {
            // The score -> softmax -> P chain is the latency-critical part of a step; O += V^T P
            // is throughput work without dependents.  Raising this wave's priority for the
            // first and dropping it for the second lets the other wave of the SIMD fill the
            // gaps of the chain with its PV MFMAs (13 % fewer cycles in the three-tile loop).
            __builtin_amdgcn_s_setprio(1);
            uint4 kf[2][KQ];
            load_k_frags(Kb, kf);
#pragma unroll
            for (int t = 0; t < NA; ++t) {
                f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    s0 = mfma16<T>(kf[0][kk], qf[t][kk], s0);
                    s1 = mfma16<T>(kf[1][kk], qf[t][kk], s1);
                }
                if constexpr (kEarlyV) {
#pragma unroll
                    for (int u = 0; u < NT / 2; ++u) vf[u] = load_v_frag(Vb, u);
                    __builtin_amdgcn_sched_barrier(0x400);
                }
                if constexpr (kGuarded) {
                    // The reference stays until a score lies more than `room` above it.  The row then moves it to
                    // its highest score, as the exact loop does, and rescales its accumulators (rare; uniform branch).
                    // Not above that: fp16 has nothing below 2^-25, and the many small weights would pay for the
                    // head room (one score 20.5 above the rest of 16K: error 9e-6, with 4 of head room 7e-4).
                    const float tm = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
                                           fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
                    // detection needs no cross-lane step: any lane's own keys can raise the alarm
                    if (__builtin_amdgcn_ballot_w64(__builtin_fmaf(tm, c_log2, -m[t]) > room) != 0) {
                        const float sc = quad_column_max(tm) * c_log2;
                        const float mn = sc > m[t] + room ? sc : m[t];
                        const float alpha = fast_exp2(m[t] - mn);
                        m[t] = mn;
#pragma unroll
                        for (int u = 0; u <= NT; ++u) O[t][u] *= alpha;
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s0[r] = fast_exp2(__builtin_fmaf(s0[r], c_log2, -m[t]));
                    s1[r] = fast_exp2(__builtin_fmaf(s1[r], c_log2, -m[t]));
                }
                pf[t].x = pack2<T>(s0[0], s0[1]);
                pf[t].y = pack2<T>(s0[2], s0[3]);
                pf[t].z = pack2<T>(s1[0], s1[1]);
                pf[t].w = pack2<T>(s1[2], s1[3]);
            }
#pragma unroll
            for (int u = kEarlyV ? NT / 2 : 0; u < NT; ++u) vf[u] = load_v_frag(Vb, u);
        }
    };
    auto fast_pv = [&](const uint4 (&pf)[TPW], const uint4 (&vf)[NT], auto ntag) {
        constexpr int NA = decltype(ntag)::value;
        if constexpr (!kF32 && NA > 0) {
            __builtin_amdgcn_s_setprio(0);
            const uint4 ones = make_uint4(ones2<T>(), ones2<T>(), ones2<T>(), ones2<T>());
#pragma unroll
            for (int u = 0; u < NT; ++u) {
#pragma unroll
                for (int t = 0; t < NA; ++t) O[t][u] = mfma16<T>(vf[u], pf[t], O[t][u]);
            }
#pragma unroll
            for (int t = 0; t < NA; ++t) O[t][NT] = mfma16<T>(ones, pf[t], O[t][NT]);
        }
    };

    // ---- pipelined fast loop (WK == 1, up to two tiles per wave) ----
    // Iteration i runs three mutually independent instruction streams over
    // 32-key steps: the matrix stream does O += V^T P of step i-1 and the
    // scores of step i+1, the vector stream turns the scores of step i into P
    // (fma, exp2, pack), and the LDS stream fetches each K / V^T fragment PF
    // MFMA groups before its use (one group = one fragment's MFMAs for all tiles
    // of the wave).  The streams are woven together group by group, with a
    // scheduling fence after every group so that the order written here is the
    // order issued: a wave can issue only one instruction every few cycles, so
    // what keeps the matrix pipe busy is a short, evenly mixed stream per wave.
    // Ring offsets are compile-time (the stage loop is unrolled over the ring)
    // and travel in the LDS instructions' offset fields: no address arithmetic
    // is left in the loop.
    constexpr bool kPipe = !kF32 && WK == 1 && TPW <= 2;      // three tiles: not enough registers
    constexpr int PF = 3;                                      // fragment prefetch distance (groups, <= NT)
    uint32_t k_off[KQ], v_off[NT];
    if constexpr (kPipe) {
#pragma unroll
        for (int kk = 0; kk < KQ; ++kk) k_off[kk] = j * ROWB + (((4 * kk + qd) ^ (j & KSWZ)) << 4);
#pragma unroll
        for (int u = 0; u < NT; ++u) v_off[u] = VREG + v_lane_off + ((((2 * u) ^ v_swz) | (v_c >> 1)) << 4);
    }
    // V^T fragment of channel tile u / K fragment (kt, kk) at ring offset `off` (bytes, compile-time)
    auto pipe_v = [&](auto off, auto uu) -> uint4 {
        constexpr uint32_t C = decltype(off)::value;
        const unsigned char *a = smem + v_off[decltype(uu)::value];
        const uint2 lo = lds_read_tr16(a + C);
        const uint2 hi = lds_read_tr16(a + (C + 16 * ROWB));
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    };
    auto pipe_k = [&](auto off, auto ktt, auto kkk) -> uint4 {
        constexpr uint32_t C = decltype(off)::value + decltype(ktt)::value * 16 * ROWB;
        return *reinterpret_cast<const uint4 *>(smem + k_off[decltype(kkk)::value] + C);
    };
    // vprev / knext / vnext: ring offsets of V of step i-1, K of step i+1, V of step i
    auto pipe_iter = [&](f32x4 (&Sc)[TPW][2], f32x4 (&Sn)[TPW][2], const uint4 (&Pp)[TPW], uint4 (&Pc)[TPW],
                         uint4 (&vpre)[PF], auto vprev, auto knext, auto vnext, auto haspv, auto ntag) {
        constexpr int NA = decltype(ntag)::value;
        constexpr bool kPV = decltype(haspv)::value;
        if constexpr (kPipe && NA > 0) {
            constexpr int G = NT + 1 + 2 * KQ;           // MFMA groups: PV tiles, row sum, score fragments
            constexpr int NV = NA * 8;                   // scores per lane
            const uint4 ones = make_uint4(ones2<T>(), ones2<T>(), ones2<T>(), ones2<T>());
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            uint4 fr[G];
            if constexpr (kPV) static_for<0, PF>([&](auto uu) { fr[decltype(uu)::value] = vpre[decltype(uu)::value]; });
            static_for<0, G>([&](auto nn) {
                constexpr int n = decltype(nn)::value;
                // first half of an iteration (PV groups + the bulk of the exponentials) above the
                // other wave of the SIMD, second half below it: 2-3 % fewer cycles than equal priority
                if constexpr (n == 0) __builtin_amdgcn_s_setprio(1);
                if constexpr (n == NT + 1) __builtin_amdgcn_s_setprio(0);
                // LDS stream
                constexpr int pn = n + PF;
                if constexpr (pn < NT) {
                    if constexpr (kPV) fr[pn] = pipe_v(vprev, std::integral_constant<int, pn>{});
                } else if constexpr (pn > NT && pn < G) {
                    fr[pn] = pipe_k(knext, std::integral_constant<int, (pn - NT - 1) & 1>{},
                                    std::integral_constant<int, ((pn - NT - 1) >> 1)>{});
                } else if constexpr (pn >= G) {
                    vpre[pn - G] = pipe_v(vnext, std::integral_constant<int, pn - G>{});
                }
                if constexpr (!kPV && n == 0) {          // the first PF score fragments, not prefetched by anyone
                    static_for<NT + 1, (NT + 1 + PF < G ? NT + 1 + PF : G)>([&](auto gg) {
                        constexpr int g2 = decltype(gg)::value;
                        fr[g2] = pipe_k(knext, std::integral_constant<int, (g2 - NT - 1) & 1>{},
                                        std::integral_constant<int, ((g2 - NT - 1) >> 1)>{});
                    });
                }
                // matrix stream
                static_for<0, NA>([&](auto tt) {
                    constexpr int t = decltype(tt)::value;
                    if constexpr (n < NT) {
                        if constexpr (kPV) O[t][n] = mfma16<T>(fr[n], Pp[t], O[t][n]);
                    } else if constexpr (n == NT) {
                        if constexpr (kPV) O[t][NT] = mfma16<T>(ones, Pp[t], O[t][NT]);
                    } else {
                        constexpr int kt = (n - NT - 1) & 1, kk = (n - NT - 1) >> 1;
                        if constexpr (kk == 0) Sn[t][kt] = mfma16<T>(fr[n], qf[t][kk], zero);
                        else Sn[t][kt] = mfma16<T>(fr[n], qf[t][kk], Sn[t][kt]);
                    }
                });
                // vector stream: scores [done1, done2) in this group, packs of the scores of the group before
                constexpr int done0 = n >= 2 ? ((n - 1) * NV / (G - 1) < NV ? (n - 1) * NV / (G - 1) : NV) : 0;
                constexpr int done1 = n >= 1 ? (n * NV / (G - 1) < NV ? n * NV / (G - 1) : NV) : 0;
                constexpr int done2 = (n + 1) * NV / (G - 1) < NV ? (n + 1) * NV / (G - 1) : NV;
                static_for<done1, done2>([&](auto ii) {
                    constexpr int idx = decltype(ii)::value;
                    constexpr int t = idx >> 3, kt = (idx >> 2) & 1, r = idx & 3;
                    float e = fast_exp2(__builtin_fmaf(Sc[t][kt][r], c_log2, -m[t]));
                    asm volatile("" : "+v"(e));          // pins the computation of the value to this group
                    Sc[t][kt][r] = e;
                });
                static_for<done0 / 2, done1 / 2>([&](auto cc) {
                    constexpr int cidx = decltype(cc)::value;
                    constexpr int t = cidx >> 2, kt = (cidx >> 1) & 1, h = cidx & 1;
                    uint32_t w = pack2<T>(Sc[t][kt][2 * h], Sc[t][kt][2 * h + 1]);
                    asm volatile("" : "+v"(w));
                    if constexpr (kt == 0 && h == 0) Pc[t].x = w;
                    else if constexpr (kt == 0) Pc[t].y = w;
                    else if constexpr (h == 0) Pc[t].z = w;
                    else Pc[t].w = w;
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        }
    };

    // ---- fp16 only: is the frozen reference good? ----
    // A wavefront that finds it is not raises an alarm, which all read behind a later barrier.  It looks
    //   before the loops        if the scores of its first step span more than 2^14 in some lane (ten standard deviations of
    //                           the scores of unit-variance inputs: a long tail, and a later score is likely to pass the head
    //                           room above the first step's maximum); in the pipelined loop, also at those of the second
    //   at stages 4, 16, 64...  of a frozen loop, behind the barrier, if a row sum has overflowed (three tiles a wavefront: at
    //                           stage 1 too, whose plain loop has seen 32 keys by then)
    // and what the last look misses the check behind the loops finds.  Looks lie two barriers apart or more, the plain loops
    // have none at stage 0, and there is one word for before the loops and one for within: no wavefront writes a word that
    // another may still have to read.  Before, every piece formed the scores of its first one to three stages twice to measure
    // their spread, and every overflow was redone with the exact loop.  us, 8 heads: 24 rows, 2.5K tokens 10.8 -> 10.5, 64 rows,
    // 20K 24.8 -> 21.6, 240 rows, 5K / 20K 18.0 -> 17.9 / 34.9 -> 34.1, four sequences of 900-9K 35.0 -> 33.2.  (Looks at 8, 32,
    // ... as well: 240 rows, 5K 17.9 -> 18.0; 320 rows, 64K with one key in twenty eight times as long 107.8, without the look at
    // stage 1 112.8.)
    auto alarm = [&](bool bad, int word) {
        if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) s_any[word] = 1;
    };
    auto alarmed = [&](int word) -> bool { return __builtin_amdgcn_readfirstlane(s_any[word]) != 0; };
    auto watch_sums = [&]() {
        bool bad = false;
#pragma unroll
        for (int t = 0; t < TPW; ++t) bad |= !(O[t][NT][0] < 1.0e30f);
        alarm(bad, 1);
    };
    auto watched = [](int s) {                       // 0, 4, 16, 64, ..., and 1 with three tiles a wavefront
        return (s & (s - 1)) == 0 && (s & (TPW > 2 ? 0x2AAAAAAA : 0x2AAAAAAB)) == 0;
    };
    auto is_wide = [&](const f32x4 &s0, const f32x4 &s1, float high) {
        const float low = fminf(fminf(fminf(s0[0], s0[1]), fminf(s0[2], s0[3])),
                                fminf(fminf(s1[0], s1[1]), fminf(s1[2], s1[3])));
        return (high - low) * c_log2 > 14.0f;
    };
    auto highest = [](const f32x4 &s0, const f32x4 &s1) {
        return fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
    };

    // ---- reference m of every row tile from one unmasked step (before the fast loop) ----
    auto init_reference = [&](int buf, int ks, [[maybe_unused]] float head_room, f32x4 (&keep)[TPW][2]) {
        if constexpr (!kF32) {
            // (Formed here: as an address that the compiler kept from before the stages were requested, it came back from
            // scratch memory in the three-tile kernel, and the wait for it drained the whole ring before the first step.)
            int off = buf * STAGE + ks * 32 * ROWB;
            asm volatile("" : "+s"(off));
            const unsigned char *Kb = smem + off;
            uint4 kf[2][KQ];
            load_k_frags(Kb, kf);
            bool wide = false;
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    s0 = mfma16<T>(kf[0][kk], qf[t][kk], s0);
                    s1 = mfma16<T>(kf[1][kk], qf[t][kk], s1);
                }
                keep[t][0] = s0;
                keep[t][1] = s1;
                const float tm = highest(s0, s1);
                // fp16 holds 2^(x - m) only up to 2^16: its reference sits a little above the
                // first step's maximum, which trades low-end resolution for head room
                m[t] = quad_column_max(tm) * c_log2 + (kGuard ? head_room : 0.0f);
                if constexpr (kGuard) wide |= is_wide(s0, s1, tm);
            }
            if constexpr (kGuard) alarm(wide, 0);
        }
    };

    // ---- careful softmax of one row tile over one 32-key step: mask + exact online rescale ----
    // Straight-line code, so that the chains of a wavefront's tiles overlap: the visible keys of a row
    // come as one 32-bit word per step, and the rescale is done whether or not a reference moved
    // (a factor of one changes nothing).
    auto softmax_step = [&](f32x4 &s0, f32x4 &s1, int t, int step_pos) {
        if (step_pos + 32 > L) {                     // reaches drafts or the ragged end (uniform)
            uint64_t anc = 0;                        // the drafts row t sees; a row without a node sees all of them
            if (has_drafts) anc = irow[t] >= 0 ? s_anc[irow[t]] : ~(uint64_t)0 >> (64 - Nb);
            const int ahead = L - step_pos;          // prefix keys in this step (< 32), or minus the drafts before it
            const uint32_t word = ahead >= 0 ? ((1u << ahead) - 1u) | (uint32_t)(anc << ahead)
                                             : (-ahead < 64 ? (uint32_t)(anc >> -ahead) : 0u);
            const uint32_t va = word >> (4 * qd), vb = va >> 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s0[r] = (va >> r) & 1u ? s0[r] : -INFINITY;
                s1[r] = (vb >> r) & 1u ? s1[r] : -INFINITY;
            }
        }
        float tm = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])),
                         fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
        tm = quad_column_max(tm);
        const float mn = fmaxf(m[t], tm * c_log2);
        const float alpha = fast_exp2(m[t] - mn);
        m[t] = mn;
#pragma unroll
        for (int u = 0; u <= NT; ++u) O[t][u] *= alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s0[r] = fast_exp2(__builtin_fmaf(s0[r], c_log2, -m[t]));
            s1[r] = fast_exp2(__builtin_fmaf(s1[r], c_log2, -m[t]));
        }
    };

    // ---- careful step: any step, any type ----
    auto careful_step = [&](int buf, int ks, int step_pos) {
        if (my_nt == 0) return;
        const unsigned char *Kb = smem + buf * STAGE + ks * 32 * ROWB;
        const unsigned char *Vb = Kb + VREG;
        if constexpr (kF32) {
            // fp32 path: 16x16x4 MFMA, one channel (QK) / one key (PV) per quad and instruction; one softmax for both halves of the
            // step.  The order of the channels is free as long as both operands agree, so an LDS read brings a lane four at once:
            // K and Q take channels 16 c + 4 quad .. +3 one after the other, and tile u, lane j of V^T is channel
            // 64 (u / 4) + 4 j + u % 4 (the epilogue puts them back).  The loop is bound by the LDS and its instructions.  us, one value a
            // read and a softmax for each half -> now: head_dim 64, 16 rows, 512 tokens 10.1 -> 9.5, 128 rows, 2K 21.4 -> 17.4, head_dim 128, 16
            // rows, 2K 14.4 -> 13.05, 64 rows 17.4 -> 14.05, 128 rows 33.9 -> 26.9.  (One softmax alone 21.4 -> 20.7 and 33.7 -> 32.6.)
            static_assert(TPW == 1 && NT % 4 == 0, "one tile a wavefront, channels in blocks of 64");
            f32x4 sc[2];
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                f32x4 kf[QREGS / 4];
                const int key = kt * 16 + j;
#pragma unroll
                for (int c = 0; c < QREGS / 4; ++c)
                    kf[c] = *reinterpret_cast<const f32x4 *>(Kb + key * ROWB + (((4 * c + qd) ^ (key & KSWZ)) << 4));
                sc[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < QREGS; ++kk)
                    sc[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kk / 4][kk % 4], qs[0][kk], sc[kt], 0, 0, 0);
            }
            softmax_step(sc[0], sc[1], 0, step_pos);
#pragma unroll
            for (int kt = 0; kt < 2; ++kt) {
                f32x4 vf[4][NT / 4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int vkey = kt * 16 + 4 * qd + r;
                    const int vs = (vkey & VSWM) << 1;
#pragma unroll
                    for (int b4 = 0; b4 < NT / 4; ++b4)
                        vf[r][b4] = *reinterpret_cast<const f32x4 *>(Vb + vkey * ROWB + (((16 * b4 + j) ^ vs) << 4));
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        O[0][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][u / 4][u % 4], sc[kt][r], O[0][u], 0, 0, 0);
                    O[0][NT] = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, sc[kt][r], O[0][NT], 0, 0, 0);
                }
            }
        } else {
            uint4 kf[2][KQ];
            load_k_frags(Kb, kf);
            uint4 pf[TPW];
#pragma unroll
            for (int t = 0; t < TPW; ++t) {          // (a tile the wavefront does not own has zero queries and is dropped)
                f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KQ; ++kk) {
                    s0 = mfma16<T>(kf[0][kk], qf[t][kk], s0);
                    s1 = mfma16<T>(kf[1][kk], qf[t][kk], s1);
                }
                softmax_step(s0, s1, t, step_pos);
                pf[t].x = pack2<T>(s0[0], s0[1]);
                pf[t].y = pack2<T>(s0[2], s0[3]);
                pf[t].z = pack2<T>(s1[0], s1[1]);
                pf[t].w = pack2<T>(s1[2], s1[3]);
            }
            const uint4 ones = make_uint4(ones2<T>(), ones2<T>(), ones2<T>(), ones2<T>());
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                const uint4 vf = load_v_frag(Vb, u);
#pragma unroll
                for (int t = 0; t < TPW; ++t) O[t][u] = mfma16<T>(vf, pf[t], O[t][u]);
            }
#pragma unroll
            for (int t = 0; t < TPW; ++t) O[t][NT] = mfma16<T>(ones, pf[t], O[t][NT]);
        }
    };

    // ---- stage loop skeleton: keep NS-1 stages in flight ahead of the one computed ----
    int issued = 0;
    auto wait_stage = [&](int s) {
        // stage s has landed once at most (younger stages) * LPS loads remain
        const int ahead = issued - (s + 1);
        if (NS > 3 && ahead >= 2) wait_vmcnt<(NS > 3 ? 2 : 0) * LPS>();
        else if (NS > 2 && ahead == 1) wait_vmcnt<(NS > 2 ? 1 : 0) * LPS>();
        else wait_vmcnt<0>();
    };
    // careful stages [s_begin, s_end)
    auto run_careful = [&](int s_begin, int s_end) {
        for (int s = s_begin; s < s_end; ++s) {
            wait_stage(s);
            __syncthreads();     // everyone's part of stage s is in; stage s-1 is fully consumed
            if (issued < nstages) {
                issue_stage(issued);                // refills the slot stage s-1 occupied
                ++issued;
            }
            const int sbase = pos0 + s * SK;
            auto step = [&](int ks) {
                if (ks % WK != wk) return;
                if (sbase + ks * 32 >= pos1) return;         // uniform: nothing left in this step
                careful_step(s % NS, ks, sbase + ks * 32);
            };
            if constexpr (kF32) {
#pragma unroll 1                                             // (two copies of the step spill at head_dim 128: 32 rows, 2K 18.5 -> 15.4 us)
                for (int ks = 0; ks < KSTEPS; ++ks) step(ks);
            } else {
#pragma unroll
                for (int ks = 0; ks < KSTEPS; ++ks) step(ks);
            }
        }
    };
    // A fast loop returns n_fast, or the stage at whose barrier the alarm was seen: its last.

    // fast stages [0, n_fast); the caller has admitted stage 0.
    // The two waves of a SIMD (w and w + 4) would run in lockstep if both took
    // the per-stage barrier at the same place in their instruction stream, and
    // their MFMA phases and their exp/convert phases would collide.  So waves
    // 4..7 take it one PV block later than waves 0..3: they carry the last PV of
    // a stage (its P and V^T fragments are in registers by then, so the stage's
    // ring slot is free all the same) across the barrier.  After every barrier
    // the two waves of a SIMD are then half a step apart, and one's matrix work
    // overlaps the other's vector work.
    auto run_fast_n = [&](int n_fast, auto ntag, auto gtag, [[maybe_unused]] float room) -> int {
        if constexpr (!kF32) {
            constexpr bool kWatch = kGuard && !decltype(gtag)::value;
            const bool late = wave >= kWaves / 2;
            auto kptr = [&](int s, int ks) -> const unsigned char * {
                return smem + (s % NS) * STAGE + ks * 32 * ROWB;
            };
            int end = n_fast;
            auto admit = [&](int s) {
                if constexpr (kWatch)
                    if (watched(s)) watch_sums();
                wait_stage(s);
                __syncthreads();     // stage s is in; all LDS reads of stage s-1 have completed
                if constexpr (kWatch)
                    if (watched(s) && alarmed(1)) end = s;
                if (issued < nstages) {
                    issue_stage(issued);
                    ++issued;
                }
            };
            uint4 pf[TPW], vf[NT];
            auto stage = [&](int s) {
                if constexpr (WK == 1) {
                    if (s > 0) {
                        if (!late) fast_pv(pf, vf, ntag);       // early waves finish stage s-1 first
                        admit(s);
                        if (late) fast_pv(pf, vf, ntag);        // late waves carry it over
                    }
                    fast_sx(kptr(s, 0), kptr(s, 0) + VREG, pf, vf, ntag, gtag, room);
                    fast_pv(pf, vf, ntag);
                    fast_sx(kptr(s, 1), kptr(s, 1) + VREG, pf, vf, ntag, gtag, room);
                } else {
                    if (s > 0) {
                        if (!late) fast_pv(pf, vf, ntag);
                        admit(s);
                        if (late) fast_pv(pf, vf, ntag);
                    }
                    fast_sx(kptr(s, wk), kptr(s, wk) + VREG, pf, vf, ntag, gtag, room);
                }
            };
            if constexpr (kGuard && (TPW > 1 || !kWatch)) {
#pragma unroll 1                                             // (with their first stages peeled off, these loops' kernels spill)
                for (int s = 0; s < end; ++s) stage(s);
            } else {
                for (int s = 0; s < end; ++s) stage(s);
            }
            fast_pv(pf, vf, ntag);
            return end;
        } else {
            return 0;
        }
    };
    // Pipelined fast stages [0, n_fast); the caller has admitted stage 0 and Sa
    // holds the scores of step 0.  V of a step is read one iteration after its
    // K, so a ring slot is refilled one stage later than in the plain loop: at
    // the barrier in front of step 2s+1 every wave is done with stage s-1.
    auto run_pipe_n = [&](int n_fast, f32x4 (&Sa)[TPW][2], auto ntag) -> int {
        int end = n_fast;
        if constexpr (kPipe) {
            constexpr int NA = decltype(ntag)::value;
            using yes = std::true_type;
            using no = std::false_type;
            f32x4 Sb[TPW][2];
            uint4 Pa[TPW], Pb[TPW], vpre[PF];
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                Pa[t] = Pb[t] = make_uint4(0, 0, 0, 0);
                Sb[t][0] = Sb[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < PF; ++u) vpre[u] = make_uint4(0, 0, 0, 0);
            // step 0: P of step 0, scores of step 1; no V^T P yet
            pipe_iter(Sa, Sb, Pb, Pa, vpre, std::integral_constant<uint32_t, 0>{},
                      std::integral_constant<uint32_t, 32 * ROWB>{}, std::integral_constant<uint32_t, 0>{}, no{}, ntag);
            if constexpr (kGuard) {
                bool wide = false;
#pragma unroll
                for (int t = 0; t < NA; ++t) wide |= is_wide(Sb[t][0], Sb[t][1], highest(Sb[t][0], Sb[t][1]));
                alarm(wide, 1);
            }
            for (int s4 = 0; s4 < end; s4 += NS) {
                static_for<0, NS>([&](auto bb) {
                    constexpr uint32_t B = decltype(bb)::value, B1 = (B + 1) % NS;
                    constexpr uint32_t cur0 = B * STAGE, cur1 = B * STAGE + 32 * ROWB;
                    constexpr uint32_t nxt0 = B1 * STAGE, nxt1 = B1 * STAGE + 32 * ROWB;
                    const int s = s4 + (int)B;
                    if (s < end) {                                      // uniform
                        // stage s+1 in; every wave is done with stage s-1: refill its slot
                        const int pg = stage_page(issued);
                        constexpr bool kLook = kGuard && B == 0;
                        if constexpr (kLook)
                            if (s > 0 && watched(s)) watch_sums();
                        wait_stage(s + 1);
                        __syncthreads();
                        if constexpr (kLook)
                            if (watched(s) && alarmed(1)) end = s;
                        if (issued < nstages && issued <= s + NS - 1) {
                            issue_stage_pg(issued, pg);
                            ++issued;
                        }
                        // step 2s+1: its P; O += V^T P of step 2s; scores of step 2s+2
                        pipe_iter(Sb, Sa, Pa, Pb, vpre, std::integral_constant<uint32_t, cur0>{},
                                  std::integral_constant<uint32_t, nxt0>{}, std::integral_constant<uint32_t, cur1>{},
                                  yes{}, ntag);
                        // step 2s+2: its P; O += V^T P of step 2s+1; scores of step 2s+3.  After the
                        // last fast stage only the V^T P part counts: the P and the scores it
                        // produces belong to steps the careful loop redoes, and are dropped.
                        pipe_iter(Sa, Sb, Pb, Pa, vpre, std::integral_constant<uint32_t, cur1>{},
                                  std::integral_constant<uint32_t, nxt1>{}, std::integral_constant<uint32_t, nxt0>{},
                                  yes{}, ntag);
                    }
                });
            }
        }
        return end;
    };
    // the fast loop is compiled once per possible tile count of a wave, so that
    // its body has no per-tile branches
    auto run_fast_tag = [&](int n_fast, bool guarded, float room, f32x4 (&Sa)[TPW][2], auto ntag) -> int {
        if constexpr (kGuard)
            if (guarded) return run_fast_n(n_fast, ntag, std::true_type{}, room);      // uniform over the workgroup
        if constexpr (kPipe) {
            return run_pipe_n(n_fast, Sa, ntag);
        } else {
            return run_fast_n(n_fast, ntag, std::false_type{}, 0.f);
        }
    };
    auto run_fast = [&](int n_fast, bool guarded, float room, f32x4 (&Sa)[TPW][2]) -> int {
        if (my_nt == TPW) return run_fast_tag(n_fast, guarded, room, Sa, std::integral_constant<int, TPW>{});
        if (TPW > 1 && my_nt == TPW - 1)
            return run_fast_tag(n_fast, guarded, room, Sa, std::integral_constant<int, (TPW > 1 ? TPW - 1 : 0)>{});
        if (TPW > 2 && my_nt == TPW - 2)
            return run_fast_tag(n_fast, guarded, room, Sa, std::integral_constant<int, (TPW > 2 ? TPW - 2 : 0)>{});
        return run_fast_tag(n_fast, guarded, room, Sa, std::integral_constant<int, 0>{});
    };
    static_assert(TPW <= 3, "run_fast dispatches on at most three tile counts");

    // The set-up loads are drained here, so that vmcnt counts the K/V stages from now on.
    wait_vmcnt<0>();

    // Pass 0: stages that lie wholly inside the prefix run the fast step with a
    // frozen reference; the rest (drafts, ragged end) run the careful step.
    // The last pass happens only if a row sum of the one before is not a modest finite
    // number: the whole split is redone with the careful step.  bf16 shares fp32's
    // exponent range, so that happens only for scores ~100 above the reference.
    // An fp16 P overflows 16 above it: fp16 has a pass between the two, the fast loop
    // with a guarded reference.  It serves pieces whose first scores already show a long
    // tail and redoes those that overflowed later on, these without room above the
    // reference: no weight is above 1 then, as in the exact loop, and none less exact
    // (with room a row's largest weight is rounded too, and the error of a redone piece
    // was up to 1.2 times as large).  With one tile a wavefront and two key groups the
    // exact loop is the faster redo.  us, exact loop and guarded without room, 8 heads, one
    // key in 200 eight times as long: 240 rows, 5K in four row groups 27.1 and 28.1, 64
    // rows, 20K 29.9 and 30.8; 104 rows, 16 sequences of 8K-20K 268 and 256, 320 rows,
    // 64K 170 and 137.
    // fp32 is the small correctness shape and has no fast loop.
    constexpr bool kHasFast = !kF32;
    constexpr int kPasses = kGuard ? 3 : 2;
    // With one tile a wavefront the piece is bound by its K/V, and all that the ring holds is requested at once.  With more it
    // is bound by the loop, which should begin early: when every workgroup asks for its whole ring at the same time, stage 0
    // arrives in the middle of 33 MB (4 us), so the first stages go out one after the other, behind the queries (320 rows,
    // 20K tokens 41.5 -> 40.6 us, 240 rows, 64K 79.7 -> 79.3).
    constexpr bool kPaced = !kF32 && TPW >= 2;
    if constexpr (!kF32) {
        if constexpr (kPaced) {
            issue_queries();
            issue_stage(0);                           // (a piece is not empty)
            issued = 1;
        } else {
            // stage 0, the queries, and the stages whose slots the queries leave free
            issue_stage(0);
            issue_queries();
            for (issued = 1; issued < kQSlot0 && issued < nstages; ++issued) issue_stage(issued);
        }
    }
    if (has_drafts && wave == 0) {
        const uint64_t set = ancestor_sets(s_parent[min(lane, p.N - 1)], lane, Nb, p.dev_status);
        if (lane < Nb) s_anc[lane] = set;
    }
    if constexpr (!kF32) {
        if constexpr (kPaced) wait_vmcnt<LPS>();
        else wait_stage(0);                           // the queries were requested before stage 1: they are in as well
        take_queries();
        __syncthreads();                              // everyone has; their slots are free
        if constexpr (kPaced) {
            if (nstages > 1) issue_stage(issued++);
            wait_stage(0);
            __syncthreads();
        }
    }
    // (fp16) An overflow leaves a row sum infinite.  One that is no number comes from the inputs, and no other reference mends it.
    auto not_a_number = [&]() -> bool {
        bool any = false;
#pragma unroll
        for (int t = 0; t < TPW; ++t) any |= O[t][NT][0] != O[t][NT][0];
        return workgroup_any(any, wave, lane, s_any + kWaves);
    };
    [[maybe_unused]] bool kept = false;               // (fp16) the ring still holds the first stages
    for (int pass = 0; pass < kPasses; ++pass) {
        if constexpr (kGuard) {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                m[t] = kMInit;
#pragma unroll
                for (int u = 0; u <= NT; ++u) O[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        int n_fast = 0;
        if (kHasFast && pass < kPasses - 1) n_fast = max(0, min(nstages, (L - pos0) / SK));
        if (pass > 0 && !(kGuard && kept)) issued = 0;        // a redo starts over
        // (the careful loop begins by filling the last slot itself)
        for (const int fill = n_fast > 0 ? NS : NS - 1; issued < fill && issued < nstages; ++issued) issue_stage(issued);
        if (n_fast > 0) {
            stamp(2);
            f32x4 Sa[TPW][2];
            [[maybe_unused]] float room = kGuardRoom;
            if constexpr (kGuard) {
                if (pass == 1 && !kept) {             // an overflowed piece
                    room = 0.f;
                    wait_stage(0);
                    __syncthreads();
                }
            }
            init_reference(0, wk, room > 0.f ? 4.f : 0.f, Sa);
            if constexpr (kGuard) {
                __syncthreads();
                if (alarmed(0)) pass = 1;              // uniform over the workgroup
            }
            [[maybe_unused]] const int end = run_fast(n_fast, pass == 1, room, Sa);
            if constexpr (kGuard) {
                kept = end == 0;
                if (end < n_fast) {                   // a redo begins once no transfer is under way and no wavefront reads the ring
                    if (!kept) {
                        wait_vmcnt<0>();
                        if (kExactRedo || not_a_number()) pass = 1;
                    }
                    __syncthreads();
                    continue;
                }
            }
        } else {
            if constexpr (kGuard) pass = kPasses - 1;         // a redo would do the same once more
            stamp(2);
        }
        stamp(3);
        run_careful(n_fast, nstages);
        stamp(4);
        if (!kHasFast || pass == kPasses - 1) break;
        bool bad = false;
#pragma unroll
        for (int t = 0; t < TPW; ++t) bad |= !(O[t][NT][0] < 1.0e30f);
        if (!workgroup_any(bad, wave, lane, s_any + kWaves)) break;
        if constexpr (kGuard) {
            __syncthreads();
            if (kExactRedo || not_a_number()) pass = 1;
        } else {
#pragma unroll
            for (int t = 0; t < TPW; ++t) {
                m[t] = kMInit;
#pragma unroll
                for (int u = 0; u <= NT; ++u) O[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }

    // ---- merge the two key groups of a row group through LDS (reuses the ring), 16 bytes a lane ----
    // With one tile a wavefront the second group hands its tile to the first.  With two, each hands one over and finishes
    // the other, so that all eight wavefronts write partials.
    constexpr int kGive = WK == 2 ? TPW : 0;
    const int mine = kGive == 2 ? wk : 0;                             // the tile this wavefront finishes
    if constexpr (WK == 2) {
        static_assert(TPW <= 2, "a tile for each key group");
        __syncthreads();
        constexpr int PER_TILE = NT * 64 * 16 + 64 * 8;
        auto tile_of = [&](int w) -> unsigned char * { return smem + (w * WR + wr) * PER_TILE; };
        if (kGive == 2 || wk == 1) {
            unsigned char *dst = tile_of(kGive == 2 ? wk : 0);
#pragma unroll
            for (int u = 0; u < NT; ++u)
                reinterpret_cast<f32x4 *>(dst)[u * 64 + lane] = kGive == 2 && wk == 0 ? O[TPW - 1][u] : O[0][u];
            reinterpret_cast<float2 *>(dst + NT * 1024)[lane] = kGive == 2 && wk == 0 ? make_float2(m[TPW - 1], O[TPW - 1][NT][0])
                                                                                      : make_float2(m[0], O[0][NT][0]);
        }
        __syncthreads();
        if (kGive == 2 || wk == 0) {
            const unsigned char *src = tile_of(kGive == 2 ? 1 - wk : 0);
            if (kGive == 2 && wk == 1) {                              // from here on the tile sits in the first place
                m[0] = m[TPW - 1];
#pragma unroll
                for (int u = 0; u <= NT; ++u) O[0][u] = O[TPW - 1][u];
            }
            const float2 ml = reinterpret_cast<const float2 *>(src + NT * 1024)[lane];
            const float mn = fmaxf(m[0], ml.x);
            const float a1 = fast_exp2(m[0] - mn), a2 = fast_exp2(ml.x - mn);
            m[0] = mn;
#pragma unroll
            for (int u = 0; u < NT; ++u) O[0][u] = O[0][u] * a1 + reinterpret_cast<const f32x4 *>(src)[u * 64 + lane] * a2;
            O[0][NT][0] = O[0][NT][0] * a1 + ml.y * a2;
        }
    }

    // ---- write this split's partial ----
    // fp32 partials (fp32 inputs, or on request): the accumulator fragments as they are, float4 [slot][u][lane] =
    // channels 16*u + 4*quad .. +3 of row lane%16.  Otherwise: each row normalised by its row sum and by its largest magnitude s, as fp16,
    // uint4 [slot][u/2][lane] = the four halves of channel tile u (even) and of u + 1; (m, l, l s) beside it.
    if (wk == 0 || kGive == 2) {
#pragma unroll
        for (int t = 0; t < (WK == 2 ? 1 : TPW); ++t) {
            const int tile = (t + mine) * WR + wr, tg = rg * p.group_tiles + tile;
            if (tile >= p.group_tiles || tg >= p.RT) continue;
            const size_t slot = pc.slot + tg;
            const float l = O[t][NT][0];
            if (kF32 || !p.half_partials) {                          // uniform over the launch
                float4 *po = static_cast<float4 *>(p.part_o) + slot * (size_t)(NT * 64);
                if constexpr (kF32) {
                    // element r of tile u is channel 64 (u / 4) + 4 (4 quad + r) + u % 4: element u % 4 of lane 16 r + j, tile 4 (u / 4) + quad
#pragma unroll
                    for (int u = 0; u < NT; u += 4)
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            po[(u + qd) * 64 + 16 * r + j] = make_float4(O[t][u][r], O[t][u + 1][r], O[t][u + 2][r], O[t][u + 3][r]);
                } else {
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        po[u * 64 + lane] = make_float4(O[t][u][0], O[t][u][1], O[t][u][2], O[t][u][3]);
                }
                if (qd == 0) {
                    float *stats = p.part_ml + slot * kPartMl + 3 * j;
                    stats[0] = m[t];
                    stats[1] = l;
                    stats[2] = 1.0f;
                }
            } else {
                const float inv_l = l > 0.f ? 1.0f / l : 0.f;          // a row that saw no key: all zeros
                float big = 0.f;
#pragma unroll
                for (int u = 0; u < NT; ++u)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        O[t][u][r] *= inv_l;
                        big = fmaxf(big, fabsf(O[t][u][r]));
                    }
                big = quad_column_max(big);                             // over the four lanes that hold this row
                const float inv_s = big > 0.f ? 1.0f / big : 0.f;
                uint4 *po = static_cast<uint4 *>(p.part_o) + slot * (size_t)(NT / 2 * 64) + lane;
#pragma unroll
                for (int u = 0; u < NT; u += 2)
                    po[(u / 2) * 64] = make_uint4(pack2<_Float16>(O[t][u][0] * inv_s, O[t][u][1] * inv_s),
                                                   pack2<_Float16>(O[t][u][2] * inv_s, O[t][u][3] * inv_s),
                                                   pack2<_Float16>(O[t][u + 1][0] * inv_s, O[t][u + 1][1] * inv_s),
                                                   pack2<_Float16>(O[t][u + 1][2] * inv_s, O[t][u + 1][3] * inv_s));
                if (qd == 0) {
                    float *stats = p.part_ml + slot * kPartMl + 3 * j;
                    stats[0] = m[t];
                    stats[1] = l;
                    stats[2] = l * big;
                }
            }
        }
    }
}

template <typename T, int D, int TPW, int WR, int WK, bool TL>
__global__ void __launch_bounds__(kThreads) splitkv_kernel(const KParams p)
{
    using GEO = Geo<T, D, TPW, WR, WK>;
    extern __shared__ __align__(16) unsigned char smem[];
    fetch_args<void(KParams)>();
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Workgroups go to the chip's eight XCDs round-robin in launch order, whether or not
    // they have work.  KV heads (all with the same amount of work) vary fastest, so that
    // splits that do not exist for a short sequence do not leave whole XCDs idle.
    // n numbers the workgroups in launch order; a "stream" is one (KV head, share of the K/V).
    // Row groups (workgroups that take different row tiles of the same stream, each reading its
    // K/V) are laid out so that the groups of a stream follow each other on ONE XCD: stream u sits
    // on XCD u mod 8, its groups in consecutive slots of that XCD, and all but the first find the
    // K/V in that XCD's L2.  With a single row group this is the plain order (n = u).
    // (the host keeps the workgroup count of a launch below 2^31)
    uint32_t n = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    int rg = 0;
    if (p.row_groups > 1) {                          // the host pads the stream count to a multiple of 8
        const uint32_t slot = n >> 3;
        rg = (int)(slot % (uint32_t)p.row_groups);
        n = ((slot / (uint32_t)p.row_groups) << 3) | (n & 7);
    }
    const uint32_t item = n / (uint32_t)p.Hkv;       // worker, or (split, sequence) with splits fastest
    // An XCD stays with its heads, and finds their query rows in its L2.  (Rotating the heads from one row of eight
    // workgroups to the next: 24 rows, 8 heads, 5K tokens 13.1 -> 13.2 us, four sequences of 3K-16K, 240 rows, 52.5 -> 53.7,
    // eight of 2K-9K, 4 heads, 39.6 -> 40.5.)
    const int g = (int)(n % (uint32_t)p.Hkv);
    const size_t head_slots = (size_t)g * p.n_slots;

    // timeline of this workgroup (profiling instantiations only; the production kernels
    // carry neither the pointer nor a branch)
    long long *tl = nullptr, last = 0, loop_clock = 0;
    if constexpr (TL) {
        const long long flat = blockIdx.x + (long long)gridDim.x * (blockIdx.y + (long long)gridDim.y * blockIdx.z);
        tl = p.timeline + 10 * flat;
        if (tid == 0) {
            last = wall_clock64();
            tl[0] = last;
            tl[1] = tl[2] = tl[3] = tl[4] = tl[5] = tl[8] = tl[9] = 0;
            // XCC_ID register (bits 3:0) above the shader-engine / CU id: one value per compute unit
            tl[6] = ((long long)(__builtin_amdgcn_s_getreg((3 << 11) | 20) & 15) << 16) | __smid();
            tl[7] = flat;
        }
    }
    // tl[k] sums, over the pieces of the share, the time from the stamp before to stamp k, tl[9] the shader cycles of the
    // fast loops (their rate is the clock the chip really ran at); the last lines of the kernel turn them into points in time.
    auto add = [&](int k, long long v) { atomicAdd(reinterpret_cast<unsigned long long *>(tl + k), (unsigned long long)v); };
    auto stamp = [&](int k) {
        if constexpr (TL) {
            if (tid == 0) {
                const long long now = wall_clock64();
                add(k, now - last);
                last = now;
                if (k == 2) loop_clock = clock64();
                if (k == 3) add(9, clock64() - loop_clock);
            }
        }
    };

    // The share: units [x, x1), the first of them in sequence b, which begins at unit `before`; the
    // partials of its piece in sequence b go to slot `slot0 + b`.
    int b = 0, before = 0, x, x1, slot0;
    Ahead ahead{-1, 0, false, {}, 0};
    Deal deal = p.full;
    int window = p.C;                                 // tokens of the window that is asked for ahead
    if (!p.dealt) {                                   // equal splits of C tokens, of one sequence each
        const int c = (int)(item % gridDim.y);
        b = (int)(item / gridDim.y);
        if (b >= p.B || c >= p.max_splits) return;    // padding of the grid
        x = c * (p.C / kSplitQuantum);
        x1 = x + p.C / kSplitQuantum;
        slot0 = b * p.max_splits + c - b;
    } else {
        if ((int)item >= p.rule.max_workers) return;  // padding of the grid
        x = deal_begin(deal, min((int)item, deal.workers - 1));
        window = (deal.q + 1) * kSplitQuantum;
    }
    // Most lone sequences are as long as announced: their pages and parents are asked for along with the length.
    PagePair pages{};
    int parent = 0;
    if (!p.dealt || p.B == 1) {
        ahead.pos0 = x * kSplitQuantum;
        ahead.parents = true;
        pages = load_pages(p, tid, b, ahead.pos0, 0);
        parent = p.parent[(int64_t)b * p.N + min(tid, p.N - 1)];
    }
    SeqSize size{0, 0};                               // of the first sequence, once known
    bool sized = false;
    if (p.dealt) {
        const int worker = (int)item;
        if (p.B == 1) {
            size = SeqSize{load_ctx_len(p.ctx_lens, 0, p.max_ctx_len, p.dev_status), load_n_draft(p.n_draft_seq, 0, p.N, p.dev_status)};
            const int T1 = size.drafts == 0 ? 0 : size.len + size.drafts;
            if (T1 != p.max_ctx_len + p.N) deal = deal_units(p, max(seq_units(p, T1), 1));
        } else {
            const BatchUnits u = batch_units(p);
            if (u.total == 0) return;                 // not one sequence has drafts
            deal = deal_units(p, u.total);
            if (worker < deal.workers) find_unit(p, u, deal_begin(deal, worker), &b, &before);
            size = size_of(p, u, b);
        }
        sized = true;
        if (worker >= deal.workers) return;
        x = deal_begin(deal, worker);
        x1 = deal_begin(deal, worker + 1);
        slot0 = worker;
    }
    if constexpr (TPW == 3) {
        if (ahead.parents) {
            int32_t *s_pages = reinterpret_cast<int32_t *>(smem + GEO::PAGES), *s_parent = reinterpret_cast<int32_t *>(smem + GEO::PARENT);
            ahead.kept = min((min(window, p.max_ctx_len + p.N - ahead.pos0) + kPage - 1) / kPage, 2 * kThreads);
            bool bad = false;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int idx = tid + r * kThreads, pg = pages.page[r];
                bad |= idx < ahead.kept && (pg < 0 || pg >= p.n_pool_pages || (p.page_table && ahead.pos0 / kPage + idx >= p.max_pages));
                s_pages[idx] = pg;
            }
            if (__builtin_amdgcn_ballot_w64(bad)) ahead.pos0 = -1;
            if (tid < p.N) s_parent[tid] = parent;
        }
    } else {
        ahead.pages = pages;
        ahead.parent = parent;
    }
    for (bool again = false; b < p.B; ++b) {
        if (!sized) size = SeqSize{load_ctx_len(p.ctx_lens, b, p.max_ctx_len, p.dev_status), load_n_draft(p.n_draft_seq, b, p.N, p.dev_status)};
        sized = false;
        const int L = size.len, Nb = size.drafts;
        const int T_b = Nb == 0 ? 0 : L + Nb;
        const int s0 = x - before, s1 = min(x1 - before, stages_of(T_b));
        if (s0 < s1) {
            if (again) __syncthreads();               // LDS is free again
            again = true;
            const Piece pc{b, L, Nb, s0 * kSplitQuantum, min(s1 * kSplitQuantum, T_b),
                           (head_slots + slot0 + b) * p.RT};
            run_piece<T, D, TPW, WR, WK>(p, smem, wave, g, rg, pc, ahead, stamp);
            stamp(5);
            ahead.pos0 = -1;
            ahead.parents = false;
        }
        before += seq_units(p, T_b);
        if (before >= x1 || !p.dealt) break;
        x = before;
    }
    if constexpr (TL) {
        __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the partial stores have left
        stamp(5);
        if (tid == 0) {
            long long at = tl[0];
            for (int k = 1; k <= 5; ++k) {
                at += (long long)atomicAdd(reinterpret_cast<unsigned long long *>(tl + k), 0ull);     // read where it was added
                tl[k] = at;
            }
            tl[8] = loop_clock;
            add(9, loop_clock);
        }
    }
}

// ---------------------------------------------------------------------------
// instantiations
// ---------------------------------------------------------------------------
template <typename T, int D, int TPW, int WR, int WK, bool TL>
static void launch_variant(const KParams &p, dim3 grid, hipStream_t s, hipEvent_t start, hipEvent_t stop)
{
    using GEO = Geo<T, D, TPW, WR, WK>;
    if (start || stop)
        hipExtLaunchKernelGGL((splitkv_kernel<T, D, TPW, WR, WK, TL>), grid, dim3(kThreads), GEO::LDS, s, start, stop, 0, p);
    else
        hipLaunchKernelGGL((splitkv_kernel<T, D, TPW, WR, WK, TL>), grid, dim3(kThreads), GEO::LDS, s, p);
}

#define OWL_VARIANT(DT, T, D, TPW, WR, WK, TL)                                          \
    Variant { DT, D, TPW, WR, WK, TL, Geo<T, D, TPW, WR, WK>::LDS,                     \
              &launch_variant<T, D, TPW, WR, WK, TL>,                                   \
              reinterpret_cast<const void *>(&splitkv_kernel<T, D, TPW, WR, WK, TL>) }

#define OWL_VARIANTS_16BIT(DT, T, D, TL)                                                \
    OWL_VARIANT(DT, T, D, 1, 4, 2, TL), OWL_VARIANT(DT, T, D, 1, 8, 1, TL),             \
    OWL_VARIANT(DT, T, D, 2, 4, 2, TL), OWL_VARIANT(DT, T, D, 2, 8, 1, TL), OWL_VARIANT(DT, T, D, 3, 8, 1, TL)

static const Variant kVariants[] = {
    OWL_VARIANTS_16BIT(OWL_BF16, __bf16, 128, false),
    OWL_VARIANTS_16BIT(OWL_BF16, __bf16, 64, false),
    OWL_VARIANTS_16BIT(OWL_F16, _Float16, 128, false),
    OWL_VARIANTS_16BIT(OWL_F16, _Float16, 64, false),
    OWL_VARIANT(OWL_F32, float, 64, 1, 8, 1, false),
    OWL_VARIANT(OWL_F32, float, 128, 1, 8, 1, false),
    // copies with the per-workgroup timeline hook: the benchmark's type and head size only
    OWL_VARIANTS_16BIT(OWL_BF16, __bf16, 128, true),
};

const Variant *find_variant(int dtype, int D, int tpw, int wr, int wk, bool timeline)
{
    for (const Variant &v : kVariants)
        if (v.dtype == dtype && v.D == D && v.tpw == tpw && v.wr == wr && v.wk == wk && v.timeline == timeline)
            return &v;
    return nullptr;
}

int variant_index(const Variant *v) { return v ? static_cast<int>(v - kVariants) : -1; }

}  // namespace owl
