// One step of the drafter's recurrent cell (Sec. 3.2.1, Eq. 1-8 of the paper):
//     e   = E[t]                                   s^m = W^m h + alpha e,  m in {f, i, o, c}
//     g^m = sigmoid(s^m), m in {f, i, o}           c   = f(s^c) g^i
//     z'  = z g^f + c                              h'  = f(z') g^o
// with f = layer normalisation over the d channels followed by GeLU.
//
// The projection W^m h reads every weight exactly once (4 d d_in
// elements, 1.2 GB for the paper's d = 12288 with a square W) against at most
// 64 state rows: a streaming read of HBM with a thin contraction on the side,
// done with MFMA only because 64 rows x 4 d x d_in multiply-adds per step are
// beyond the vector ALUs at that rate.  Weights go from global memory straight
// into the MFMA operand registers: no element is used twice, so there is
// nothing to stage in LDS.  The gates then need whole-row statistics twice (of
// s^c and of z'): two small launches, see below.
#include <type_traits>

#include "owl_device.h"

namespace owl {

typedef float d_f32x4 __attribute__((ext_vector_type(4)));
typedef int d_i32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 d_bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 d_f16x8 __attribute__((ext_vector_type(8)));

template <bool kF16>
__device__ __forceinline__ d_f32x4 mfma16(d_i32x4 a, d_i32x4 b, d_f32x4 c)
{
    if constexpr (kF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(d_f16x8, a),
                                                      __builtin_bit_cast(d_f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(d_bf16x8, a),
                                                       __builtin_bit_cast(d_bf16x8, b), c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Projection.  The four W^m, each [d][d_in] (one output channel's weights
// contiguous), are one matrix of 4d rows.  A workgroup of four wavefronts owns
// GR groups of 64 consecutive rows (four 16-row MFMA tiles); every wavefront works on all
// the tiles, so that a fragment of h is loaded once per 4 GR weight fragments,
// and the wavefronts split the contraction dimension: wavefront w takes the
// k-blocks w, w + 4, ... of 128 elements.  In MFMA terms A = h (rows = states),
// B = W^T (columns = weight rows): lane l supplies the 8 consecutive k values of
// group l / 16 for state row / weight row l % 16, 16 bytes straight from memory.
// The four partial sums meet in LDS and are added in a fixed order.
//     s [P][4d] fp32, s[p][m * d + j] = (W^m h_p)[j]
//
// Two weight layouts.  OWL_W_ROWS is the matrix as it stands: a load instruction
// then touches 16 rows with 64 bytes each and the chip holds ~50 000 row streams
// open at once, which DRAM serves at 4.4-4.9 TB/s.  OWL_W_TILED stores the same
// numbers in the order the kernel consumes them,
//     granule(row, k) = ((row / 64 * KS + k / 32) * 4 + row % 64 / 16) * 64 + (k % 32 / 8) * 16 + row % 16
// in units of 16 bytes (8 elements), KS = d_in / 32, rows padded with zeros to a
// multiple of 64: one load instruction reads 1 KB contiguous, a workgroup reads
// contiguous runs of 64 d_in elements from end to end, and the same kernel
// reaches 6.7-6.9 TB/s, what a plain streaming read gets on this chip.
// ---------------------------------------------------------------------------
constexpr int kProjWaves = 4;
constexpr int kProjTiles = 4;     // 16-row weight tiles per group of 64 rows (fixed by the tiled layout)
constexpr int kProjUnroll = 4;    // consecutive k-steps of 32 that one wavefront takes
static_assert(kProjTiles <= kProjWaves, "wavefront w adds up and stores weight tile w");

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), unrolled at compile time.
template <int N, typename F>
__device__ __forceinline__ void each(F &&f)
{
    if constexpr (N > 0) {
        each<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// A wavefront works on GR groups of 64 weight rows at once: a fragment of h is then loaded once per 4 GR weight
// fragments.  GR > 1 pays with more than 16 states (proj_wide).
// k-steps (4 GR weight fragments and PT fragments of h each) that a wavefront keeps in flight: as many as leave room
// for 4 - GR wavefronts per SIMD.
constexpr int proj_depth(int PT, int GR)
{
    if (GR == 3) return PT == 2 ? 5 : PT == 3 ? 4 : 3;
    if (GR == 2) return PT == 2 ? 3 : 2;
    return PT == 1 ? 6 : PT == 2 ? 4 : PT == 3 ? 3 : 2;
}

template <bool kF16, int PT, bool kTiled, int GR>
__global__ void __launch_bounds__(kProjWaves * 64, 4 - GR) drafter_proj_kernel(const uint16_t *__restrict__ h,
                                                                               const uint16_t *__restrict__ w,
                                                                               float *__restrict__ s, int P, int d_in,
                                                                               int n_rows)
{
    constexpr int kTiles = GR * kProjTiles;
    __shared__ d_f32x4 red[kProjWaves][kTiles][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kg = lane >> 4;
    const int n_tiles = n_rows / 16;
    const int tile0 = blockIdx.x * kTiles;
    const int k_steps = d_in / 32;

    // w_base[q] + ks * w_step + w_off[nb] is this lane's 16 bytes of k-step ks of weight tile nb of group q (w_off in
    // bytes, the rest in elements and uniform over the wavefront; d_in <= 2^20 keeps all offsets below 2^28).
    // A tile or group past the end re-reads the last one (in bounds); its sums are not stored.
    static_assert(kTiled || GR == 1, "the row layout comes one group at a time");
    const uint16_t *w_base[GR];
    int w_step;
    uint32_t w_off[kProjTiles];
    if constexpr (kTiled) {
        w_step = kProjTiles * 512;
#pragma unroll
        for (int q = 0; q < GR; ++q) {
            const int group = min((int)blockIdx.x * GR + q, (n_tiles + kProjTiles - 1) / kProjTiles - 1);
            w_base[q] = w + (int64_t)group * k_steps * (kProjTiles * 512);
        }
#pragma unroll
        for (int nb = 0; nb < kProjTiles; ++nb) w_off[nb] = nb * 1024 + lane * 16;
    } else {
        w_step = 32;
        w_base[0] = w + (int64_t)tile0 * 16 * d_in;
#pragma unroll
        for (int nb = 0; nb < kProjTiles; ++nb) w_off[nb] = 2 * ((min(nb, n_tiles - 1 - tile0) * 16 + n) * d_in + kg * 8);
    }
    uint32_t h_off[PT];                                      // state rows past P read row P - 1 and are not stored either
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) h_off[pt] = 2 * (min(pt * 16 + n, P - 1) * d_in + kg * 8);

    d_f32x4 acc[PT][kTiles];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
        for (int nb = 0; nb < kTiles; ++nb) acc[pt][nb] = d_f32x4{0.f, 0.f, 0.f, 0.f};

    // This wavefront's k-steps, in its own order: blocks of kProjUnroll consecutive ones, dealt out to the wavefronts.
    // With more than 16 state rows the h fragments weigh as much as the weights in the L1/L2
    // traffic, and every workgroup of the chip asks for the same lines of h at the same time if
    // all sweep k in the same order: each starts at a round of its own instead.
    constexpr int kRound = kProjWaves * kProjUnroll;
    const int rounds = k_steps / kRound;
    const int n_mine = rounds * kProjUnroll + min(max(k_steps - rounds * kRound - wave * kProjUnroll, 0), kProjUnroll);
    const int first = PT > 1 && rounds > 1 ? (int)((blockIdx.x * 7u) % (unsigned)rounds) * kProjUnroll : 0;
    auto k_step_of = [&](int i) -> int {
        i += first;
        if (i >= n_mine) i -= n_mine;
        return (i / kProjUnroll) * kRound + wave * kProjUnroll + i % kProjUnroll;
    };

    if constexpr (!kTiled) {
        // A k-step is 64 bytes of a row here, half a memory line, and the weights are not kept in the caches: several k-steps
        // at a time, asked for row by row, so that the two halves of a line are asked for one right after the other.
        // (Through the ring below, one k-step after the other, lines were fetched twice; whole cell, us: d = d_in = 12288
        // with 10 / 40 states 361 -> 271 / 398 -> 316, 8192 with 20 180 -> 124, 4096 with 1 52 -> 39; rings of pairs or
        // fours gain nothing more.)
        constexpr int kStep = PT <= 2 ? 4 : 2;
        auto steps = [&](auto count, int i) {
            constexpr int n_steps = decltype(count)::value;
            d_i32x4 b[n_steps][kTiles], a[n_steps][PT];
            int ks[n_steps];
#pragma unroll
            for (int u = 0; u < n_steps; ++u) ks[u] = k_step_of(i + u);
#pragma unroll
            for (int nb = 0; nb < kTiles; ++nb)
#pragma unroll
                for (int u = 0; u < n_steps; ++u)
                    b[u][nb] = __builtin_nontemporal_load(reinterpret_cast<const d_i32x4 *>(
                        reinterpret_cast<const char *>(w_base[0] + (int64_t)ks[u] * w_step) + w_off[nb]));
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                for (int u = 0; u < n_steps; ++u)
                    a[u][pt] = *reinterpret_cast<const d_i32x4 *>(reinterpret_cast<const char *>(h + ks[u] * 32) + h_off[pt]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < n_steps; ++u)
#pragma unroll
                for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                    for (int nb = 0; nb < kTiles; ++nb) acc[pt][nb] = mfma16<kF16>(a[u][pt], b[u][nb], acc[pt][nb]);
            __builtin_amdgcn_sched_barrier(0);
        };
        int i = 0;
        for (; i + kStep <= n_mine; i += kStep) steps(std::integral_constant<int, kStep>{}, i);
        for (; i < n_mine; ++i) steps(std::integral_constant<int, 1>{}, i);
    } else {
        // The stream: a ring of kDepth k-steps in registers.  A slot's loads are issued as soon as the MFMAs
        // have read it and are waited for kDepth - 1 steps later; the scheduling fences keep them apart (left to itself the
        // compiler moved every load next to its use and waited for one after the other: with 40 states it kept 7 of a
        // wavefront's 28 loads in flight; d = 4096, d_in = 12288, 40 states: 116 -> 83 us).
        constexpr int kDepth = proj_depth(PT, GR);
        d_i32x4 b[kDepth][kTiles], a[kDepth][PT];
        auto load = [&](auto slot, int i) {
            constexpr int S = decltype(slot)::value;
            const int ks = k_step_of(i);
            const char *hk = reinterpret_cast<const char *>(h + ks * 32);
            // every weight is used once: a non-temporal load, which leaves the caches to h (re-read by
            // every workgroup) and is worth 11 % on this chip (square step: 206 -> 183 us)
#pragma unroll
            for (int q = 0; q < GR; ++q) {
                const char *wk = reinterpret_cast<const char *>(w_base[q] + (int64_t)ks * w_step);
#pragma unroll
                for (int nb = 0; nb < kProjTiles; ++nb)
                    b[S][q * kProjTiles + nb] = __builtin_nontemporal_load(reinterpret_cast<const d_i32x4 *>(wk + w_off[nb]));
            }
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) a[S][pt] = *reinterpret_cast<const d_i32x4 *>(hk + h_off[pt]);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto use = [&](auto slot) {
            constexpr int S = decltype(slot)::value;
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                for (int nb = 0; nb < kTiles; ++nb) acc[pt][nb] = mfma16<kF16>(a[S][pt], b[S][nb], acc[pt][nb]);
            __builtin_amdgcn_sched_barrier(0);
        };
        int i = 0;                                               // k-steps requested so far
        if (n_mine >= kDepth) {
            each<kDepth>([&](auto slot) { load(slot, i++); });
            for (; i + kDepth <= n_mine; i += kDepth)
                each<kDepth>([&](auto slot) {
                    use(slot);
                    load(slot, i + decltype(slot)::value);
                });
            const int rest = n_mine - i;                         // fewer than kDepth
            each<kDepth>([&](auto slot) {
                use(slot);
                if (decltype(slot)::value < rest) load(slot, i + decltype(slot)::value);
            });
            each<kDepth - 1>([&](auto slot) {
                if (decltype(slot)::value < rest) use(slot);
            });
        } else {
            for (; i < n_mine; ++i) {
                load(std::integral_constant<int, 0>{}, i);
                use(std::integral_constant<int, 0>{});
            }
        }
    }

    // Accumulator layout: lane l holds, for weight row l % 16, the state rows 4 (l / 16) + i.
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        if (pt) __syncthreads();
#pragma unroll
        for (int nb = 0; nb < kTiles; ++nb) red[wave][nb][lane] = acc[pt][nb];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < GR; ++q) {
            const int mine = q * kProjTiles + wave, tile = tile0 + mine;
            if (tile >= n_tiles) continue;
            d_f32x4 v = red[0][mine][lane];
#pragma unroll
            for (int ww = 1; ww < kProjWaves; ++ww) v += red[ww][mine][lane];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = pt * 16 + kg * 4 + i;
                if (p < P) s[(int64_t)p * n_rows + tile * 16 + n] = v[i];
            }
        }
    }
}

static int proj_groups(int d) { return (4 * d / 16 + kProjTiles - 1) / kProjTiles; }

// Groups per workgroup.  With more than 16 states the h fragments that every group asks L2 for weigh as much as its
// weights; GR groups that share them cut that to a GRth (whole cell, us, one
// group -> shared: d = d_in = 12288 with 20 / 40 / 64 states 199 -> 187 / 228 -> 190 / 281 -> 198; 9600 with 48 states 190 -> 137).  With up to 16 states the weights alone
// fill the memory pipe (6.9 TB/s) and nothing is left to gain.  Taken where no compute unit is left with more groups than
// it has when they come one by one: below that the lost balance costs more than the sharing gives.
static int proj_wide(int P, int d, int n_cus)
{
    const int groups = proj_groups(d), most = (groups + n_cus - 1) / n_cus;
    if (P <= 16) return 1;
    for (int gr = 3; gr > 1; --gr)
        if (gr * (((groups + gr - 1) / gr + n_cus - 1) / n_cus) <= most) return gr;
    return 1;
}

template <bool kF16, int PT, bool kTiled, int GR>
static hipError_t launch_proj_gr(const void *h, const void *w, float *s, int P, int d_in, int d, hipStream_t st)
{
    hipLaunchKernelGGL((drafter_proj_kernel<kF16, PT, kTiled, GR>), dim3((proj_groups(d) + GR - 1) / GR), dim3(kProjWaves * 64), 0, st,
                       static_cast<const uint16_t *>(h), static_cast<const uint16_t *>(w), s, P, d_in, 4 * d);
    return hipGetLastError();
}

template <bool kF16, int PT>
static hipError_t launch_proj_pt(const void *h, const void *w, bool tiled, float *s, int P, int d_in, int d, int n_cus,
                                 hipStream_t st)
{
    if (!tiled) return launch_proj_gr<kF16, PT, false, 1>(h, w, s, P, d_in, d, st);
    if constexpr (PT > 1) {
        const int gr = proj_wide(P, d, n_cus);
        if (gr == 3) return launch_proj_gr<kF16, PT, true, 3>(h, w, s, P, d_in, d, st);
        if (gr == 2) return launch_proj_gr<kF16, PT, true, 2>(h, w, s, P, d_in, d, st);
    }
    return launch_proj_gr<kF16, PT, true, 1>(h, w, s, P, d_in, d, st);
}

template <bool kF16>
static hipError_t launch_proj_dt(const void *h, const void *w, bool tiled, float *s, int P, int d_in, int d, int n_cus,
                                 hipStream_t st)
{
    switch ((P + 15) / 16) {
    case 1: return launch_proj_pt<kF16, 1>(h, w, tiled, s, P, d_in, d, n_cus, st);
    case 2: return launch_proj_pt<kF16, 2>(h, w, tiled, s, P, d_in, d, n_cus, st);
    case 3: return launch_proj_pt<kF16, 3>(h, w, tiled, s, P, d_in, d, n_cus, st);
    default: return launch_proj_pt<kF16, 4>(h, w, tiled, s, P, d_in, d, n_cus, st);
    }
}

hipError_t launch_drafter_proj(int dtype, const void *h, const void *w, bool tiled, float *s, int P, int d_in,
                               int d, int n_cus, hipStream_t st)
{
    return dtype == OWL_F16 ? launch_proj_dt<true>(h, w, tiled, s, P, d_in, d, n_cus, st)
                            : launch_proj_dt<false>(h, w, tiled, s, P, d_in, d, n_cus, st);
}

// Bytes of the tiled copy of the weights: whole groups of 64 rows.
size_t drafter_tiled_bytes(int d_in, int d) { return (size_t)proj_groups(d) * (d_in / 32) * kProjTiles * 1024; }

// One thread per 16-byte granule of the tiled layout: find the (row, k) it holds
// and copy it from the row layout, zeros for the padding rows.
__global__ void __launch_bounds__(256) drafter_tile_weights_kernel(const uint4 *__restrict__ w_rows,
                                                                   uint4 *__restrict__ w_tiled, int d_in,
                                                                   int n_rows, int64_t n_granules)
{
    const int64_t gi = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gi >= n_granules) return;
    const int k_steps = d_in / 32;
    const int lane = (int)(gi & 63);
    const int nb = (int)((gi >> 6) % kProjTiles);
    const int64_t rest = (gi >> 6) / kProjTiles;
    const int ks = (int)(rest % k_steps);
    const int64_t g = rest / k_steps;
    const int64_t row = g * (kProjTiles * 16) + nb * 16 + (lane & 15);
    const int k = ks * 32 + (lane >> 4) * 8;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < n_rows) v = w_rows[(row * d_in + k) / 8];
    w_tiled[gi] = v;
}

hipError_t launch_drafter_tile_weights(const void *w_rows, void *w_tiled, int d_in, int d, hipStream_t st)
{
    const int64_t n_granules = (int64_t)(drafter_tiled_bytes(d_in, d) / 16);
    const int64_t blocks = (n_granules + 255) / 256;
    hipLaunchKernelGGL(drafter_tile_weights_kernel, dim3((unsigned)blocks), dim3(256), 0, st,
                       static_cast<const uint4 *>(w_rows), static_cast<uint4 *>(w_tiled), d_in, 4 * d, n_granules);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gates and state update.  f needs the mean and variance of a whole row twice
// (of s^c, then of z'), and the transcendental work of one row (three sigmoids
// and two GeLUs per channel) keeps a single compute unit busy for ~20 us, so a
// row is spread over workgroups of 256 threads x C channels, in two launches:
//   1. z' = z g^f + f(s^c) g^i, and per unit of 256 or 512 channels the mean and centred sum of squares of z'
//   2. merge those; h' = f(z') g^o
// The statistics of s^c need no transcendentals: every workgroup of launch 1 forms them from the whole row by itself, in
// registers, while its own operands are on their way: 48 KB of s^c and 24 KB of embedding from L2 at d = 12288, against a launch
// of its own with a round trip through memory (whole cell, us: d_in = 4096, 1 state, 10 rows 75.3 -> 73.7; d_in = 12288 with 10 / 40
// states and rows 188.5 -> 186.9 / 189.5 -> 188.9).
// The partials of z' are (mean, M2) pairs merged with the pairwise update
//     M2 = sum_c M2_c + n_c (mean_c - mean)^2 ,
// which keeps the variance as accurate as a two-pass sum.
// A row comes out the same, bit for bit, whatever C is, and with it however many rows are in the call: a unit depends on d
// alone, its sums form one balanced tree over its channels (in a lane, then over the lanes, then over the wavefronts), and where
// the compiler could contract a product into a sum or not, the code says which.
// ---------------------------------------------------------------------------
constexpr int kGateThreads = 256;
constexpr int kRowChunk = kGateThreads * 4;                // channels that a workgroup reads at a time for a whole row
constexpr int kRowMaxChunks = 16;                          // d <= 16384
constexpr int kGateMaxUnits = 32;                          // units of a row: one lane of a wavefront each, and what the scratch holds
__host__ __device__ constexpr int gate_unit(int d) { return d <= 256 * kGateMaxUnits ? 256 : 512; }
static_assert(kRowChunk * kRowMaxChunks <= gate_unit(kRowChunk * kRowMaxChunks) * kGateMaxUnits, "a row's units fit the scratch");

// Sum over the workgroup, the same in every thread.  Each call of a kernel has words of its own in `scratch`, so that one
// barrier is enough.  (Shuffles through LDS and two barriers a sum, and a loop over the chunks' partials in the hidden kernel:
// first launch 5.9 -> 5.4 us; whole cell d = d_in = 4096, 4 states, 30 rows 34.2 -> 33.5, 2048 16.1 -> 15.4.)
constexpr int kGateWaves = kGateThreads / 64;
__device__ __forceinline__ float block_sum(float v, float *scratch)
{
    const float sum = wave_sum(v);
    if ((threadIdx.x & 63) == 0) scratch[threadIdx.x >> 6] = sum;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kGateWaves; ++i) t += scratch[i];          // same order in every thread
    return t;
}

__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + expf(-x)); }
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

template <bool kF16> __device__ __forceinline__ float widen16(uint16_t b)
{
    if constexpr (kF16) return (float)__builtin_bit_cast(_Float16, b);
    else return __builtin_bit_cast(float, (uint32_t)b << 16);
}

template <bool kF16> __device__ __forceinline__ uint16_t narrow16(float x)
{
    if constexpr (kF16) {
        return __builtin_bit_cast(uint16_t, (_Float16)x);   // round to nearest even in hardware
    } else {
        uint32_t u = __builtin_bit_cast(uint32_t, x);
        if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);   // NaN stays NaN
        u += 0x7fffu + ((u >> 16) & 1u);                    // round to nearest even
        return (uint16_t)(u >> 16);
    }
}

// C consecutive channels (1, 2 or 4), and how they are read and written in one piece.
template <int C> struct Chan {
    float x[C];
};
template <int C> struct Bits16 {
    uint16_t x[C];
};
template <int C> __device__ __forceinline__ Chan<C> ld(const float *p)
{
    typedef float V __attribute__((ext_vector_type(C)));
    return __builtin_bit_cast(Chan<C>, *reinterpret_cast<const V *>(p));
}
template <> __device__ __forceinline__ Chan<1> ld<1>(const float *p) { return Chan<1>{{*p}}; }
template <int C> __device__ __forceinline__ void st(float *p, const Chan<C> &v)
{
    typedef float V __attribute__((ext_vector_type(C)));
    *reinterpret_cast<V *>(p) = __builtin_bit_cast(V, v);
}
template <> __device__ __forceinline__ void st<1>(float *p, const Chan<1> &v) { *p = v.x[0]; }
template <int C> __device__ __forceinline__ Chan<C> ld_or(const float *p, int j, float fill)
{
    if (p) return ld<C>(p + j);
    Chan<C> v;
#pragma unroll
    for (int i = 0; i < C; ++i) v.x[i] = fill;
    return v;
}
// s + alpha * (a 16-bit embedding row), C consecutive channels
template <bool kF16, int C> __device__ __forceinline__ Chan<C> add_emb(const float *s, const uint16_t *e, float alpha)
{
    typedef uint16_t V __attribute__((ext_vector_type(C == 1 ? 2 : C)));
    Bits16<C == 1 ? 2 : C> raw;
    if constexpr (C == 1) raw.x[0] = *e;
    else raw = __builtin_bit_cast(Bits16<C>, *reinterpret_cast<const V *>(e));
    Chan<C> v = ld<C>(s);
#pragma unroll
    for (int i = 0; i < C; ++i) v.x[i] = __builtin_fmaf(alpha, widen16<kF16>(raw.x[i]), v.x[i]);
    return v;
}

struct GateArgs {
    const float *s, *z;
    const int32_t *tokens, *parent_row;
    const uint16_t *emb;
    const float *gamma_c, *beta_c, *gamma_z, *beta_z;
    uint16_t *h_out;
    float *h_out_f32, *z_out;
    float *part_z;                // [M][kGateMaxUnits][2]: mean and centred sum of squares per unit
    int P, d, vocab;
    float alpha, eps;
    uint32_t *status;
};

// What every gate kernel needs first: the row's state, its token's embedding
// row and the embedding weight (0 for a token outside the table).
struct GateRow {
    const float *sp, *zp;
    const uint16_t *ep;
    float alpha;
};

__device__ __forceinline__ GateRow gate_row(const GateArgs &a, int r, bool flag)
{
    int p = a.parent_row ? a.parent_row[r] : r;
    if (p < 0 || p >= a.P) {
        if (flag && threadIdx.x == 0) flag_status(a.status, OWL_DEV_BAD_ROW);
        p = 0;
    }
    int tok = a.tokens[r];
    float alpha = a.alpha;
    if (tok < 0 || tok >= a.vocab) {
        if (flag && threadIdx.x == 0) flag_status(a.status, OWL_DEV_BAD_TOKEN);
        tok = 0;
        alpha = 0.f;
    }
    return GateRow{a.s + (int64_t)p * 4 * a.d, a.z + (int64_t)p * a.d, a.emb + (int64_t)tok * a.d, alpha};
}

// Sum of the C numbers of a lane over a unit of W wavefronts, the same in each of their threads.
template <int C, int W> __device__ __forceinline__ float unit_sum(const Chan<C> &v, float *scratch)
{
    float sum = v.x[0];
    if constexpr (C == 2) sum += v.x[1];
    if constexpr (C == 4) sum = (sum + v.x[1]) + (v.x[2] + v.x[3]);
    sum = wave_sum(sum);
    if constexpr (W == 1) {
        return sum;
    } else {
        const int wave = threadIdx.x >> 6;
        if ((threadIdx.x & 63) == 0) scratch[wave] = sum;
        __syncthreads();
        const float *u = scratch + wave / W * W;
        return W == 2 ? u[0] + u[1] : (u[0] + u[1]) + (u[2] + u[3]);
    }
}

// Mean and centred sum of squares of the live channels (from channel j on) of each unit of this workgroup.
template <int C, int UNIT> __device__ __forceinline__ void unit_stats(Chan<C> v, int j, int d, float *scratch, float *part)
{
#pragma clang fp contract(off)
    constexpr int kWaves = UNIT / (64 * C);
    static_assert(kWaves >= 1 && kWaves <= kGateWaves && (kWaves & (kWaves - 1)) == 0, "a workgroup holds whole units");
    const int unit = j / UNIT, n_live = min(UNIT, d - unit * UNIT);      // (of a unit behind the row: not above zero, not stored)
#pragma unroll
    for (int i = 0; i < C; ++i) v.x[i] = j < d ? v.x[i] : 0.f;
    const float mean = unit_sum<C, kWaves>(v, scratch) / (float)n_live;
#pragma unroll
    for (int i = 0; i < C; ++i) v.x[i] = j < d ? (v.x[i] - mean) * (v.x[i] - mean) : 0.f;
    const float m2 = unit_sum<C, kWaves>(v, scratch + kGateWaves);
    if (threadIdx.x % (64 * kWaves) == 0 && n_live > 0) part[2 * unit] = mean, part[2 * unit + 1] = m2;
}

// Mean and 1 / sqrt(variance + eps) of a row from its units' partials, one unit a lane: a loop over them waits for each.
__device__ __forceinline__ void merge_stats(const float2 part, int d, float eps, float *mean_out, float *rstd_out)
{
    const int u = threadIdx.x & 63, unit = gate_unit(d);
    const float n = (float)max(min(unit, d - u * unit), 0);                  // channels of the lane's unit
    const float mean = wave_sum(n > 0.f ? part.x * n : 0.f) / (float)d;
    const float dm = part.x - mean;
    const float m2 = wave_sum(n > 0.f ? __builtin_fmaf(n * dm, dm, part.y) : 0.f);
    *mean_out = mean;
    *rstd_out = 1.0f / sqrtf(m2 / (float)d + eps);
}

// Mean and 1 / sqrt(variance + eps) of s^c over a row of at most MAXC pieces of kRowChunk channels, in two passes over registers; the
// same in every workgroup of the row.
template <bool kF16, int MAXC>
__device__ __forceinline__ void row_stats(const GateArgs &a, const GateRow &g, float *scratch, float *mean_out, float *rstd_out)
{
    const int j0 = threadIdx.x * 4;
    Chan<4> v[MAXC];
#pragma unroll
    for (int c = 0; c < MAXC; ++c) {                        // past the end: the last channels once more, not counted
        const int j = min(c * kRowChunk + j0, a.d - 4);
        v[c] = add_emb<kF16, 4>(g.sp + 3 * a.d + j, g.ep + j, g.alpha);
    }
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
        if (c * kRowChunk + j0 < a.d) sum += (v[c].x[0] + v[c].x[1]) + (v[c].x[2] + v[c].x[3]);
    const float mean = block_sum(sum, scratch) / (float)a.d;
    float sq = 0.f;
#pragma unroll
    for (int c = 0; c < MAXC; ++c)
        if (c * kRowChunk + j0 < a.d) {
            const float4 x = make_float4(v[c].x[0] - mean, v[c].x[1] - mean, v[c].x[2] - mean, v[c].x[3] - mean);
            sq += __builtin_fmaf(x.x, x.x, x.y * x.y) + __builtin_fmaf(x.z, x.z, x.w * x.w);
        }
    *mean_out = mean;
    *rstd_out = 1.0f / sqrtf(block_sum(sq, scratch + kGateWaves) / (float)a.d + a.eps);
}

// (64 rows of 12 chunks are three wavefronts a SIMD: the compiler need not aim for more.  Where it did, it loaded the row in
// rounds, each a trip to L2.  us of this launch, rows loaded in rounds -> all at once: bf16, 12 chunks, 10 rows 8.0 -> 5.8, 40 rows
// 9.7 -> 8.3; 16 chunks, 10 rows bf16 9.2 -> 6.2, fp16 6.8 -> 6.0, 64 rows bf16 13.6 -> 12.4.  Others had all of it in flight already
// and stay as they are: fp16, 12 chunks, 10 rows 5.3.)
template <bool kF16, int MAXC, int C>
__global__ void __launch_bounds__(kGateThreads) __attribute__((amdgpu_waves_per_eu(1, 3))) drafter_state_kernel(GateArgs a)
{
    __shared__ float scratch[4 * kGateWaves];
    constexpr int kChunk = kGateThreads * C;
    const int c = blockIdx.x, r = blockIdx.y, j = c * kChunk + threadIdx.x * C;
    const GateRow g = gate_row(a, r, c == 0);
    const bool live = j < a.d;
    const int jl = live ? j : 0;
    const Chan<C> sf = add_emb<kF16, C>(g.sp + jl, g.ep + jl, g.alpha), si = add_emb<kF16, C>(g.sp + a.d + jl, g.ep + jl, g.alpha),
                  sc = add_emb<kF16, C>(g.sp + 3 * a.d + jl, g.ep + jl, g.alpha);
    const Chan<C> zo = ld<C>(g.zp + jl), ga = ld_or<C>(a.gamma_c, jl, 1.f), be = ld_or<C>(a.beta_c, jl, 0.f);
    float mean, rstd;
    row_stats<kF16, MAXC>(a, g, scratch, &mean, &rstd);
    Chan<C> zn;
#pragma unroll
    for (int i = 0; i < C; ++i)
        zn.x[i] = __builtin_fmaf(zo.x[i], sigmoid_f(sf.x[i]),
                                 gelu_f(__builtin_fmaf((sc.x[i] - mean) * rstd, ga.x[i], be.x[i])) * sigmoid_f(si.x[i]));
    if (live) st<C>(a.z_out + (int64_t)r * a.d + j, zn);
    unit_stats<C, gate_unit(MAXC * kRowChunk)>(zn, j, a.d, scratch + 2 * kGateWaves, a.part_z + (int64_t)r * kGateMaxUnits * 2);
}

template <bool kF16, int C>
__global__ void __launch_bounds__(kGateThreads) drafter_hidden_kernel(GateArgs a)
{
    constexpr int kChunk = kGateThreads * C;
    const int c = blockIdx.x, r = blockIdx.y, j = c * kChunk + threadIdx.x * C;
    // (everything is asked for before the statistics are merged; lanes past the last unit read unit 0 and do not count)
    const int u = threadIdx.x & 63;
    const float2 part = reinterpret_cast<const float2 *>(a.part_z)[(int64_t)r * kGateMaxUnits + (u * gate_unit(a.d) < a.d ? u : 0)];
    const bool live = j < a.d;
    const int jl = live ? j : 0;
    const Chan<C> zn = ld<C>(a.z_out + (int64_t)r * a.d + jl), ga = ld_or<C>(a.gamma_z, jl, 1.f), be = ld_or<C>(a.beta_z, jl, 0.f);
    const GateRow g = gate_row(a, r, false);
    const Chan<C> so = add_emb<kF16, C>(g.sp + 2 * a.d + jl, g.ep + jl, g.alpha);
    float mean, rstd;
    merge_stats(part, a.d, a.eps, &mean, &rstd);
    if (!live) return;
    Chan<C> hn;
    Bits16<C> out;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        hn.x[i] = gelu_f(__builtin_fmaf((zn.x[i] - mean) * rstd, ga.x[i], be.x[i])) * sigmoid_f(so.x[i]);
        out.x[i] = narrow16<kF16>(hn.x[i]);
    }
    if (a.h_out) {
        if constexpr (C == 1) {
            a.h_out[(int64_t)r * a.d + j] = out.x[0];
        } else {
            typedef uint16_t V __attribute__((ext_vector_type(C)));
            *reinterpret_cast<V *>(a.h_out + (int64_t)r * a.d + j) = __builtin_bit_cast(V, out);
        }
    }
    if (a.h_out_f32) st<C>(a.h_out_f32 + (int64_t)r * a.d + j, hn);
}

size_t drafter_gate_scratch_floats(int M) { return (size_t)M * kGateMaxUnits * 2; }

template <bool kF16, int MAXC, int C> static void launch_gates_as(const GateArgs &a, int M, hipStream_t st)
{
    const dim3 grid((a.d + kGateThreads * C - 1) / (kGateThreads * C), M), block(kGateThreads);
    hipLaunchKernelGGL((drafter_state_kernel<kF16, MAXC, C>), grid, block, 0, st, a);
    hipLaunchKernelGGL((drafter_hidden_kernel<kF16, C>), grid, block, 0, st, a);
}

template <bool kF16, int C> static void launch_gates_c(const GateArgs &a, int M, hipStream_t st)
{
    const int rounds = (a.d + 4 * kRowChunk - 1) / (4 * kRowChunk);
    if (rounds == 1) launch_gates_as<kF16, 4, C>(a, M, st);
    else if (rounds == 2) launch_gates_as<kF16, 8, C>(a, M, st);
    else if constexpr (C > 1) {                             // (one channel a lane: no workgroup holds a unit of 512, see launch_gates_dt)
        if (rounds == 3) launch_gates_as<kF16, 12, C>(a, M, st);
        else launch_gates_as<kF16, kRowMaxChunks, C>(a, M, st);
    }
}

// Channels a lane: a lane's sigmoids and GeLUs follow each other, so it takes as few as leave no more than one workgroup a
// compute unit (each reads its whole row) and whole units in each.  us per cell, four a lane -> as
// few as that (up to 512 workgroups, up to 1024): bf16, 10 rows, 2048 from 2048 15.4 -> 13.9 (13.9, 14.4), 4096 from 4096 31.3 -> 30.0 (30.0, 30.0),
// 12288 from 4096 72.7 -> 71.6 (71.6, 71.6); fp16, 16384 from 4096 92.6 -> 92.8 (93.4, 93.4); 40 rows, 12288 77.4 -> 77.5 (77.6, 78.9).
template <bool kF16> static hipError_t launch_gates_dt(const GateArgs &a, int M, int n_cus, hipStream_t st)
{
    static_assert(gate_unit(8 * kRowChunk) <= kGateThreads && gate_unit(8 * kRowChunk + 1) > kGateThreads,
                  "one channel a lane serves rows of up to two rounds, see launch_gates_c");
    auto fits = [&](int channels) {
        const int chunk = kGateThreads * channels;
        return gate_unit(a.d) <= chunk && (a.d + chunk - 1) / chunk * M <= n_cus;
    };
    if (fits(1)) launch_gates_c<kF16, 1>(a, M, st);
    else if (fits(2)) launch_gates_c<kF16, 2>(a, M, st);
    else launch_gates_c<kF16, 4>(a, M, st);
    return hipGetLastError();
}

hipError_t launch_drafter_gates(int dtype, const float *s, const float *z, const int32_t *tokens,
                                const int32_t *parent_row, const void *emb, const float *gamma_c,
                                const float *beta_c, const float *gamma_z, const float *beta_z, void *h_out,
                                float *h_out_f32, float *z_out, float *gate_scratch, int P, int M, int d, int vocab,
                                float alpha, float eps, uint32_t *status, int n_cus, hipStream_t st)
{
    GateArgs a;
    a.s = s, a.z = z, a.tokens = tokens, a.parent_row = parent_row, a.emb = static_cast<const uint16_t *>(emb);
    a.gamma_c = gamma_c, a.beta_c = beta_c, a.gamma_z = gamma_z, a.beta_z = beta_z;
    a.h_out = static_cast<uint16_t *>(h_out), a.h_out_f32 = h_out_f32, a.z_out = z_out;
    a.part_z = gate_scratch;
    a.P = P, a.d = d, a.vocab = vocab, a.alpha = alpha, a.eps = eps, a.status = status;
    return dtype == OWL_F16 ? launch_gates_dt<true>(a, M, n_cus, st) : launch_gates_dt<false>(a, M, n_cus, st);
}

}  // namespace owl
