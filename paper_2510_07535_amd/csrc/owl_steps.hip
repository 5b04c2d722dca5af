// The integer / data-movement steps on either side of the verify attention
// (Algorithm 1 of the paper): Prepare (Sec. 3.2.2, one extra token per tree
// node, mask and position ids), the greedy choice of the accepted path
// (Sec. 1 / Sec. 2: the target keeps the longest drafted path that agrees with
// its own next tokens), and the commit of that path's K/V rows into the
// context (Algorithm 1: l <- l;d, N <- N + |d|).  All results are exact.
#include <type_traits>

#include "owl_device.h"

namespace owl {

// ---------------------------------------------------------------------------
// Prepare: one workgroup per sequence, thread i < 2n owns token i of the verify
// input.  Tokens 0..n-1 are the tree nodes, token n+k is the extra token of node
// k: its parent is k, so it is one more node of the tree, with a mask and depth like any other.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) prepare_kernel(const int32_t *parent, const int32_t *ctx_lens, int n,
                                                     int32_t *parent2, uint64_t *anc, int32_t *depth,
                                                     int32_t *pos, uint32_t *status)
{
    fetch_args<decltype(prepare_kernel)>();
    const int b = blockIdx.x, i = threadIdx.x, n2 = 2 * n;
    const int L = pos ? load_uniform(ctx_lens, b) : 0;
    int p = i < n ? parent[(int64_t)b * n + i] : i - n;
    const uint64_t a = ancestor_sets(p, i, n2, status);
    if (i < n2) {
        if (p < -1 || p >= i) p = -1;                      // flagged above; keep the output a valid tree
        const int d = __popcll(a);
        const int64_t o = (int64_t)b * n2 + i;
        parent2[o] = p;
        anc[o] = a;
        if (depth) depth[o] = d;
        if (pos) pos[o] = L + d - 1;
    }
}

hipError_t launch_prepare(const int32_t *parent, const int32_t *ctx_lens, int B, int n, int32_t *parent2,
                          uint64_t *anc, int32_t *depth, int32_t *pos, uint32_t *status, hipStream_t s)
{
    hipLaunchKernelGGL(prepare_kernel, dim3(B), dim3(64), 0, s, parent, ctx_lens, n, parent2, anc, depth, pos,
                       status);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Acceptance: one wavefront per sequence, lane i owns node i.  A node "agrees"
// if its token is the target's next token at its parent (at the context end for
// a root); it is reachable if it and all its ancestors agree.  Parents precede
// children, so reachability spreads one tree level per round of a ballot loop
// that ends when a round adds nothing (at most depth rounds; the rounds look at
// the nodes of the round before only: 60 nodes 350 -> 190 instructions in all,
// 5.2 -> 4.7 us).  The answer is the reachable node of greatest depth, smallest
// index on ties; its root path is written from the root down.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(64) accept_kernel(const int32_t *tokens, const int32_t *parent,
                                                    const int32_t *target_root, const int32_t *target_next,
                                                    int N, int n_cand, int32_t *accepted, int32_t *n_accept,
                                                    int32_t *bonus, int32_t *last, uint32_t *status)
{
    fetch_args<decltype(accept_kernel)>();
    const int b = blockIdx.x, i = threadIdx.x;
    const int64_t row = (int64_t)b * N;
    // everything in one memory round trip; what the target says after the parent comes from the parent's lane
    const int64_t at = row + min(i, N - 1);
    int p = parent[at];
    const int token = tokens[at], next = target_next[at], root = load_uniform(target_root, b);
    const bool bad = i < N && (p < -1 || p >= i);
    if (bad) flag_status(status, OWL_DEV_BAD_PARENT);
    p = i < N && !bad ? p : -1;
    const int said = __shfl(next, max(p, 0));
    const bool agrees = i < N && i < n_cand && p < n_cand && token == (p < 0 ? root : said);
    // `fresh`: the nodes that the last round reached, each in one round only
    uint64_t fresh = __builtin_amdgcn_ballot_w64(agrees && p < 0), reach = fresh;
    const uint64_t up = agrees && p >= 0 ? (uint64_t)1 << p : 0;
    int depth = 1;                                          // of the lane's node, once reached
    for (int round = 2; fresh; ++round) {                   // uniform; a parent precedes its children, so it ends
        const bool now = (up & fresh) != 0;
        if (now) depth = round;
        fresh = __builtin_amdgcn_ballot_w64(now);
        reach |= fresh;
    }
    // deepest reachable node, smallest index on ties: key = depth * 64 + (63 - i)
    const int key = wave_max(((reach >> i) & 1) ? depth * 64 + (63 - i) : -1);
    const int best = key < 0 ? -1 : 63 - (key & 63);
    const int na = key < 0 ? 0 : key >> 6;
    // The path is walked in scalar registers; the node at depth k goes to place k - 1, the places behind it get -1.
    uint64_t path = 0;
    for (int node = best; node >= 0; node = __builtin_amdgcn_readlane(p, node)) path |= (uint64_t)1 << node;   // decreasing indices
    const int after = __builtin_amdgcn_readlane(next, max(best, 0));
    if ((path >> i) & 1) accepted[row + depth - 1] = i;
    if (i >= na && i < N) accepted[row + i] = -1;
    if (i == 0) {
        n_accept[b] = na;
        last[b] = best;
        bonus[b] = best < 0 ? root : after;
    }
}

hipError_t launch_accept(const int32_t *tokens, const int32_t *parent, const int32_t *target_root,
                         const int32_t *target_next, int B, int N, int n_cand, int32_t *accepted,
                         int32_t *n_accept, int32_t *bonus, int32_t *last, uint32_t *status, hipStream_t s)
{
    hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(64), 0, s, tokens, parent, target_root, target_next, N,
                       n_cand, accepted, n_accept, bonus, last, status);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// KV commit: one workgroup per (KV head, sequence, tensor).  Row i of the
// accepted path moves from logical position L + accepted[i] to L + i.  A source
// slot can be another row's destination (accepted = (1, 2): slot 1 is read by
// row 0 and written by row 1), so every thread loads all its 16-byte pieces
// first, the workgroup meets at a barrier, and only then anything is stored.
// accepted[] must be strictly increasing (a root path in a tree whose parents
// precede their children is); anything else is flagged and nothing is moved.
// The same holds for pages: every source and destination page of the sequence
// is looked up before anything is loaded, and one entry outside the pool (or a
// position beyond the table) means OWL_DEV_BAD_PAGE, no row of that sequence
// moves, and its new length equals the old one.  A kernel that writes must not
// replace a bad page by some other page.
// Every wavefront looks the path up for itself, lane = row (length, count and path in one memory round trip, the pages in the next),
// and hands the byte offsets of a row's source and destination to the lanes that move it: one barrier, and nothing of it in
// scratch memory: what remains of 4.65 us are four cold round trips.  (One wavefront for all by way of LDS, two barriers, divisions
// by the pieces of a row and the moved rows in scratch memory: 5.03.)
// ---------------------------------------------------------------------------
constexpr int kCommitThreads = 256;
constexpr int kCommitMaxPieces = 8;                         // 64 rows x 32 pieces / 256 threads

__device__ __forceinline__ int64_t shfl64(int64_t v, int lane)
{
    const uint32_t lo = __shfl((uint32_t)v, lane), hi = __shfl((uint32_t)((uint64_t)v >> 32), lane);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__global__ void __launch_bounds__(kCommitThreads) commit_kernel(
    unsigned char *k_cache, unsigned char *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
    const int32_t *accepted, const int32_t *n_accept, int N, int max_pages, int max_ctx_len,
    int64_t n_pool_pages, int log_pieces, int es, int64_t stride_page, int64_t stride_head,
    int64_t stride_token, int32_t *new_ctx_lens, uint32_t *status)
{
    fetch_args<decltype(commit_kernel)>();
    const int g = blockIdx.x, b = blockIdx.y;
    unsigned char *cache = (blockIdx.z ? v_cache : k_cache) + g * stride_head * es;
    const int tid = threadIdx.x, lane = tid & 63;
    const int a = accepted[(int64_t)b * N + min(lane, N - 1)];
    int na = load_uniform(n_accept, b), L = load_uniform(ctx_lens, b);
    asm volatile("" : "+s"(na), "+s"(L));                   // (both asked for before either is looked at)
    if (L < 0 || L > max_ctx_len) {
        if (tid == 0) flag_status(status, OWL_DEV_BAD_CTX_LEN);
        L = L < 0 ? 0 : max_ctx_len;
    }
    if (na < 0 || na > N) {
        if (tid == 0) flag_status(status, OWL_DEV_BAD_ACCEPT);
        na = 0;
    }
    // row `lane` of the path: physical pages of its source and destination, unchecked ids
    const int before = __shfl_up(a, 1), from = L + min(max(a, 0), N - 1), to = L + lane;
    const int from_lp = from / kPage, to_lp = to / kPage;
    int from_page = from_lp, to_page = to_lp;
    if (page_table) {
        const int32_t *pages = page_table + (int64_t)b * max_pages;
        from_page = pages[min(from_lp, max_pages - 1)];
        to_page = pages[min(to_lp, max_pages - 1)];
    }
    const bool bad_page = (page_table && max(from_lp, to_lp) >= max_pages) || min(from_page, to_page) < 0 || max(from_page, to_page) >= n_pool_pages;
    const bool mine = lane < na, bad = a < 0 || a >= N || (lane > 0 && a <= before);
    const bool any_bad = __builtin_amdgcn_ballot_w64(mine && bad) != 0;          // the same in every wavefront
    if (any_bad || __builtin_amdgcn_ballot_w64(mine && bad_page) != 0) {
        if (tid == 0) flag_status(status, any_bad ? OWL_DEV_BAD_ACCEPT : OWL_DEV_BAD_PAGE);
        na = 0;
    }
    if (g == 0 && blockIdx.z == 0 && tid == 0 && new_ctx_lens) new_ctx_lens[b] = L + na;

    const int64_t src = ((int64_t)from_page * stride_page + from % kPage * stride_token) * es;
    const int64_t dst = ((int64_t)to_page * stride_page + to % kPage * stride_token) * es;
    // The path climbs, so the rows that are in place already are its first ones.  16-byte piece `id` of the others belongs to row
    // first + (id >> log_pieces); past the end: the last row once more, not stored
    const uint64_t moved = __builtin_amdgcn_ballot_w64(lane < na && src != dst);
    if (moved == 0) return;                                 // uniform over the workgroup, as are the others
    const int first = __builtin_ctzll(moved), rows = na - first;
    const int total = rows << log_pieces, piece = (tid & ((1 << log_pieces) - 1)) * 16;
    typedef uint32_t Piece __attribute__((ext_vector_type(4)));          // (an array of the struct uint4 goes to scratch memory)
    auto move = [&](auto pieces) {
        constexpr int n = decltype(pieces)::value;
        Piece held[n];
        int64_t at[n];
#pragma unroll
        for (int r = 0; r < n; ++r) {
            const int id = tid + r * kCommitThreads, i = first + min(id >> log_pieces, rows - 1);
            const int64_t s = shfl64(src, i), d = shfl64(dst, i);
            at[r] = id < total && s != d ? d + piece : -1;  // (two table entries may name one page)
            held[r] = *reinterpret_cast<const Piece *>(cache + s + piece);
        }
        __syncthreads();                                    // all reads done before the first write
#pragma unroll
        for (int r = 0; r < n; ++r)
            if (at[r] >= 0) *reinterpret_cast<Piece *>(cache + at[r]) = held[r];
    };
    if (total <= kCommitThreads) move(std::integral_constant<int, 1>{});
    else move(std::integral_constant<int, kCommitMaxPieces>{});
}

hipError_t launch_commit(const owl_verify_desc &d, void *k_cache, void *v_cache, const int32_t *page_table,
                         const int32_t *ctx_lens, const int32_t *accepted, const int32_t *n_accept,
                         int32_t *new_ctx_lens, uint32_t *status, hipStream_t s)
{
    const int es = d.qkv_dtype == OWL_F32 ? 4 : 2;
    static_assert(64 * 32 <= kCommitThreads * kCommitMaxPieces, "64 rows of up to 512 bytes fit the held pieces");
    int log_pieces = 3;                                     // rows of 128, 256 or 512 bytes
    while (16 << log_pieces < d.head_dim * es) ++log_pieces;
    hipLaunchKernelGGL(commit_kernel, dim3(d.n_kv_heads, d.batch, 2), dim3(kCommitThreads), 0, s,
                       static_cast<unsigned char *>(k_cache), static_cast<unsigned char *>(v_cache), page_table,
                       ctx_lens, accepted, n_accept, d.n_draft, d.max_pages_per_seq, d.max_ctx_len,
                       d.n_pool_pages, log_pieces, es, d.kv_stride_page, d.kv_stride_head, d.kv_stride_token,
                       new_ctx_lens, status);
    return hipGetLastError();
}

}  // namespace owl
