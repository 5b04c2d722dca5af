// The integer / data-movement steps on either side of the verify attention
// (Algorithm 1 of the paper): Prepare (Sec. 3.2.2, one extra token per tree
// node, mask and position ids), the greedy choice of the accepted path
// (Sec. 1 / Sec. 2: the target keeps the longest drafted path that agrees with
// its own next tokens), and the commit of that path's K/V rows into the
// context (Algorithm 1: l <- l;d, N <- N + |d|).  All results are exact.
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
// that ends when a round adds nothing (at most depth rounds).  The answer is the
// reachable node of greatest depth, smallest index on ties; its root path is
// written from the root down.
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
    if (i >= N) {
        p = -1;
    } else if (p < -1 || p >= i) {
        flag_status(status, OWL_DEV_BAD_PARENT);
        p = -1;
    }
    const int said = __shfl(next, max(p, 0));
    const bool agrees = i < N && i < n_cand && p < n_cand && token == (p < 0 ? root : said);
    uint64_t reach = 0;
    int depth = 0;                                          // depth of lane's node once reached
    for (int round = 1; round <= N; ++round) {              // uniform: `reach` is the same in every lane
        const bool now = agrees && !((reach >> i) & 1) && (p < 0 ? round == 1 : ((reach >> p) & 1));
        const uint64_t add = __builtin_amdgcn_ballot_w64(now);
        if (now) depth = round;
        if (add == 0) break;
        reach |= add;
    }
    // deepest reachable node, smallest index on ties: key = depth * 64 + (63 - i)
    int key = ((reach >> i) & 1) ? depth * 64 + (63 - i) : -1;
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) key = max(key, __shfl_xor(key, off));
    key = __builtin_amdgcn_readfirstlane(key);
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
// ---------------------------------------------------------------------------
constexpr int kCommitThreads = 256;
constexpr int kCommitMaxPieces = 8;                         // 64 rows x 32 pieces / 256 threads

__global__ void __launch_bounds__(kCommitThreads) commit_kernel(
    unsigned char *k_cache, unsigned char *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
    const int32_t *accepted, const int32_t *n_accept, int N, int max_pages, int max_ctx_len,
    int64_t n_pool_pages, int row_bytes, int es, int64_t stride_page, int64_t stride_head,
    int64_t stride_token, int32_t *new_ctx_lens, uint32_t *status)
{
    __shared__ int32_t s_src[64];
    __shared__ int64_t s_src_page[64], s_dst_page[64];
    __shared__ int s_bad, s_bad_page;
    fetch_args<decltype(commit_kernel)>();
    const int g = blockIdx.x, b = blockIdx.y;
    unsigned char *cache = blockIdx.z ? v_cache : k_cache;
    const int tid = threadIdx.x;
    // length, count and path in one memory round trip, the pages in the next (one after the other: 4.6 -> 4.1 us a launch)
    int a = 0;
    if (tid < 64) a = accepted[(int64_t)b * N + min(tid, N - 1)];
    int na = load_uniform(n_accept, b);
    const int L = load_ctx_len(ctx_lens, b, max_ctx_len, status);
    if (na < 0 || na > N) {
        if (tid == 0) flag_status(status, OWL_DEV_BAD_ACCEPT);
        na = 0;
    }
    if (tid < 64) {                                         // one wavefront, lane = row of the path
        const int prev = __shfl_up(a, 1);
        const bool mine = tid < na;
        bool bad = false, bad_page = false;
        if (mine) {
            bad = a < 0 || a >= N || (tid > 0 && a <= prev);
            s_src[tid] = a;
            // physical pages of the row's source and destination, unchecked ids; -1 = not in the table
            auto page_of = [&](int pos) -> int64_t {
                const int lp = pos / kPage;
                if (!page_table) return lp;
                return lp < max_pages ? (int64_t)page_table[(int64_t)b * max_pages + lp] : -1;
            };
            const int64_t sp = (a >= 0 && a < N) ? page_of(L + a) : 0, dp = page_of(L + tid);
            bad_page = sp < 0 || sp >= n_pool_pages || dp < 0 || dp >= n_pool_pages;
            s_src_page[tid] = sp;
            s_dst_page[tid] = dp;
        }
        const bool any_bad = __builtin_amdgcn_ballot_w64(bad) != 0, any_page = __builtin_amdgcn_ballot_w64(bad_page) != 0;
        if (tid == 0) s_bad = any_bad, s_bad_page = any_page;
    }
    __syncthreads();
    if (s_bad) {                                            // uniform over the workgroup
        if (tid == 0) flag_status(status, OWL_DEV_BAD_ACCEPT);
        na = 0;
    } else if (s_bad_page) {
        if (tid == 0) flag_status(status, OWL_DEV_BAD_PAGE);
        na = 0;
    }
    if (g == 0 && blockIdx.z == 0 && tid == 0 && new_ctx_lens) new_ctx_lens[b] = L + na;

    const int ppr = row_bytes / 16;
    const int total = na * ppr;
    uint4 held[kCommitMaxPieces];
#pragma unroll
    for (int r = 0; r < kCommitMaxPieces; ++r) {
        const int id = tid + r * kCommitThreads;
        if (id < total && s_src[id / ppr] != id / ppr) {    // a row already in place is left alone
            const int i = id / ppr, piece = id % ppr;
            const int pos = L + s_src[i];
            const int64_t off = (s_src_page[i] * stride_page + g * stride_head + (pos % kPage) * stride_token) * es;
            held[r] = *reinterpret_cast<const uint4 *>(cache + off + piece * 16);
        }
    }
    __syncthreads();                                        // all reads done before the first write
#pragma unroll
    for (int r = 0; r < kCommitMaxPieces; ++r) {
        const int id = tid + r * kCommitThreads;
        if (id < total) {
            const int i = id / ppr, piece = id % ppr;
            if (s_src[i] != i) {
                const int pos = L + i;
                const int64_t off = (s_dst_page[i] * stride_page + g * stride_head + (pos % kPage) * stride_token) * es;
                *reinterpret_cast<uint4 *>(cache + off + piece * 16) = held[r];
            }
        }
    }
}

hipError_t launch_commit(const owl_verify_desc &d, void *k_cache, void *v_cache, const int32_t *page_table,
                         const int32_t *ctx_lens, const int32_t *accepted, const int32_t *n_accept,
                         int32_t *new_ctx_lens, uint32_t *status, hipStream_t s)
{
    const int es = d.qkv_dtype == OWL_F32 ? 4 : 2;
    const int row_bytes = d.head_dim * es;
    static_assert(64 * 32 <= kCommitThreads * kCommitMaxPieces, "64 rows of up to 512 bytes fit the held pieces");
    hipLaunchKernelGGL(commit_kernel, dim3(d.n_kv_heads, d.batch, 2), dim3(kCommitThreads), 0, s,
                       static_cast<unsigned char *>(k_cache), static_cast<unsigned char *>(v_cache), page_table,
                       ctx_lens, accepted, n_accept, d.n_draft, d.max_pages_per_seq, d.max_ctx_len,
                       d.n_pool_pages, row_bytes, es, d.kv_stride_page, d.kv_stride_head, d.kv_stride_token,
                       new_ctx_lens, status);
    return hipGetLastError();
}

}  // namespace owl
