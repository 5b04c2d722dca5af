// Host side of the C ABI: argument checks, the split plan, kernel launches.
#include <math.h>
#include <string.h>

#include <atomic>
#include <mutex>

#include "owl_internal.h"
#include "owl_probe.h"

using namespace owl;

namespace {

int elem_size(int dtype) { return dtype == OWL_F32 ? 4 : 2; }

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Compute units of the current device; 256 (an MI355X) when no device answers,
// so that planning stays usable for host-only checks.
int device_cus()
{
    static std::atomic<int> cached[16];            // zero-initialised; callers may be on any thread
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

owl_status check_desc(const owl_verify_desc *d)
{
    if (!d) return OWL_ERR_INVALID_ARG;
    if (d->batch < 1 || d->n_draft < 1 || d->n_q_heads < 1 || d->n_kv_heads < 1) return OWL_ERR_INVALID_ARG;
    if (d->n_draft > 64) return OWL_ERR_TOO_MANY_DRAFT;
    if (d->n_q_heads % d->n_kv_heads) return OWL_ERR_INVALID_ARG;
    if (d->qkv_dtype != OWL_BF16 && d->qkv_dtype != OWL_F32 && d->qkv_dtype != OWL_F16) return OWL_ERR_UNSUPPORTED;
    if (d->head_dim != 64 && d->head_dim != 128) return OWL_ERR_UNSUPPORTED;
    if (d->page_size != kPage) return OWL_ERR_UNSUPPORTED;
    if (d->max_ctx_len < 0 || d->max_ctx_len > (1 << 30)) return OWL_ERR_INVALID_ARG;
    if (d->max_pages_per_seq < 0 || d->n_pool_pages < 1) return OWL_ERR_INVALID_ARG;
    if (d->split_tokens < 0) return OWL_ERR_INVALID_ARG;
    if (d->out_dtype != OWL_F32 && d->out_dtype != OWL_BF16 && d->out_dtype != OWL_F16) return OWL_ERR_UNSUPPORTED;
    if ((d->flags & ~(int32_t)OWL_FLAG_FP32_PARTIALS) != 0 || d->reserved_ != 0) return OWL_ERR_INVALID_ARG;
    if (!(d->scale > 0.0f) || !isfinite(d->scale)) return OWL_ERR_INVALID_ARG;
    const int es = elem_size(d->qkv_dtype);
    const int64_t st[3] = {d->kv_stride_page, d->kv_stride_head, d->kv_stride_token};
    for (int64_t s : st)
        if (s < 0 || (s * es) % 16 != 0) return OWL_ERR_INVALID_ARG;
    if (d->kv_stride_token < d->head_dim) return OWL_ERR_INVALID_ARG;
    if ((int64_t)d->n_q_heads / d->n_kv_heads * d->n_draft > 64 * 64) return OWL_ERR_UNSUPPORTED;
    return OWL_OK;
}

struct FullPlan {
    owl_plan pub;
    const Variant *variant;
    size_t part_o_bytes;
    bool half_partials;       // normalised fp16 partials (16-bit inputs unless the caller asks for fp32 ones)
    int32_t group_tiles;
    bool dealt;               // the kernels cut the work by the actual lengths (deal_units)
    DealRule rule;
    int32_t n_slots;
    Deal full;                // one sequence of the greatest length
    dim3 grid;                // of the split-KV pass
};

owl_status make_plan(const owl_verify_desc *d, FullPlan *fp)
{
    owl_status st = check_desc(d);
    if (st != OWL_OK) return st;
    const int G = d->n_q_heads / d->n_kv_heads;
    const int R = G * d->n_draft;
    const int RT = (R + kRowTile - 1) / kRowTile;
    const int64_t T = (int64_t)d->max_ctx_len + d->n_draft;
    // shortest split the planner uses: the fp16 partials of a split (R rows) stay below an eighth of the K/V it reads
    int64_t cmin = align_up((size_t)(4 * R), kSplitQuantum);
    if (cmin < 256) cmin = 256;
    // Eight wavefronts per workgroup: WR of them split the row tiles, WK the
    // 32-key steps of a stage; a wave holds up to three tiles in accumulators.
    // A workgroup takes up to 4 (WK = 2) or 8, 16, 24 (WK = 1; 7 and 8 on long
    // shares WK = 2) row tiles; more tiles than that go to further row groups, workgroups that read the same
    // split.  Few KV streams (one or two KV heads of a tensor-parallel shard, one
    // sequence) cannot fill the chip by splits alone without the partials
    // outgrowing the K/V they summarise: then the rows are cut into more, smaller
    // groups instead, each re-reading the split from its XCD's L2.
    int tpw, wr, wk, rgs, group_tiles;
    if (d->qkv_dtype == OWL_F32) {
        tpw = 1; wr = 8; wk = 1; rgs = (RT + 7) / 8;
        group_tiles = (RT + rgs - 1) / rgs;
    } else {
        static const int caps[4] = {24, 16, 8, 4};
        auto groups_of = [&](int l) { return (RT + caps[l] - 1) / caps[l]; };
        auto splits_of = [&](int64_t least) { return T <= least ? (int64_t)1 : (T + least - 1) / least; };
        // (three quarters of the compute units will do: larger groups do more per K/V byte they read)
        auto fills = [&](int groups, int64_t least) {
            return 4 * (int64_t)d->batch * d->n_kv_heads * splits_of(least) * groups >= 3 * (int64_t)device_cus();
        };
        const int largest = RT <= 4 ? 3 : (RT <= 8 ? 2 : (RT <= 16 ? 1 : 0));
        int li = largest;
        while (li < 3 && !fills(groups_of(li), d->split_tokens > 0 ? (int64_t)align_up((size_t)d->split_tokens, kSplitQuantum) : cmin)) ++li;
        // Where splits of 4 R tokens reach that only with more than two groups, two are taken all the same if splits of `least`
        // tokens reach it: more groups re-read the K/V from L2 more often than the longer shares cost.  How far below
        // 4 R that holds was measured against the plan by 4 R.  Lone sequences in bf16, two groups / that plan, at 2 R, 2.5 R, 3.2 R and 4 R:
        //   9-12 tiles, from three groups: 6 heads 1.03 1.02 0.99 0.99, but 1 head 1.04 1.04 1.01 1.00, 3 heads 1.05 1.04 1.02
        //   1.01 (two groups leave a SIMD two tiles, three groups one; with 1 head a row has 128 partials to merge, not 80).  With 6 to
        //   8 heads, bf16 and fp16, between 2.75 R and 3.75 R: 9 tiles 0.96-1.02 with no trend, 10 to 12 tiles 0.95-1.02 below and
        //   0.95-1.00 from 3.3 R on but for one of 30 (1.026);
        //   13-16, from four: 6 heads 0.97 0.94 0.93 0.90, 1 head 1.03 0.99 0.97 0.94, 3 heads 1.02 0.97 0.96 0.93;
        //   13-20, 1 head, head_dim 64, at 2 R, 2.5 R, 3 R and 3.5 R: 1.03 1.02 0.99 0.97 (few bytes, and again the merge; 22 tiles 0.92);
        //   17-32, from three to six: 0.96 0.94 0.92 0.90, never above 1.006 but for one run;
        //   37-40, and all from five or six: 0.95 0.94 0.92 0.91;
        //   33-36 and 41-48, from three groups of two tiles a wavefront, head_dim 128: 1.05 1.04 1.03 1.02 and 1.01 1.00 1.00 1.00
        //   (a SIMD has two times five or six tiles against three times three or four, in the kernel that spills; with 37-40 it is
        //   two times five against three times four); head_dim 64: 0.96.
        // In a batch the lengths are bounds, and how sequences fall on the workers decides.  500 random batches of 2 to 16, two groups at
        // 2 R / the plan by 4 R: from three groups 1.02 on average (0.88-1.18), from five 1.01, from six 0.93 (0.81-1.03 but for one
        // of very uneven lengths 1.13); from four 0.99 (0.86-1.14), but 0.96 (1.05 at most) where the batch in all, without
        // rounding each sequence up, comes to splits of 3 R.
        const int more = groups_of(li);
        if (d->split_tokens == 0 && more > 2) {
            const bool level = RT >= 37 && RT <= 40, many_heads = d->n_kv_heads >= 6;
            int eighths = 8;                            // of 4 R
            if (d->batch > 1) {
                const bool enough = 4 * (int64_t)d->batch * T * d->n_kv_heads * 2 >= 3 * (int64_t)device_cus() * (cmin * 6 / 8);
                if (more >= 6 || (more == 4 && enough)) eighths = 4;
            } else if (RT <= 12) eighths = !many_heads || RT == 9 ? 8 : 7;
            else if (RT <= 20 && d->head_dim == 64 && d->n_kv_heads == 1) eighths = 6;
            else if (RT <= 16) eighths = many_heads ? 4 : 5;
            else if (RT <= 32 || more > 3 || level || d->head_dim == 64) eighths = 4;
            int two = largest;
            while (groups_of(two) < 2) ++two;
            const int64_t least = cmin * eighths / 8;
            if (groups_of(two) == 2 && fills(2, least)) li = two;
        }
        rgs = (RT + caps[li] - 1) / caps[li];
        group_tiles = (RT + rgs - 1) / rgs;
        rgs = (RT + group_tiles - 1) / group_tiles;
        // Seven or eight tiles: eight wavefronts with one each, or four pairs with two each, a pair splitting the steps of a
        // stage.  That halves the fragments read from LDS, and with them the power that limits the loop, but a workgroup then
        // has a merge of its own in every piece and no pipelined loop: it pays where a worker has many stages and its pieces are
        // not short, the sooner the fuller the pairs are.  us, one tile -> two, 8 KV heads, bf16, sequences of S stages each, a
        // worker's share 256 stages (64 where it says so): 104 rows, S = 8 / 32 / 128 / 512 / 2048 1004 -> 1020 / 477 -> 476 /
        // 377 -> 370 / 361 -> 343 / 358 -> 341, but with shares of 64 121 -> 121 / 102.4 -> 103.0 / 98.1 -> 99.0 / 96.4 -> 93.9
        // from S = 32 on; 128 rows 1093 -> 1109 / 498 -> 497 / 396 -> 382 / 381 -> 360 / 378 -> 356, and with 64 126 -> 126 /
        // 104.7 -> 104.4 / 102.5 -> 99.5 / 101.2 -> 96.8.  A caller's splits of 1 / 4 / 16 / 64 stages, 104 rows: 1858 -> 2089 /
        // 717 -> 750 / 460 -> 464 / 390 -> 388.  fp16 and head_dim 64 gain more from S = 32 on (1-7 %) and lose as much at S = 8
        // (1-4 %).  What is known here is the greatest length: 128 rows announced as 128K and 4K long take 16.1 instead of
        // 15.6.  Five and six tiles gain nothing (80 rows, share 512: 442 -> 441).
        const int64_t stages = (T + kSplitQuantum - 1) / kSplitQuantum;
        const int64_t share = (int64_t)d->batch * stages * d->n_kv_heads * rgs / device_cus();
        const int64_t split = (int64_t)align_up((size_t)d->split_tokens, kSplitQuantum) / kSplitQuantum;
        const int64_t piece = d->split_tokens > 0 && split < stages ? split : stages;
        if (caps[li] == 4) { tpw = 1; wr = 4; wk = 2; }
        else if (caps[li] == 8 && group_tiles >= 7 && piece >= 32 && share >= (group_tiles == 8 ? 64 : 256)) { tpw = 2; wr = 4; wk = 2; }
        else { wr = 8; wk = 1; tpw = (group_tiles + 7) / 8; }
    }
    const Variant *v = find_variant(d->qkv_dtype, d->head_dim, tpw, wr, wk);
    if (!v) return OWL_ERR_UNSUPPORTED;
    fp->group_tiles = group_tiles;
    int64_t C;
    if (d->split_tokens > 0) {
        C = align_up((size_t)d->split_tokens, kSplitQuantum);
    } else {
        // Enough workgroups to occupy every compute unit (several rounds when
        // many independent KV streams exist, which evens out ragged batches),
        // but splits long enough that the partials they write stay a small
        // fraction of the K/V bytes they read (ratio ~ R / 2C with fp16 partials).
        const int64_t streams = (int64_t)d->batch * d->n_kv_heads * rgs;
        const int rounds = streams >= 64 ? 4 : 1;
        const int64_t want = (int64_t)device_cus() * rounds;      // one workgroup per CU at a time
        // A single round must not spill a few workgroups into a second one.  With row groups the
        // kernel keeps the groups of a (KV head, split) on one XCD, streams dealt round-robin over
        // the eight XCDs: what has to fit is an XCD's share of the streams times the groups.
        int64_t S = (want + streams - 1) / streams;
        if (rounds == 1) {
            S = want / streams;
            if (rgs > 1) {
                const int64_t per_xcd = device_cus() / 8 / rgs;              // streams an XCD can hold at once
                const int64_t heads = (int64_t)d->batch * d->n_kv_heads;
                if (per_xcd >= 1 && 8 * per_xcd / heads >= 1) S = 8 * per_xcd / heads;
            }
        }
        if (S < 1) S = 1;
        C = align_up((size_t)((T + S - 1) / S), kSplitQuantum);
        if (C < cmin) C = cmin;
    }
    if (C > kMaxSplitTokens) C = kMaxSplitTokens;
    if (C < kSplitQuantum) C = kSplitQuantum;
    int64_t max_splits = (T + C - 1) / C;
    // A library-chosen split size: what is launched is a set of workers that share out the actual
    // lengths (deal_units), one workgroup per compute unit.  The worker count follows the same two rules as
    // above: fill the compute units in one round, and keep the row groups of a stream on one XCD.
    // A share is never below R tokens: there the fp16 partials it leaves are half the K/V it reads (a share of
    // 4 R, which keeps them to an eighth, costs a 5K context with 240 rows 2 us of 20 and a 512-token fp32
    // call 9 us of 20: short calls are bound by the chain of stages, not by bytes; R / 4 gains nothing more).
    // Beyond its stages a sequence counts 8 units in a batch, where the worker that ends it begins the next
    // one with a set-up and an empty ring (0 instead of 8: 284 against 259 us on four sequences of 3K-16K
    // tokens with 240 rows in four layers; 4: 268, 10: 260), and 1-2 for the masked steps of a lone sequence.
    const int64_t stages_at_most = (T + kSplitQuantum - 1) / kSplitQuantum;
    fp->rule.seq_extra = d->batch == 1 ? (RT > 4 ? 2 : 1) : 8;
    const int64_t units_at_most = (int64_t)d->batch * (stages_at_most + fp->rule.seq_extra);
    fp->dealt = d->split_tokens == 0 && units_at_most < ((int64_t)1 << 30);
    const int64_t head_groups = (int64_t)d->n_kv_heads * rgs;
    int64_t per_round = 1;
    for (int k = 1; k <= 4; ++k) {                  // more heads than compute units divide evenly into: up to four rounds
        per_round = (int64_t)device_cus() * k / head_groups;
        if (rgs > 1) {
            const int64_t streams = (int64_t)(device_cus() / 8 / rgs) * 8 * k;
            if (streams >= d->n_kv_heads) per_round = streams / d->n_kv_heads;
        }
        if (per_round >= 1 && 20 * per_round * head_groups >= 17 * (int64_t)device_cus() * k) break;
        if (per_round > 4) break;
    }
    if (per_round < 1) per_round = 1;
    fp->rule.round_workers = (int32_t)per_round;
    fp->rule.min_units = (R + kSplitQuantum - 1) / kSplitQuantum;
    fp->rule.merge = d->batch == 1 && RT <= 4 && d->qkv_dtype != OWL_F32 ? kMergeUnits : 0;
    int64_t workers = fp->rule.max_workers = 1;
    fp->full = Deal{1, 0, 0};
    if (fp->dealt) {                                // (no shorter length asks for more workers than the greatest)
        fp->rule.max_workers = workers = most_workers(fp->rule, (int)units_at_most);
        fp->full = deal_units(fp->rule, (int)units_at_most);
    }
    // Workspace: the partials that are written, and never less than equal splits of half the planned size
    // would need for a batch (the planned size for one sequence).
    fp->half_partials = d->qkv_dtype != OWL_F32 && !(d->flags & OWL_FLAG_FP32_PARTIALS);
    const size_t o_bytes = (size_t)d->head_dim * kRowTile * (fp->half_partials ? 2 : 4), ml_bytes = kPartMl * sizeof(float);
    auto bytes_of = [&](size_t slots, size_t unit) -> size_t { return align_up((size_t)d->n_kv_heads * slots * RT * unit, 256); };
    auto partials = [&](size_t slots) -> size_t { return bytes_of(slots, o_bytes) + bytes_of(slots, ml_bytes); };
    int64_t sized_splits = max_splits;
    if (d->split_tokens == 0 && d->batch > 1 && units_at_most < ((int64_t)1 << 30)) {
        int64_t c_floor = align_up((size_t)(C / 2), kSplitQuantum);
        if (c_floor < cmin) c_floor = cmin < C ? cmin : C;
        sized_splits = (T + c_floor - 1) / c_floor;
    }
    const size_t sized = partials((size_t)d->batch * (size_t)sized_splits), dealt_bytes = partials((size_t)(workers + d->batch - 1));
    // A dealt launch leaves one partial per worker, in a batch also one per sequence: that may be several times what few
    // equal splits of short sequences leave.  What owl_verify_attn_noalloc admits must not depend on how the work is
    // dealt out, so a launch that fits its scratch in equal splits only has as many workers as fit, or, where those
    // would be fewer than the splits, equal splits.
    if (fp->dealt && dealt_bytes > OWL_NOALLOC_SCRATCH_BYTES && sized <= OWL_NOALLOC_SCRATCH_BYTES) {
        int64_t room = (int64_t)(OWL_NOALLOC_SCRATCH_BYTES / partials(1)) - (d->batch - 1);      // partials(1) is rounded up
        if (room >= (int64_t)d->batch * max_splits && (units_at_most + room - 1) / room <= kMaxPieceUnits) {
            fp->rule.max_workers = workers = room;
            fp->full = deal_units(fp->rule, (int)units_at_most);
        } else {
            fp->dealt = false;
        }
    }
    const size_t n_slots = fp->dealt ? (size_t)(workers + d->batch - 1) : (size_t)d->batch * (size_t)max_splits;
    fp->n_slots = (int32_t)n_slots;
    if (fp->dealt) max_splits = sized_splits;
    fp->part_o_bytes = bytes_of(n_slots, o_bytes);
    fp->variant = v;
    owl_plan &pl = fp->pub;
    pl.reserved_ = 0;
    pl.split_tokens = (int32_t)C;
    pl.max_splits = (int32_t)max_splits;
    pl.rows_per_kv = R;
    pl.row_tiles = RT;
    pl.row_groups = rgs;
    pl.tiles_per_wave = tpw;
    pl.kernel_variant = variant_index(v);
    // KV heads vary fastest (see the kernel's block-index comment).
    // With row groups the kernel deals the workgroups out in units of eight (KV head, share) streams: the
    // grid is padded so that their number is a multiple of 8 (the surplus exits at once).
    int64_t grid_y = fp->dealt ? workers : max_splits;
    const int64_t grid_z = fp->dealt ? 1 : d->batch;
    if (rgs > 1)
        while (((int64_t)d->n_kv_heads * grid_y * grid_z) % 8 != 0) ++grid_y;
    fp->grid = dim3(d->n_kv_heads * rgs, (unsigned)grid_y, (unsigned)grid_z);
    if ((int64_t)fp->grid.x * fp->grid.y * fp->grid.z >= ((int64_t)1 << 31)) return OWL_ERR_UNSUPPORTED;   // the kernel numbers them in 32 bits
    pl.n_workgroups = (int32_t)((int64_t)fp->grid.x * fp->grid.y * fp->grid.z);
    pl.workspace_bytes = partials(n_slots) > sized ? partials(n_slots) : sized;
    return OWL_OK;
}

// Kernels that need more than the default dynamic LDS must say so once per
// device before their first launch.
owl_status ensure_lds_attr(const Variant *v)
{
    static std::mutex mu;
    static bool done[16][64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return OWL_ERR_HIP;
    const int vi = variant_index(v);
    if (dev < 0 || dev >= 16 || vi < 0 || vi >= 64) return OWL_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev][vi]) {
        if (hipFuncSetAttribute(v->func, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)v->lds_bytes) != hipSuccess)
            return OWL_ERR_HIP;
        done[dev][vi] = true;
    }
    return OWL_OK;
}

// Device memory of owl_verify_attn_noalloc: the split partials live here instead of in a
// caller's workspace.  One copy per GPU that loads the library, held until the process ends.
// In host code the array's name is only a handle: its device address comes from
// hipGetSymbolAddress, once per device (scratch_address), and only that address is ever
// handed to a kernel.
static __device__ __align__(256) unsigned char scratch[OWL_NOALLOC_SCRATCH_BYTES];

owl_status scratch_address(void **out)
{
    static std::mutex mu;
    static void *addr[16] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 16) return OWL_ERR_HIP;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return OWL_ERR_HIP;
        addr[dev] = ptr;
    }
    *out = addr[dev];
    return OWL_OK;
}

bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) != 0; }

}  // namespace

extern "C" {

owl_status owl_verify_attn_plan(const owl_verify_desc *desc, owl_plan *plan)
{
    if (!plan) return OWL_ERR_INVALID_ARG;
    FullPlan fp;
    owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    *plan = fp.pub;
    return OWL_OK;
}

owl_status owl_verify_attn_workspace_size(const owl_verify_desc *desc, size_t *bytes)
{
    if (!bytes) return OWL_ERR_INVALID_ARG;
    FullPlan fp;
    owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    *bytes = fp.pub.workspace_bytes;
    return OWL_OK;
}

owl_status owl_verify_attn(const owl_verify_desc *desc, const void *q, const void *k_cache,
                           const void *v_cache, const int32_t *page_table,
                           const int32_t *ctx_lens, const int32_t *tree_parent, void *out,
                           void *workspace, size_t workspace_bytes, uint32_t *dev_status,
                           void *stream)
{
    return owl_verify_attn_phases(desc, q, k_cache, v_cache, page_table, ctx_lens, tree_parent, out,
                                  workspace, workspace_bytes, dev_status, stream, OWL_PHASE_ALL);
}

static owl_status verify_impl(const owl_verify_desc *desc, const void *q, const void *k_cache,
                              const void *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
                              const int32_t *tree_parent, const int32_t *n_draft_seq, void *out,
                              void *workspace, size_t workspace_bytes, uint32_t *dev_status, void *stream,
                              int32_t phases, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);

owl_status owl_verify_attn_phases(const owl_verify_desc *desc, const void *q, const void *k_cache,
                                  const void *v_cache, const int32_t *page_table,
                                  const int32_t *ctx_lens, const int32_t *tree_parent, void *out,
                                  void *workspace, size_t workspace_bytes, uint32_t *dev_status,
                                  void *stream, int32_t phases)
{
    return verify_impl(desc, q, k_cache, v_cache, page_table, ctx_lens, tree_parent, nullptr, out, workspace,
                       workspace_bytes, dev_status, stream, phases);
}

owl_status owl_verify_attn_ragged(const owl_verify_desc *desc, const void *q, const void *k_cache,
                                  const void *v_cache, const int32_t *page_table,
                                  const int32_t *ctx_lens, const int32_t *tree_parent,
                                  const int32_t *n_draft_seq, void *out, void *workspace,
                                  size_t workspace_bytes, uint32_t *dev_status, void *stream)
{
    if (!n_draft_seq) return OWL_ERR_INVALID_ARG;
    return verify_impl(desc, q, k_cache, v_cache, page_table, ctx_lens, tree_parent, n_draft_seq, out,
                       workspace, workspace_bytes, dev_status, stream, OWL_PHASE_ALL);
}

static owl_status verify_impl(const owl_verify_desc *desc, const void *q, const void *k_cache,
                              const void *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
                              const int32_t *tree_parent, const int32_t *n_draft_seq, void *out,
                              void *workspace, size_t workspace_bytes, uint32_t *dev_status, void *stream,
                              int32_t phases, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (phases < 1 || phases > OWL_PHASE_ALL) return OWL_ERR_INVALID_ARG;
    FullPlan fp;
    owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    if (!q || !k_cache || !v_cache || !ctx_lens || !tree_parent || !out) return OWL_ERR_INVALID_ARG;
    if (misaligned(q, 16) || misaligned(k_cache, 16) || misaligned(v_cache, 16) || misaligned(out, 16))
        return OWL_ERR_INVALID_ARG;
    if (page_table &&
        (int64_t)desc->max_pages_per_seq * kPage < (int64_t)desc->max_ctx_len + desc->n_draft)
        return OWL_ERR_INVALID_ARG;
    if (!workspace || workspace_bytes < fp.pub.workspace_bytes) return OWL_ERR_WORKSPACE;
    if (misaligned(workspace, 256)) return OWL_ERR_INVALID_ARG;

    // the profiling copy of the kernel, if the timeline hook is on and has room for this grid
    const Variant *variant = fp.variant;
    const TimelineHook hook = timeline_hook();
    if (hook.buffer && fp.pub.n_workgroups <= hook.capacity) {
        const Variant *tv = find_variant(variant->dtype, variant->D, variant->tpw, variant->wr, variant->wk, true);
        if (tv) variant = tv;
    }
    st = ensure_lds_attr(variant);
    if (st != OWL_OK) return st;

    // workspace: partial O | partial (m, l, s)
    char *ws = static_cast<char *>(workspace);
    KParams p;
    memset(&p, 0, sizeof p);
    p.q = q; p.k = k_cache; p.v = v_cache;
    p.page_table = page_table; p.ctx_lens = ctx_lens; p.parent = tree_parent;
    p.n_draft_seq = n_draft_seq;
    p.part_o = ws;
    p.half_partials = fp.half_partials ? 1 : 0;
    p.part_ml = reinterpret_cast<float *>(ws + fp.part_o_bytes);
    p.out = out;
    p.out_dtype = desc->out_dtype;
    p.dev_status = dev_status;
    p.B = desc->batch; p.N = desc->n_draft; p.Hq = desc->n_q_heads; p.Hkv = desc->n_kv_heads;
    p.G = p.Hq / p.Hkv; p.R = fp.pub.rows_per_kv;
    p.max_pages = desc->max_pages_per_seq; p.max_ctx_len = desc->max_ctx_len;
    p.C = fp.pub.split_tokens; p.max_splits = fp.pub.max_splits;
    p.dealt = fp.dealt ? 1 : 0; p.rule = fp.rule; p.n_slots = fp.n_slots;
    p.full = fp.full;
    p.full_pieces = fp.dealt ? deal_worker(fp.full, stages_of((int)(desc->max_ctx_len + desc->n_draft)) - 1) + 1 : 0;
    p.RT = fp.pub.row_tiles; p.row_groups = fp.pub.row_groups; p.group_tiles = fp.group_tiles;
    p.stride_page = desc->kv_stride_page; p.stride_head = desc->kv_stride_head;
    p.stride_token = desc->kv_stride_token; p.n_pool_pages = desc->n_pool_pages;
    p.c_log2 = desc->scale * 1.4426950408889634f;
    p.timeline = variant->timeline ? hook.buffer : nullptr;

    hipStream_t s = static_cast<hipStream_t>(stream);
    if (phases & OWL_PHASE_SPLIT) {
        variant->launch(p, fp.grid, s, ev_start, ev_stop);
        if (hipGetLastError() != hipSuccess) return OWL_ERR_HIP;
    }
    if (phases & OWL_PHASE_COMBINE)
        if (launch_combine(p, desc->head_dim, fp.half_partials, s) != hipSuccess) return OWL_ERR_HIP;
    return OWL_OK;
}

// ---- measurement aids that need the verify path itself (declared in owl_probe.h) ----
owl_status owl_verify_attn_split_timed(const owl_verify_desc *desc, const void *q, const void *k_cache,
                                       const void *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
                                       const int32_t *tree_parent, void *out, void *workspace, size_t workspace_bytes,
                                       uint32_t *dev_status, void *stream, void *start_event, void *stop_event)
{
    if (!start_event || !stop_event) return OWL_ERR_INVALID_ARG;
    return verify_impl(desc, q, k_cache, v_cache, page_table, ctx_lens, tree_parent, nullptr, out, workspace,
                       workspace_bytes, dev_status, stream, OWL_PHASE_SPLIT, static_cast<hipEvent_t>(start_event),
                       static_cast<hipEvent_t>(stop_event));
}

owl_status owl_probe_deal(const owl_verify_desc *desc, const int32_t *tokens, int32_t capacity, int32_t *pieces,
                          int32_t *ranges, int32_t *info)
{
    if (!tokens || !pieces || !ranges || !info || capacity < 0) return OWL_ERR_INVALID_ARG;
    FullPlan fp;
    const owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    int64_t total = 0;
    for (int b = 0; b < desc->batch; ++b) {
        if (tokens[b] < 0 || tokens[b] > (int64_t)desc->max_ctx_len + desc->n_draft) return OWL_ERR_INVALID_ARG;
        if (fp.dealt) total += seq_units(fp.rule, tokens[b]);
    }
    int32_t n = 0;
    auto piece = [&](int worker, int b, int first, int end, int slot) {
        if (n < capacity) {
            const int32_t row[5] = {worker, b, first, end, slot};
            memcpy(pieces + 5 * (size_t)n, row, sizeof row);
        }
        ++n;
    };
    info[1] = fp.n_slots;
    info[2] = fp.dealt ? 1 : 0;
    info[3] = fp.dealt ? fp.rule.max_workers : desc->batch * fp.pub.max_splits;
    if (!fp.dealt) {
        for (int b = 0; b < desc->batch; ++b) {
            const int splits = (int)(((int64_t)tokens[b] + fp.pub.split_tokens - 1) / fp.pub.split_tokens);
            for (int c = 0; c < splits; ++c) {
                const int64_t end = ((int64_t)c + 1) * fp.pub.split_tokens;
                piece(b * fp.pub.max_splits + c, b, c * fp.pub.split_tokens, (int)(end < tokens[b] ? end : tokens[b]),
                      b * fp.pub.max_splits + c);
            }
            ranges[2 * b] = b * fp.pub.max_splits;
            ranges[2 * b + 1] = splits;
        }
        info[0] = n;
        return OWL_OK;
    }
    const Deal deal = desc->batch == 1 && tokens[0] == desc->max_ctx_len + desc->n_draft
                          ? fp.full : deal_units(fp.rule, total > 0 ? (int)total : 1);
    for (int w = 0; w < deal.workers && total > 0; ++w) {
        const int x0 = deal_begin(deal, w), x1 = deal_begin(deal, w + 1);
        for (int b = 0, before = 0; b < desc->batch; before += seq_units(fp.rule, tokens[b]), ++b) {
            const int s0 = (x0 > before ? x0 : before) - before;
            const int s1 = x1 - before < stages_of(tokens[b]) ? x1 - before : stages_of(tokens[b]);
            if (s0 < s1)
                piece(w, b, s0 * kSplitQuantum, s1 * kSplitQuantum < tokens[b] ? s1 * kSplitQuantum : tokens[b], w + b);
        }
    }
    for (int b = 0, before = 0; b < desc->batch; before += seq_units(fp.rule, tokens[b]), ++b) {
        ranges[2 * b] = ranges[2 * b + 1] = 0;
        if (tokens[b] == 0) continue;
        const int w0 = deal_worker(deal, before);
        ranges[2 * b] = w0 + b;
        ranges[2 * b + 1] = deal_worker(deal, before + stages_of(tokens[b]) - 1) - w0 + 1;
    }
    info[0] = n;
    return OWL_OK;
}

owl_status owl_probe_event_create(void **event)
{
    if (!event) return OWL_ERR_INVALID_ARG;
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return OWL_ERR_HIP;
    *event = e;
    return OWL_OK;
}

owl_status owl_probe_event_destroy(void *event)
{
    if (!event) return OWL_ERR_INVALID_ARG;
    return hipEventDestroy(static_cast<hipEvent_t>(event)) == hipSuccess ? OWL_OK : OWL_ERR_HIP;
}

owl_status owl_probe_event_elapsed_ms(void *start_event, void *stop_event, float *ms_host)
{
    if (!start_event || !stop_event || !ms_host) return OWL_ERR_INVALID_ARG;
    if (hipEventSynchronize(static_cast<hipEvent_t>(stop_event)) != hipSuccess) return OWL_ERR_HIP;
    return hipEventElapsedTime(ms_host, static_cast<hipEvent_t>(start_event), static_cast<hipEvent_t>(stop_event)) == hipSuccess
               ? OWL_OK : OWL_ERR_HIP;
}

owl_status owl_verify_attn_init(const owl_verify_desc *desc)
{
    FullPlan fp;
    owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    st = ensure_lds_attr(fp.variant);
    if (st != OWL_OK) return st;
    if (load_aux_kernels() != hipSuccess) return OWL_ERR_HIP;
    void *ptr = nullptr;
    return scratch_address(&ptr);
}

owl_status owl_verify_attn_noalloc(const owl_verify_desc *desc, const void *q, const void *k_cache,
                                   const void *v_cache, const int32_t *page_table, const int32_t *ctx_lens,
                                   const int32_t *tree_parent, void *out, uint32_t *dev_status, void *stream)
{
    FullPlan fp;
    owl_status st = make_plan(desc, &fp);
    if (st != OWL_OK) return st;
    if (fp.pub.workspace_bytes > (size_t)OWL_NOALLOC_SCRATCH_BYTES) return OWL_ERR_WORKSPACE;
    void *ptr = nullptr;
    st = scratch_address(&ptr);
    if (st != OWL_OK) return st;
    return verify_impl(desc, q, k_cache, v_cache, page_table, ctx_lens, tree_parent, nullptr, out, ptr,
                       (size_t)OWL_NOALLOC_SCRATCH_BYTES, dev_status, stream, OWL_PHASE_ALL);
}

owl_status owl_build_tree_mask(const int32_t *tree_parent, int32_t batch, int32_t n_draft,
                               uint64_t *anc_mask, int32_t *depth, uint32_t *dev_status,
                               void *stream)
{
    if (!tree_parent || !anc_mask || batch < 1 || n_draft < 1) return OWL_ERR_INVALID_ARG;
    if (n_draft > 64) return OWL_ERR_TOO_MANY_DRAFT;
    if (launch_tree_mask(tree_parent, batch, n_draft, anc_mask, depth, dev_status,
                         static_cast<hipStream_t>(stream)) != hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

owl_status owl_prepare_spec_tree(const int32_t *tree_parent, const int32_t *ctx_lens, int32_t batch,
                                 int32_t n_nodes, int32_t *tree_parent2, uint64_t *anc_mask,
                                 int32_t *depth, int32_t *pos_ids, uint32_t *dev_status, void *stream)
{
    if (!tree_parent || !ctx_lens || !tree_parent2 || !anc_mask || batch < 1 || n_nodes < 1)
        return OWL_ERR_INVALID_ARG;
    if (n_nodes > 32) return OWL_ERR_TOO_MANY_DRAFT;
    if (launch_prepare(tree_parent, ctx_lens, batch, n_nodes, tree_parent2, anc_mask, depth, pos_ids,
                       dev_status, static_cast<hipStream_t>(stream)) != hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

owl_status owl_accept_greedy(const int32_t *tokens, const int32_t *tree_parent, const int32_t *target_root,
                             const int32_t *target_next, int32_t batch, int32_t n_draft, int32_t n_cand,
                             int32_t *accepted, int32_t *n_accept, int32_t *bonus, int32_t *last,
                             uint32_t *dev_status, void *stream)
{
    if (!tokens || !tree_parent || !target_root || !target_next || !accepted || !n_accept || !bonus || !last)
        return OWL_ERR_INVALID_ARG;
    if (batch < 1 || n_draft < 1 || n_cand < 0 || n_cand > n_draft) return OWL_ERR_INVALID_ARG;
    if (n_draft > 64) return OWL_ERR_TOO_MANY_DRAFT;
    if (launch_accept(tokens, tree_parent, target_root, target_next, batch, n_draft, n_cand, accepted,
                      n_accept, bonus, last, dev_status, static_cast<hipStream_t>(stream)) != hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

owl_status owl_commit_kv(const owl_verify_desc *desc, void *k_cache, void *v_cache, const int32_t *page_table,
                         const int32_t *ctx_lens, const int32_t *accepted, const int32_t *n_accept,
                         int32_t *new_ctx_lens, uint32_t *dev_status, void *stream)
{
    owl_status st = check_desc(desc);
    if (st != OWL_OK) return st;
    if (!k_cache || !v_cache || !ctx_lens || !accepted || !n_accept) return OWL_ERR_INVALID_ARG;
    if (new_ctx_lens == ctx_lens) return OWL_ERR_INVALID_ARG;
    if (misaligned(k_cache, 16) || misaligned(v_cache, 16)) return OWL_ERR_INVALID_ARG;
    if (page_table &&
        (int64_t)desc->max_pages_per_seq * kPage < (int64_t)desc->max_ctx_len + desc->n_draft)
        return OWL_ERR_INVALID_ARG;
    if (launch_commit(*desc, k_cache, v_cache, page_table, ctx_lens, accepted, n_accept, new_ctx_lens,
                      dev_status, static_cast<hipStream_t>(stream)) != hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

static owl_status check_drafter(const owl_drafter_desc *d)
{
    if (!d) return OWL_ERR_INVALID_ARG;
    if (d->d_in < 1 || d->d < 1 || d->n_states < 1 || d->n_rows < 1 || d->vocab < 1) return OWL_ERR_INVALID_ARG;
    if (!(d->eps >= 0.f) || d->alpha != d->alpha) return OWL_ERR_INVALID_ARG;
    if (d->n_states > 64 || d->n_rows > 64) return OWL_ERR_TOO_MANY_DRAFT;
    if (d->dtype != OWL_BF16 && d->dtype != OWL_F16) return OWL_ERR_UNSUPPORTED;
    if (d->d_in % 32 != 0 || d->d % 16 != 0 || d->d > 16384 || d->d_in > (1 << 20)) return OWL_ERR_UNSUPPORTED;
    if (d->w_layout != OWL_W_ROWS && d->w_layout != OWL_W_TILED) return OWL_ERR_UNSUPPORTED;
    return OWL_OK;
}

owl_status owl_drafter_tiled_weight_bytes(const owl_drafter_desc *desc, size_t *bytes)
{
    owl_status st = check_drafter(desc);
    if (st != OWL_OK) return st;
    if (!bytes) return OWL_ERR_INVALID_ARG;
    *bytes = drafter_tiled_bytes(desc->d_in, desc->d);
    return OWL_OK;
}

owl_status owl_drafter_tile_weights(const owl_drafter_desc *desc, const void *w_rows, void *w_tiled, void *stream)
{
    owl_status st = check_drafter(desc);
    if (st != OWL_OK) return st;
    if (!w_rows || !w_tiled || misaligned(w_rows, 16) || misaligned(w_tiled, 16)) return OWL_ERR_INVALID_ARG;
    if (launch_drafter_tile_weights(w_rows, w_tiled, desc->d_in, desc->d, static_cast<hipStream_t>(stream)) !=
        hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

owl_status owl_drafter_cell_workspace_size(const owl_drafter_desc *desc, size_t *bytes)
{
    owl_status st = check_drafter(desc);
    if (st != OWL_OK) return st;
    if (!bytes) return OWL_ERR_INVALID_ARG;
    // the projections [P][4d], then the chunk statistics of the two normalisations
    *bytes = ((size_t)desc->n_states * 4 * desc->d + drafter_gate_scratch_floats(desc->n_rows)) * sizeof(float);
    return OWL_OK;
}

owl_status owl_drafter_cell_phases(const owl_drafter_desc *desc, const void *h, const float *z,
                                   const int32_t *tokens, const int32_t *parent_row, const void *w,
                                   const void *emb, const float *gamma_c, const float *beta_c,
                                   const float *gamma_z, const float *beta_z, void *h_out, float *h_out_f32,
                                   float *z_out, void *workspace, size_t workspace_bytes, uint32_t *dev_status,
                                   void *stream, int32_t phases)
{
    owl_status st = check_drafter(desc);
    if (st != OWL_OK) return st;
    if (!h || !z || !tokens || !w || !emb || !z_out) return OWL_ERR_INVALID_ARG;
    if (phases < 1 || phases > OWL_DRAFTER_ALL) return OWL_ERR_INVALID_ARG;
    if (!parent_row && desc->n_rows != desc->n_states) return OWL_ERR_INVALID_ARG;
    for (const void *ptr : {h, (const void *)z, w, emb, (const void *)gamma_c, (const void *)beta_c,
                            (const void *)gamma_z, (const void *)beta_z, (const void *)h_out,
                            (const void *)h_out_f32, (const void *)z_out, (const void *)workspace})
        if (misaligned(ptr, 16)) return OWL_ERR_INVALID_ARG;      // a null pointer counts as aligned
    size_t need = 0;
    owl_drafter_cell_workspace_size(desc, &need);
    if (!workspace || workspace_bytes < need) return OWL_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *proj = static_cast<float *>(workspace);
    if (phases & OWL_DRAFTER_PROJ)
        if (launch_drafter_proj(desc->dtype, h, w, desc->w_layout == OWL_W_TILED, proj, desc->n_states, desc->d_in,
                                desc->d, device_cus(), s) != hipSuccess)
            return OWL_ERR_HIP;
    if (phases & OWL_DRAFTER_GATES)
        if (launch_drafter_gates(desc->dtype, proj, z, tokens, parent_row, emb, gamma_c, beta_c, gamma_z, beta_z,
                                 h_out, h_out_f32, z_out, proj + (size_t)desc->n_states * 4 * desc->d, desc->n_states,
                                 desc->n_rows, desc->d, desc->vocab,
                                 desc->alpha, desc->eps, dev_status, device_cus(), s) != hipSuccess)
            return OWL_ERR_HIP;
    return OWL_OK;
}

owl_status owl_drafter_cell(const owl_drafter_desc *desc, const void *h, const float *z, const int32_t *tokens,
                            const int32_t *parent_row, const void *w, const void *emb, const float *gamma_c,
                            const float *beta_c, const float *gamma_z, const float *beta_z, void *h_out,
                            float *h_out_f32, float *z_out, void *workspace, size_t workspace_bytes,
                            uint32_t *dev_status, void *stream)
{
    return owl_drafter_cell_phases(desc, h, z, tokens, parent_row, w, emb, gamma_c, beta_c, gamma_z, beta_z, h_out,
                                   h_out_f32, z_out, workspace, workspace_bytes, dev_status, stream,
                                   OWL_DRAFTER_ALL);
}

owl_status owl_drafter_alpha(int32_t max_depth, int32_t d, float *alpha_host)
{
    if (max_depth < 1 || d < 1 || !alpha_host) return OWL_ERR_INVALID_ARG;
    const double a0 = exp2(-1.0 / (2.0 * (double)max_depth));
    *alpha_host = (float)(2.0 * a0 / ((1.0 - a0 * a0) * (double)d));
    return OWL_OK;
}

owl_status owl_build_tree_mask_host(const int32_t *parent, int32_t n_draft, uint64_t *anc,
                                    int32_t *depth)
{
    if (!parent || !anc || n_draft < 1) return OWL_ERR_INVALID_ARG;
    if (n_draft > 64) return OWL_ERR_TOO_MANY_DRAFT;
    for (int i = 0; i < n_draft; ++i)
        if (parent[i] < -1 || parent[i] >= i) return OWL_ERR_BAD_TREE;
    // parents come first, so one forward sweep suffices
    for (int i = 0; i < n_draft; ++i) {
        const int pi = parent[i];
        anc[i] = ((uint64_t)1 << i) | (pi >= 0 ? anc[pi] : 0);
        if (depth) depth[i] = 1 + (pi >= 0 ? depth[pi] : 0);
    }
    return OWL_OK;
}

owl_status owl_gather_kv(const owl_verify_desc *desc, const void *cache, const int32_t *page_table,
                         int32_t seq, int64_t first_pos, int64_t n_tokens, void *dst,
                         uint32_t *dev_status, void *stream)
{
    owl_status st = check_desc(desc);
    if (st != OWL_OK) return st;
    if (!cache || !dst || seq < 0 || seq >= desc->batch || first_pos < 0 || n_tokens < 0)
        return OWL_ERR_INVALID_ARG;
    if (misaligned(cache, 16) || misaligned(dst, 16)) return OWL_ERR_INVALID_ARG;
    if (launch_gather(*desc, cache, page_table, seq, first_pos, n_tokens, dst, dev_status,
                      static_cast<hipStream_t>(stream)) != hipSuccess)
        return OWL_ERR_HIP;
    return OWL_OK;
}

const char *owl_status_str(owl_status s)
{
    switch (s) {
    case OWL_OK: return "ok";
    case OWL_ERR_INVALID_ARG: return "invalid argument";
    case OWL_ERR_BAD_TREE: return "tree_parent is not a forest in parent-first order";
    case OWL_ERR_TOO_MANY_DRAFT: return "n_draft exceeds 64";
    case OWL_ERR_UNSUPPORTED: return "unsupported head_dim, page_size, dtype or shape";
    case OWL_ERR_WORKSPACE: return "workspace missing or too small";
    case OWL_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

const char *owl_version(void) { return "0.2"; }

}  // extern "C"
