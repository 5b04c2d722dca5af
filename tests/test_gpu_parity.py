"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle
on the same seeded inputs.  Everything here needs an MI355X (-m gpu)."""
import numpy as np
import pytest
import torch

from paper_2510_07535_amd import binding as B
from paper_2510_07535_amd import workloads as W
from paper_2510_07535_amd.runner import VerifyStep, _to_dev
from util import assert_close, sample_rows
from tree_helpers import spec_tree

pytestmark = pytest.mark.gpu


def _rng(k):
    return np.random.Generator(np.random.Philox(key=k))


def _run(case, **kw):
    step = VerifyStep(case, **kw)
    step.run()
    out = step.result()
    assert step.dev_status() == 0
    return out, step


def _copies(case, n, planned):
    """One sequence n times over (same pages, queries and tree), announced with ``planned`` tokens."""
    import dataclasses
    table = np.full((1, (planned + case.N + 15) // 16), -1, dtype=np.int32)
    table[:, :case.page_table.shape[1]] = case.page_table
    rep = lambda a: np.ascontiguousarray(np.repeat(a, n, axis=0))
    return dataclasses.replace(case, B=n, q=rep(case.q), page_table=rep(table), ctx_lens=rep(case.ctx_lens),
                               tree_parent=rep(case.tree_parent), max_pages_per_seq=table.shape[1])


_LAYOUTS = ("1x4x2", "1x8x1", "2x4x2", "2x8x1", "3x8x1")        # tiles a wavefront x row wavefronts x key groups


def _layout(plan):
    return _LAYOUTS[plan.kernel_variant % 5]


# Shapes that plan each loop with splits of C tokens out of `planned`: N, G, KV heads, sequences, planned, C, layout.
# (Two KV heads and one sequence plan row groups of at most four tiles, whatever N is: the plain loop with two key groups.)
_EVERY_LOOP = [
    (6, 4, 8, 4, 10340, 1280, "1x4x2"),
    (26, 4, 8, 4, 10340, 1280, "1x8x1"),
    (16, 8, 8, 8, 20580, 2560, "2x4x2"),
    (60, 4, 8, 4, 10340, 1280, "2x8x1"),
    (40, 8, 8, 4, 10340, 1280, "3x8x1"),
]


def _run_in_layout(case, copies, planned, split, layout, **kw):
    """``copies`` equal sequences in splits of ``split`` tokens, which the plan has to give to ``layout``; all come out the same."""
    got, step = _run(_copies(case, copies, planned), split_tokens=split, max_ctx_len=planned, **kw)
    assert step.plan.row_groups == 1 and _layout(step.plan) == layout, step.plan.as_dict()
    assert all(np.array_equal(got[0], got[b]) for b in range(1, copies)), layout
    return got[:1]


# ---------------------------------------------------------------------------
# small and ragged shapes, full element-by-element comparison
# ---------------------------------------------------------------------------
def _small_cases():
    r = _rng(1234)
    mk = W.make_case
    cs = [
        # several 64-key stages, ragged tail, chain (row tiles: 2)
        mk("bf16_chain6_L1000", 101, dtype=W.DT_BF16, Hq=32, Hkv=8, D=128, ctx_lens=[1000], trees=[W.chain_tree(6)]),
        # one row tile, n_draft = 1 (plain decode)
        mk("bf16_decode_L777", 102, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[777], trees=[W.chain_tree(1)]),
        # empty prefix: only the drafts are visible
        mk("bf16_L0_tree20", 103, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[0], trees=[W.random_tree(20, 5, r)]),
        # prefix shorter than a page / exactly a page; drafts straddle pages
        mk("bf16_L15_L16_L17", 104, dtype=W.DT_BF16, Hq=4, Hkv=2, D=128, ctx_lens=[15, 16, 17],
           trees=[W.random_tree(9, 4, r) for _ in range(3)]),
        # 3..4 row tiles -> 2x2 wave layout
        mk("bf16_tree14_G4", 105, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[2500], trees=[W.random_tree(14, 4, r)]),
        # 7 row tiles (the batched configuration's tile count), ragged batch
        mk("bf16_tree26_batch3", 106, dtype=W.DT_BF16, Hq=32, Hkv=8, D=128, ctx_lens=[3000, 129, 1999],
           trees=[W.random_tree(26, 5, r) for _ in range(3)]),
        # 15 row tiles (60-node tree, G=4)
        mk("bf16_tree60", 107, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[1500], trees=[W.random_tree(60, 6, r)]),
        # 20 row tiles (40 nodes, G=8) with outlier keys
        mk("bf16_hybrid40_G8", 108, dtype=W.DT_BF16, Hq=16, Hkv=2, D=128, ctx_lens=[2100],
           trees=[W.hybrid_tree(32, 8, r)], outlier_frac=0.05),
        # maximum draft count, G=8 -> 32 row tiles -> two row groups
        mk("bf16_chain64_G8", 109, dtype=W.DT_BF16, Hq=8, Hkv=1, D=128, ctx_lens=[700], trees=[W.chain_tree(64)]),
        # head_dim 64, token-major cache layout, G=1
        mk("bf16_D64_tokmajor", 110, dtype=W.DT_BF16, Hq=4, Hkv=4, D=64, ctx_lens=[900, 64],
           trees=[W.random_tree(12, 4, r) for _ in range(2)], head_major=False),
        mk("bf16_D64_tree40", 111, dtype=W.DT_BF16, Hq=16, Hkv=4, D=64, ctx_lens=[1300], trees=[W.random_tree(40, 8, r)]),
        # identity paging (page_table NULL)
        mk("bf16_identity_pages", 112, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[555], trees=[W.random_tree(7, 3, r)],
           paged=False),
        # forest: several roots
        mk("bf16_forest", 113, dtype=W.DT_BF16, Hq=4, Hkv=1, D=128, ctx_lens=[300],
           trees=[np.array([-1, -1, 0, 1, 1, -1, 5, 2], np.int32)]),
        # fp16 storage (the paper's inference type)
        mk("f16_tree30", 114, dtype=W.DT_F16, Hq=16, Hkv=4, D=128, ctx_lens=[1100], trees=[spec_tree(W.random_tree(15, 4, r))]),
        # fp16 (the paper's dtype) through the fast loop: long enough for many fast stages; with
        # outlier keys the fp16 P overflows its stale reference and the split is redone
        mk("f16_tree60_L5000", 117, dtype=W.DT_F16, Hq=8, Hkv=2, D=128, ctx_lens=[5000], trees=[W.random_tree(60, 6, r)]),
        mk("f16_outliers_L3000", 118, dtype=W.DT_F16, Hq=16, Hkv=2, D=128, ctx_lens=[3000, 900],
           trees=[W.hybrid_tree(32, 8, r) for _ in range(2)], outlier_frac=0.05),
        # fp32 storage, both head dims
        mk("f32_D64_tree10", 115, dtype=W.DT_F32, Hq=8, Hkv=2, D=64, ctx_lens=[700, 33], trees=[W.random_tree(10, 4, r) for _ in range(2)]),
        mk("f32_D128_chain5", 116, dtype=W.DT_F32, Hq=4, Hkv=2, D=128, ctx_lens=[390], trees=[W.chain_tree(5)]),
    ]
    return cs


@pytest.mark.parametrize("case", _small_cases(), ids=lambda c: c.name)
def test_small_shapes_match_oracle(oracle_mod, case):
    want = oracle_mod.verify_attn_case(case)
    for split in (0, 64, 192, 512):
        got, step = _run(case, split_tokens=split)
        assert_close(got, want, case.dtype, f"{case.name} split={split} plan={step.plan.as_dict()}")


# ---------------------------------------------------------------------------
# 16-bit output types
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("N,G", [(6, 4), (26, 4)])
def test_sixteen_bit_outputs_are_the_rounded_fp32_result(oracle_mod, N, G):
    """out_dtype = bf16 / f16: bit for bit the fp32 output rounded to nearest even, and within the
    fp32 bar widened by one unit in the last place of the output type against the rounded oracle."""
    r = _rng(640 + N)
    case = W.make_case("out16", 640 + N, dtype=W.DT_BF16, Hq=2 * G, Hkv=2, D=128, ctx_lens=[3000, 500],
                       trees=[W.random_tree(N, 5, r) for _ in range(2)])
    ref, _ = _run(case)
    want64 = oracle_mod.verify_attn_case(case)
    for od, dt in ((B.OWL_BF16, W.DT_BF16), (B.OWL_F16, W.DT_F16)):
        got, step = _run(case, out_dtype=od)
        assert got.dtype == np.uint16
        assert np.array_equal(got, W.store(ref, dt)), od
        want = W.widen(W.store(want64.astype(np.float32), dt), dt)           # the oracle rounded to the output type
        ulp = np.abs(want) * (2.0 ** -8 if dt == W.DT_BF16 else 2.0 ** -11) + 1e-7
        err = np.abs(W.widen(got, dt) - want)
        assert (err <= 1e-2 + ulp).all() and err.mean() <= 1e-3 + ulp.mean(), (od, err.max())


# ---------------------------------------------------------------------------
# the five named configurations
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("idx", range(5), ids=W.CONFIG_NAMES)
def test_configs_reduced_context_full_compare(oracle_mod, idx):
    """Same head shapes, trees and paging as the named configuration with the
    context cut to 1/16 (config 0 runs at its full 512 tokens), every output
    element compared."""
    case = W.make_config(idx, ctx_scale=1.0 if idx == 0 else 1.0 / 16)
    want = oracle_mod.verify_attn_case(case)
    got, step = _run(case)
    assert_close(got, want, case.dtype, f"{case.name} plan={step.plan.as_dict()}")


@pytest.mark.parametrize("idx", range(5), ids=W.CONFIG_NAMES)
def test_configs_full_size_all_rows(oracle_mod, idx):
    """Full context lengths, in the launch configuration the benchmark times
    (library-chosen splits); every output element against the oracle."""
    case = W.make_config(idx)
    got, step = _run(case)
    want = oracle_mod.verify_attn_case(case)
    assert_close(got, want, case.dtype, f"{case.name} plan={step.plan.as_dict()}")


@pytest.mark.parametrize("idx", [2, 3])
def test_configs_full_size_fp16(oracle_mod, idx):
    """The long-context configurations stored as fp16 (the paper's inference type), full size, every element."""
    case = W.make_config(idx, dtype=W.DT_F16)
    got, step = _run(case)
    want = oracle_mod.verify_attn_case(case)
    assert_close(got, want, case.dtype, f"{case.name} plan={step.plan.as_dict()}")


# ---------------------------------------------------------------------------
# evaluation-order invariance and exact properties on the GPU
# ---------------------------------------------------------------------------
def test_split_count_invariance(oracle_mod):
    """1 split vs many splits vs the planner's choice: all within tolerance of
    the oracle and of each other (catches combine races and stale partials)."""
    case = W.make_case("splitinv", 201, dtype=W.DT_BF16, Hq=32, Hkv=8, D=128, ctx_lens=[6000, 4097],
                       trees=[W.random_tree(26, 5, _rng(5)) for _ in range(2)])
    want = oracle_mod.verify_attn_case(case)
    outs = []
    for split in (16384, 4096, 1024, 128, 0):
        got, _ = _run(case, split_tokens=split)
        assert_close(got, want, case.dtype, f"split={split}")
        outs.append(got)
        raw, _ = _run(case, split_tokens=split, flags=B.OWL_FLAG_FP32_PARTIALS)      # partials as fp32 accumulators
        assert_close(raw, want, case.dtype, f"split={split}, fp32 partials")
        assert np.abs(raw - got).max() < 2e-3
    for o in outs[1:]:
        assert np.abs(o - outs[0]).max() < 5e-3


def test_non_ancestor_perturbation_is_invisible():
    """Overwriting K/V of draft j must leave every row whose path does not
    contain j bit-identical."""
    tree = W.random_tree(20, 5, _rng(7))
    base_case = W.make_case("perturb", 202, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[1000], trees=[tree])
    base, _ = _run(base_case)
    on_path = np.zeros((20, 20), bool)
    for i in range(20):
        j = i
        while j != -1:
            on_path[i, j] = True
            j = int(tree[j])
    for j in (0, 3, 11, 19):
        c2 = W.make_case("perturb", 202, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[1000], trees=[tree])
        pos = 1000 + j
        page = int(c2.page_table[0, pos // 16])
        c2.k_pool[page, :, pos % 16, :] = W.store(np.full((2, 128), 2.0, np.float32), W.DT_BF16)
        c2.v_pool[page, :, pos % 16, :] = W.store(np.full((2, 128), -9.0, np.float32), W.DT_BF16)
        got, _ = _run(c2)
        for i in range(20):
            if on_path[i, j]:
                assert np.abs(got[0, i] - base[0, i]).max() > 1e-4, (i, j)
            else:
                assert np.array_equal(got[0, i], base[0, i]), (i, j)


def test_page_permutation_is_invisible():
    kw = dict(dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[3000, 700],
              trees=[W.random_tree(12, 4, _rng(8)) for _ in range(2)])
    a, _ = _run(W.make_case("perm", 203, paged=True, **kw))
    b, _ = _run(W.make_case("perm", 203, paged=False, **kw))
    c, _ = _run(W.make_case("perm", 203, paged=True, head_major=False, **kw))
    assert np.array_equal(a, b)
    assert np.array_equal(a, c)


def test_zero_query_integer_values_exact_mean():
    """q = 0, small-integer V, L + depth a power of two for the chain's last
    node: every weight is exactly 1, so the mean must be exact in fp32 -- any
    wrong, missing or doubled cache row shows up as a bit difference.  Exactness
    needs the partials in fp32 (OWL_FLAG_FP32_PARTIALS); the default partials,
    normalised and in fp16, must still be within 2^-11 of a row's largest value."""
    N, L = 4, 4096 - 4
    case = W.make_case("exact", 204, dtype=W.DT_BF16, Hq=4, Hkv=2, D=128, ctx_lens=[L], trees=[W.chain_tree(N)])
    case.q[...] = 0
    r = _rng(9)
    T = L + N
    vals = r.integers(-8, 9, size=(T, 2, 128)).astype(np.float32)
    for pos in range(T):
        page = int(case.page_table[0, pos // 16])
        case.v_pool[page, :, pos % 16, :] = W.store(vals[pos], W.DT_BF16)
    for split in (0, 128, 1024):
        want = vals.sum(axis=0, dtype=np.float64) / T            # last node sees all T rows
        got, _ = _run(case, split_tokens=split, flags=B.OWL_FLAG_FP32_PARTIALS)
        for h in range(4):
            assert np.array_equal(got[0, N - 1, h].astype(np.float64), want[h // 2]), split
        got, _ = _run(case, split_tokens=split)
        for h in range(4):
            assert np.abs(got[0, N - 1, h] - want[h // 2]).max() <= 2.0 ** -11 * np.abs(want[h // 2]).max() + 1e-6, split


def test_quad_max_lane_semantics():
    """The softmax's cross-lane maximum must cover exactly lanes l, l^16, l^32,
    l^48 (a wrong exchange would still give finite, nearly right outputs, so
    it is pinned here on its own)."""
    r = _rng(77)
    for _ in range(4):
        x = r.standard_normal(64).astype(np.float32)
        dx = torch.from_numpy(x).cuda()
        dy = torch.empty(64, dtype=torch.float32, device="cuda")
        B.owl_selftest_quad_max(dx, dy)
        torch.cuda.synchronize()
        want = x.reshape(4, 16).max(axis=0)
        assert np.array_equal(dy.cpu().numpy(), np.tile(want, 4))


# ---------------------------------------------------------------------------
# mask builder and paging: bit-exact
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("n", [1, 2, 32, 33, 63, 64])
def test_deep_and_malformed_trees(oracle_mod, n):
    """The root paths as deep as they come (a chain of n), and parents that are no parents: such a node is a root, as in
    the same tree with -1 in its place, and is flagged."""
    chain, cut = W.chain_tree(n), W.chain_tree(n)
    bad = chain.copy()
    for i, p in ((n // 3, n // 3), (n // 2, -7), (n - 1, 64)):
        bad[i], cut[i] = p, -1
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    for given, meant, flag in ((chain, chain, 0), (bad, cut, B.OWL_DEV_BAD_PARENT)):
        want_anc, want_dep = oracle_mod.tree_mask(meant)
        anc, dep = torch.zeros((1, n), dtype=torch.int64, device="cuda"), torch.zeros((1, n), dtype=torch.int32, device="cuda")
        st.zero_()
        B.owl_build_tree_mask(dev(given[None]), anc, dep, st)
        assert np.array_equal(anc.cpu().numpy().view(np.uint64)[0], want_anc) and np.array_equal(dep.cpu().numpy()[0], want_dep)
        assert int(st.item()) == flag
        case = W.make_case("deep", 40 + n, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[150], trees=[meant])
        step = VerifyStep(case)
        step.tree_parent.copy_(dev(given[None]))
        step.run()
        assert_close(step.result(), oracle_mod.verify_attn_case(case), case.dtype, f"n={n}")
        assert step.dev_status() == flag


def test_tree_mask_bit_exact(oracle_mod):
    r = _rng(10)
    trees64 = [W.random_tree(64, md, r) for md in (None, 2, 8)] + [W.chain_tree(64), np.full(64, -1, np.int32)]
    trees6 = [spec_tree([-1, 0, 0]), W.chain_tree(6)]
    for trees in (trees64, trees6, [W.chain_tree(1)]):
        par = np.stack(trees).astype(np.int32)
        Bn, N = par.shape
        dpar = torch.from_numpy(par).cuda()
        anc = torch.zeros((Bn, N), dtype=torch.int64, device="cuda")
        dep = torch.zeros((Bn, N), dtype=torch.int32, device="cuda")
        st = torch.zeros(1, dtype=torch.int32, device="cuda")
        B.owl_build_tree_mask(dpar, anc, dep, st)
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        for b in range(Bn):
            want_anc, want_dep = oracle_mod.tree_mask(par[b])
            assert np.array_equal(anc[b].cpu().numpy().view(np.uint64), want_anc)
            assert np.array_equal(dep[b].cpu().numpy(), want_dep)
            h_anc, h_dep = B.owl_build_tree_mask_host(par[b])
            assert np.array_equal(h_anc, want_anc) and np.array_equal(h_dep, want_dep)


def test_gather_bit_exact(oracle_mod):
    for head_major, dtype in ((True, W.DT_BF16), (False, W.DT_BF16), (True, W.DT_F32)):
        case = W.make_case("gather", 301, dtype=dtype, Hq=8, Hkv=4, D=128, ctx_lens=[1000, 37, 4000],
                           trees=[W.chain_tree(5)] * 3, head_major=head_major, spare_pages=7)
        step = VerifyStep(case)
        for b in range(case.B):
            T = int(case.ctx_lens[b]) + case.N
            for which, cache in (("k", step.k), ("v", step.v)):
                dst = torch.empty((T, case.Hkv, case.D), dtype=cache.dtype, device="cuda")
                B.owl_gather_kv(step.desc, cache, step.page_table, b, 0, T, dst, step.status)
                torch.cuda.synchronize()
                want = oracle_mod.gather_kv(case, which, b, 0, T)
                got = dst.cpu().numpy()
                assert np.array_equal(got.view(want.dtype), want)
        assert step.dev_status() == 0


def test_measurement_aids():
    """The streaming probes read what they claim to (their XOR folds agree with
    numpy) and the timeline hook records ordered timestamps for every workgroup."""
    r = _rng(78)
    host = r.integers(0, 2**31 - 1, size=(64 * 1024,), dtype=np.int64).astype(np.uint32)   # 256 KiB = 64 blocks
    dev = torch.from_numpy(host.view(np.int32)).cuda()
    want = int(np.bitwise_xor.reduce(host))
    sink = torch.zeros(64, dtype=torch.int32, device="cuda")
    B.owl_stream_read_probe(dev, sink, 8)
    torch.cuda.synchronize()
    assert int(np.bitwise_xor.reduce(sink.cpu().numpy().view(np.uint32)[:8])) == want
    order = torch.from_numpy(r.permutation(64).astype(np.int32)).cuda()
    sink.zero_()
    B.owl_gather_read_probe(dev, order, sink, 5)
    torch.cuda.synchronize()
    assert int(np.bitwise_xor.reduce(sink.cpu().numpy().view(np.uint32)[:5])) == want

    # the matrix-pipe probe: operands all 1.0 -> every accumulator is 32 per MFMA, 16 MFMAs deep per
    # iteration and lane: after 3 iterations sink = acc[i][0] + acc[i][3] summed over 16 accumulators
    ones = torch.ones(4096, dtype=torch.bfloat16, device="cuda")
    fs = torch.zeros(2 * 512, dtype=torch.float32, device="cuda")
    ghz = torch.zeros(2, dtype=torch.float32, device="cuda")
    B.owl_mfma_probe(ones, 3, fs, 2, clock_ghz=ghz)
    torch.cuda.synchronize()
    assert (fs.cpu().numpy() == 16 * 2 * 3 * 32.0).all()
    B.owl_mfma_probe(ones, 20000, fs, 2, clock_ghz=ghz)          # long enough for the 100 MHz counter to resolve
    torch.cuda.synchronize()
    assert ((ghz.cpu().numpy() > 0.3) & (ghz.cpu().numpy() < 3.0)).all()

    case = W.make_case("tl", 79, dtype=W.DT_BF16, Hq=32, Hkv=8, D=128, ctx_lens=[3000], trees=[W.random_tree(20, 4, r)])
    step = VerifyStep(case, split_tokens=512)
    step.run()
    ref = step.result().copy()
    nwg = step.plan.n_workgroups
    tl = torch.zeros(10 * nwg, dtype=torch.int64, device="cuda")
    B.owl_debug_set_timeline(tl)
    try:
        step.run()
        got = step.result()
    finally:
        B.owl_debug_set_timeline(None)
    assert np.array_equal(got, ref)                      # recording does not change the result
    t = tl.cpu().numpy().reshape(nwg, 10)
    ran = t[t[:, 0] > 0]
    # one workgroup per (kv head, split, row group): 48 streams do not fill the chip, so the 5 row tiles go to 2 groups
    assert step.plan.row_groups == 2 and len(ran) == 8 * ((3000 + 20 + 511) // 512) * step.plan.row_groups
    assert (np.diff(ran[:, :6], axis=1) >= 0).all()
    assert sorted(ran[:, 7]) == sorted(set(ran[:, 7]))
    assert (ran[:, 9] >= ran[:, 8]).all() and (ran[:, 8] > 0).all()   # shader cycles at both ends of the fast loop

    # a workgroup whose share has two pieces: its phases are summed over them, set-up does not swallow the first piece's loop
    two = W.make_case("tl2", 80, dtype=W.DT_BF16, Hq=64, Hkv=64, D=128, ctx_lens=[2200, 2500], trees=[W.chain_tree(6)] * 2)
    step2 = VerifyStep(two)
    pieces, _, _, dealt, _ = B.owl_probe_deal(step2.desc, [2206, 2506])
    crossing = [w for w in set(pieces[:, 0].tolist()) if (pieces[:, 0] == w).sum() == 2]
    step2.run()
    tl = torch.zeros(10 * step2.plan.n_workgroups, dtype=torch.int64, device="cuda")
    B.owl_debug_set_timeline(tl)
    try:
        step2.run()
        step2.result()
    finally:
        B.owl_debug_set_timeline(None)
    t = tl.cpu().numpy().reshape(-1, 10)
    t = t[t[:, 5] > 0]
    of_two = np.isin(t[:, 7] // 64, crossing)                         # KV heads vary fastest, one row group
    assert dealt and step2.plan.row_groups == 1 and len(crossing) == 1 and of_two.sum() == 64
    assert (np.diff(t[:, :6], axis=1) >= 0).all() and (t[:, 9] > t[:, 8]).all()
    setup = np.diff(t[:, :2], axis=1)[:, 0] / (t[:, 5] - t[:, 0])
    assert np.median(setup[of_two]) < 0.45, (np.median(setup[of_two]), np.median(setup[~of_two]))

    # the split-KV launch with events attached to its dispatch: same result, a plausible duration
    timer = B.KernelTimer()
    step.out.fill_(float("nan"))
    step.run_split_timed(timer)
    step.run(phases=B.PHASE_COMBINE)
    assert np.array_equal(step.result(), ref)
    assert 1e-3 < timer.elapsed_ms() < 50.0

    # the step probe: every wavefront reports its loop cycles, and the matrix pipe cannot be more than busy
    src = torch.randn(8192, device="cuda").to(torch.bfloat16)
    fs = torch.zeros(4 * 512, dtype=torch.float32, device="cuda")
    cyc = torch.zeros(4 * 8, dtype=torch.int64, device="cuda")
    for variant, _, tiles in B.STEP_PROBE_VARIANTS:
        cyc.zero_()
        B.owl_step_probe(variant, src, 200, fs, cyc, 4)
        torch.cuda.synchronize()
        per_step = cyc.cpu().numpy() / 200.0
        assert (per_step > tiles * 17 * 16 * 0.5).all() and (per_step < 50000).all(), (variant, per_step)
        assert np.isfinite(fs.cpu().numpy()).all()


# ---------------------------------------------------------------------------
# data errors on the device are flagged, never followed out of bounds
# ---------------------------------------------------------------------------
def test_device_side_errors_are_flagged():
    tree = W.random_tree(10, 4, _rng(11))
    def fresh():
        return W.make_case("bad", 401, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[500, 300], trees=[tree, tree])
    c = fresh()
    c.tree_parent[1, 4] = 7                      # child before parent
    s = VerifyStep(c); s.run()
    assert s.dev_status() & B.OWL_DEV_BAD_PARENT
    c = fresh()
    c.page_table[0, 3] = c.n_pool_pages + 5      # page outside the pool
    s = VerifyStep(c); s.run()
    assert s.dev_status() & B.OWL_DEV_BAD_PAGE
    c = fresh()
    s = VerifyStep(c, max_ctx_len=400)           # ctx_lens[0] = 500 > announced bound
    s.run()
    assert s.dev_status() & B.OWL_DEV_BAD_CTX_LEN
    # the sequence that was fine is still right next to a flagged one
    par = torch.from_numpy(np.array([[-1, 0, 5, 1]], np.int32)).cuda()
    anc = torch.zeros((1, 4), dtype=torch.int64, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.owl_build_tree_mask(par, anc, None, st)
    torch.cuda.synchronize()
    assert int(st.item()) & B.OWL_DEV_BAD_PARENT


# ---------------------------------------------------------------------------
# per-sequence draft counts
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("dtype,N,G,counts", [
    (W.DT_BF16, 26, 4, [26, 0, 9, 1, 17]),          # 7 row tiles, one sequence without drafts
    (W.DT_BF16, 60, 4, [60, 31, 2]),                # 15 row tiles (pipelined loop)
    (W.DT_BF16, 40, 8, [40, 13]),                   # 20 row tiles (three tiles per wave)
    (W.DT_BF16, 6, 4, [3, 6, 1, 5]),                # 2 row tiles (two key groups)
    (W.DT_F32, 10, 4, [4, 10]),
])
def test_ragged_draft_counts(oracle_mod, dtype, N, G, counts):
    r = _rng(900 + N)
    B_ = len(counts)
    ctx = [int(x) for x in r.integers(0, 3000, size=B_)]
    ctx[0] = 2500
    D = 64 if dtype == W.DT_F32 else 128
    case = W.make_case("ragged", 300 + N, dtype=dtype, Hq=2 * G, Hkv=2, D=D, ctx_lens=ctx,
                       trees=[W.random_tree(N, 6, r) for _ in range(B_)])
    want = oracle_mod.verify_attn_ragged_case(case, counts)
    for split in (0, 192):
        step = VerifyStep(case, split_tokens=split)
        nd = torch.tensor(counts, dtype=torch.int32, device=step.device)
        step.out.fill_(float("nan"))
        B.owl_verify_attn_ragged(step.desc, step.q, step.k, step.v, step.page_table, step.ctx_lens,
                                 step.tree_parent, nd, step.out, step.workspace, step.status)
        got = step.result()
        assert step.dev_status() == 0
        assert_close(got, want, case.dtype, f"ragged N={N} split={split}")
        for b, n in enumerate(counts):
            assert (got[b, n:] == 0).all()


@pytest.mark.parametrize("name,ctx,Hkv", [
    ("one long, many short", [9000] + [300] * 15, 8),            # under-filled launch: the long one is cut finer
    ("more sequences than lanes", None, 2),                      # 70 sequences: the second 64-chunk of the search
    ("equal lengths", [2000] * 12, 4),
    ("all empty prefixes", [0] * 5, 2),
])
def test_batch_split_follows_the_lengths(oracle_mod, name, ctx, Hkv):
    """A batch with a library-chosen split size: the kernels share out the actual lengths, whatever
    they are; the result must not care, and the planned grid must hold every worker (a piece that
    nobody serves would leave a row's partials unwritten and show as a mismatch)."""
    r = _rng(4242)
    if ctx is None:
        ctx = [int(x) for x in r.integers(0, 400, size=70)]
        ctx[3] = ctx[66] = 0
        ctx[69] = 1500
    n = 5
    case = W.make_case("batchsplit", 77, dtype=W.DT_BF16, Hq=4 * Hkv, Hkv=Hkv, D=128, ctx_lens=ctx,
                       trees=[W.random_tree(n, 3, r) for _ in ctx])
    want = oracle_mod.verify_attn_case(case)
    got, step = _run(case)
    assert_close(got, want, case.dtype, name)
    # the pieces that the host arithmetic gives for these lengths fit the launched grid and the partials' slots
    plan = step.plan
    pieces, _, n_slots, dealt, workers = B.owl_probe_deal(step.desc, [L + n for L in ctx])
    assert dealt and workers * Hkv * plan.row_groups <= plan.n_workgroups
    assert pieces[:, 0].max() < workers and pieces[:, 4].max() < n_slots
    assert sum(end - first for _, _, first, end, _ in pieces.tolist()) == sum(L + n for L in ctx)
    # announced longer than anything present: the plan (grid, partials) is for 65536, the lengths are not
    import dataclasses
    cols = (65536 + n + 15) // 16                        # the page table has to cover the planned length
    table = np.zeros((case.B, cols), dtype=np.int32)
    table[:, :case.page_table.shape[1]] = case.page_table
    wide = dataclasses.replace(case, page_table=table, max_pages_per_seq=cols)
    got2, step2 = _run(wide, max_ctx_len=65536)
    assert_close(got2, want, case.dtype, name + " (planned for 65536)")
    if len(ctx) <= 16:                                   # with per-sequence draft counts on top
        counts = [n if b % 3 else max(0, n - 2 - b % 2) for b in range(len(ctx))]
        counts[0] = 0 if len(ctx) > 1 else n
        want3 = oracle_mod.verify_attn_ragged_case(case, counts)
        nd = torch.tensor(counts, dtype=torch.int32, device=step.device)
        B.owl_verify_attn_ragged(step.desc, step.q, step.k, step.v, step.page_table, step.ctx_lens,
                                 step.tree_parent, nd, step.out, step.workspace, step.status)
        got3 = step.result()
        assert step.dev_status() == 0
        assert_close(got3, want3, case.dtype, name + " (ragged counts)")


@pytest.mark.parametrize("name,Hq,Hkv,D,ctx,n,dealt", [
    ("more than one round of workers", 64, 64, 64, [200_000], 3, True),    # a share would outgrow the page list: 8 workers, not 4
    ("fewer workers than compute units", 4, 1, 128, [19950], 4, True),
    ("shares of one stage", 8, 2, 128, [0, 1, 63, 64, 65, 127], 4, True),
    ("few partials per sequence", 8, 2, 64, [1500 + 37 * k for k in range(40)], 6, True),
    ("many partials per sequence", 8, 2, 128, [9000, 1, 14000], 6, True),
    ("fewer workers, to fit the fixed scratch", 64, 8, 128, [2900, 40, 8000, 700], 48, True),
    ("equal splits, to fit the fixed scratch", 28, 4, 128, [3 + k % 40 for k in range(100)], 31, False),
])
def test_work_dealt_by_length(oracle_mod, name, Hq, Hkv, D, ctx, n, dealt):
    """A library-chosen split size: equal shares of the sequences laid end to end, cut at their ends (or
    equal splits, where the partials would not fit).  The longest case reads a small pool through a table that repeats its pages."""
    import dataclasses
    r = _rng(sum(ctx) + n)
    trees = [W.random_tree(n, 3, r) for _ in ctx]
    case = W.make_case("dealt", 91, dtype=W.DT_BF16, Hq=Hq, Hkv=Hkv, D=D, ctx_lens=[min(L, 20000) for L in ctx], trees=trees)
    if max(ctx) > 20000:
        cols = (max(ctx) + n + 15) // 16
        table = case.page_table[:, np.arange(cols) % (20000 // 16)]            # full pages only
        case = dataclasses.replace(case, ctx_lens=np.array(ctx, np.int32), page_table=table, max_pages_per_seq=cols)
    # (fp32 partials where the fixed scratch of the entry point without a workspace is to be what limits the launch)
    got, step = _run(case, flags=B.OWL_FLAG_FP32_PARTIALS if "scratch" in name else 0)
    assert B.owl_probe_deal(step.desc, [L + n for L in ctx])[3] == dealt
    if sum(ctx) * n * Hq > 2e7:
        rows = sample_rows(case, 40, seed=5, always=[(0, 0, 0), (0, n - 1, Hq - 1)])
        want = oracle_mod.verify_attn_case(case, rows=rows)
        got = np.stack([got[b, i, h] for b, i, h in rows])
    else:
        want = oracle_mod.verify_attn_case(case)
    assert_close(got, want, case.dtype, f"{name} plan={step.plan.as_dict()}")


@pytest.mark.parametrize("frac,gain,tag", [(0.05, 8.0, "frequent outliers: guarded reference"),
                                           (0.0007, 40.0, "rare late outliers: frozen reference, overflow, redo"),
                                           (0.02, 3.0, "mild tail: frozen reference holds")])
@pytest.mark.parametrize("N,G", [(6, 4), (60, 4), (40, 8)])     # row groups of at most four tiles: two key groups
def test_fp16_score_range_paths(oracle_mod, frac, gain, tag, N, G):
    """fp16 probabilities overflow 2^16 above their reference.  The kernel takes a loop with a guarded (moving) reference if the
    scores of a split's first keys already show a long tail; otherwise it freezes the reference and, should a later score
    overflow it after all, redoes the split.  All routes must give the oracle's result."""
    r = _rng(77 + N)
    case = W.make_case("f16range", 910 + N, dtype=W.DT_F16, Hq=2 * G, Hkv=2, D=128, ctx_lens=[9000, 700],
                       trees=[W.random_tree(N, 6, r) for _ in range(2)], outlier_frac=frac, outlier_gain=gain)
    got, step = _run(case)
    assert_close(got, oracle_mod.verify_attn_case(case), case.dtype, f"{tag}, N={N} G={G}")


@pytest.mark.parametrize("N,G,D", [(6, 4, 128), (60, 4, 64), (26, 4, 128), (60, 4, 128), (40, 8, 128)])     # likewise
def test_fp16_overflow_found_at_every_look(oracle_mod, N, G, D):
    """A frozen fp16 loop looks for overflowed row sums at stages 4, 16, 64, ... and once more behind its last stage.  Each split
    here has one key that overflows the reference, in another place: the second step, the stages around a look, the last fast
    stage.  The first split has none."""
    C, L = 1280, 8 * 1280 + 100
    hot = [s * C + 64 * stage + slot for s, (stage, slot) in enumerate([(0, 40), (1, 9), (3, 63), (4, 0), (15, 40), (16, 3), (19, 63)], 1)]
    case = W.make_case("f16_looks", 950 + N + D, dtype=W.DT_F16, Hq=2 * G, Hkv=2, D=D, ctx_lens=[L], trees=[W.random_tree(N, 6, _rng(N))])
    for pos in hot:
        page = int(case.page_table[0, pos // 16])
        row = W.widen(case.k_pool[page, :, pos % 16, :], W.DT_F16) * 32.0
        case.k_pool[page, :, pos % 16, :] = W.store(row.astype(np.float32), W.DT_F16)
    # the premise, from the stored values: some row's score lies 2^20 or more above its reference (4 above the first keys)
    q, c = W.widen(case.q[0], W.DT_F16), case.scale * 1.4426950408889634
    for pos in hot[1:]:
        at = np.append(np.arange(pos // C * C, pos // C * C + 64), pos)
        keys = W.widen(case.k_pool[case.page_table[0, at // 16], :, at % 16, :], W.DT_F16)          # [65, Hkv, D]
        x = np.stack([c * q[:, h] @ keys[:, h // G].T for h in range(case.Hq)])                       # [Hq, N, 65]
        assert (x[..., -1] - x[..., :-1].max(axis=-1)).max() > 21.0
    want = oracle_mod.verify_attn_case(case)
    for split in (C, 0):
        got, step = _run(case, split_tokens=split)
        assert_close(got, want, case.dtype, f"N={N} G={G} D={D} split={split} plan={step.plan.as_dict()}")


@pytest.mark.parametrize("N,G,layout", [(6, 4, "1x4x2"), (26, 4, "1x8x1"), (16, 8, "2x4x2"), (60, 4, "2x8x1"), (40, 8, "3x8x1")])
def test_fp16_redone_piece_keeps_its_small_weights(oracle_mod, N, G, layout):
    """One key of 16384 lies about 17.5 (log2 units) above the frozen reference of every row: fp16's P overflows and the piece is
    redone.  All other keys then weigh 2^-20 and less, near the end of what fp16 holds, so a reference above the offender
    loses them: four above it, the output is off by a thousandth of the offender's V row."""
    C, hot, target = 16384, 20 * 64 + 9, 24.5
    case = W.make_case("f16_small", 1950 + N, dtype=W.DT_F16, Hq=8 * G, Hkv=8, D=128, ctx_lens=[C], trees=[W.random_tree(N, 6, _rng(N))])
    # channel 0 belongs to the offender: 8 in every query, nothing in the other keys
    c = case.scale * 1.4426950408889634
    case.q[..., 0] = W.store(np.full((1,), 8.0, np.float32), W.DT_F16)[0]
    case.k_pool[:, :, :, 0] = 0
    row = np.zeros((8, 128), np.float32)
    row[:, 0] = target / (8.0 * c)
    case.k_pool[int(case.page_table[0, hot // 16]), :, hot % 16, :] = W.store(row, W.DT_F16)
    got = _run_in_layout(case, 8, 33000, C, layout, flags=B.OWL_FLAG_FP32_PARTIALS)
    rows = sample_rows(case, 64, seed=N, always=[(0, 0, 0), (0, N - 1, case.Hq - 1)])
    want = oracle_mod.verify_attn_case(case, rows=rows)
    pos = np.arange(C)
    pages, q = case.page_table[0, pos // 16], W.widen(case.q[0], W.DT_F16).astype(np.float64)
    keys, vals = (W.widen(p[pages, :, pos % 16, :], W.DT_F16).astype(np.float64) for p in (case.k_pool, case.v_pool))       # [C, Hkv, D]
    over = -np.inf
    for (_, i, h), w64 in zip(rows, want):
        x = c * keys[:, h // G] @ q[i, h]
        over = max(over, x[hot] - x[:64].max() - 4.0)
        # What fp16 makes of weights 2^(x - highest): a redone piece has no worse ones.  (A lower reference keeps more of
        # them; 1e-4 covers a weight's own error, of its score in fp32 sums, and a rounding at another place.)
        w = np.exp2(x - x[hot])
        off = np.abs(w - w.astype(np.float16)) + 1e-4 * w
        bound = (off[:, None] * np.abs(vals[:, h // G] - w64)).sum(axis=0) / w.sum() + 1e-5
        err = np.abs(got[0, i, h] - w64)
        assert (err <= bound).all(), (layout, i, h, float(err.max()), float(bound.max()))
    assert over > 16.0, over


def _heat(case, hot, gain):
    for pos in hot:
        page = int(case.page_table[0, pos // 16])
        row = W.widen(case.k_pool[page, :, pos % 16, :], case.dtype) * gain
        case.k_pool[page, :, pos % 16, :] = W.store(row.astype(np.float32), case.dtype)


def _most_above(case, pos, C):
    """By how much (log2 units) the score of key pos exceeds those of the first 64 keys of its split, in the row where that is most."""
    q, c = W.widen(case.q[0], case.dtype), case.scale * 1.4426950408889634
    at = np.append(np.arange(pos // C * C, pos // C * C + 64), pos)
    keys = W.widen(case.k_pool[case.page_table[0, at // 16], :, at % 16, :], case.dtype)                  # [65, Hkv, D]
    x = np.stack([c * q[:, h] @ keys[:, h // case.G].T for h in range(case.Hq)])                          # [Hq, N, 65]
    return float((x[..., -1] - x[..., :-1].max(axis=-1)).max())


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("N,G,Hkv,n,planned,C,layout", _EVERY_LOOP)
def test_fp16_overflow_found_in_every_loop(oracle_mod, N, G, Hkv, n, planned, C, layout, D):
    """One overflowing key a split, as above, in every loop: the pipelined ones give way at stage 0 with the ring kept (second
    step), at stages 4 and 16, and behind the loop; with three tiles a wavefront there is a look at stage 1.  The stages around
    each look, and the last."""
    last = C // 64 - 1
    places = [(0, 40), (0, 63), (1, 9), (3, 63), (4, 0), (15, 40), (16, 3), (last, 63)]
    hot = [s * C + 64 * stage + slot for s, (stage, slot) in enumerate(places)]
    case = W.make_case("f16_looks", 1150 + N + D, dtype=W.DT_F16, Hq=Hkv * G, Hkv=Hkv, D=D, ctx_lens=[8 * C + 100],
                       trees=[W.random_tree(N, 6, _rng(N))])
    _heat(case, hot, 32.0)
    for pos in hot[2:]:
        assert _most_above(case, pos, C) > 21.0, pos
    got = _run_in_layout(case, n, planned, C, layout)
    _close_to_oracle(oracle_mod, case, got, f"{layout} D={D}")
    dealt, step = _run(_copies(case, n, planned), max_ctx_len=planned)
    _close_to_oracle(oracle_mod, case, dealt[-1:], f"dealt, plan={step.plan.as_dict()}")


@pytest.mark.parametrize("frac,gain", [(0.05, 8.0), (0.0007, 40.0), (0.02, 3.0)])
@pytest.mark.parametrize("N,G,Hkv,n,planned,C,layout", _EVERY_LOOP)
def test_fp16_score_range_in_every_loop(oracle_mod, N, G, Hkv, n, planned, C, layout, frac, gain):
    """Frequent, rare and mild outliers, as in test_fp16_score_range_paths, in every loop."""
    case = W.make_case("f16range", 1250 + N, dtype=W.DT_F16, Hq=Hkv * G, Hkv=Hkv, D=128, ctx_lens=[9000],
                       trees=[W.random_tree(N, 6, _rng(N))], outlier_frac=frac, outlier_gain=gain)
    got = _run_in_layout(case, n, planned, C, layout)
    _close_to_oracle(oracle_mod, case, got, f"{layout} {frac} {gain}")


@pytest.mark.parametrize("N,G,Hkv,n,planned,C,layout", _EVERY_LOOP)
def test_bf16_reference_overflow_redo_in_every_loop(oracle_mod, N, G, Hkv, n, planned, C, layout):
    """As test_bf16_reference_overflow_redo, in every loop."""
    case = W.make_case("bf16_redo", 1350 + N, dtype=W.DT_BF16, Hq=Hkv * G, Hkv=Hkv, D=128, ctx_lens=[6 * C + 77],
                       trees=[W.random_tree(N, 6, _rng(N))])
    hot = [C + 700, 2 * C + 1270, 3 * C + 100, 4 * C + 300]
    _heat(case, hot, 64.0)
    for pos in hot:
        assert _most_above(case, pos, C) > 104.0, pos
    got = _run_in_layout(case, n, planned, C, layout)
    _close_to_oracle(oracle_mod, case, got, layout)


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("N,G,L", [(6, 4, 40), (60, 4, 63), (40, 8, 20), (26, 4, 700)])
def test_fp16_non_finite_draft_stays_in_its_subtree(oracle_mod, N, G, L, bad):
    """A draft whose K row holds a value that is no number (or infinite) spoils the rows that see it and no other, in pieces
    without a whole prefix stage, which have nothing to redo, and in longer ones."""
    tree = W.random_tree(N, 6, _rng(N))
    case = W.make_case("f16_nan", 990 + N, dtype=W.DT_F16, Hq=2 * G, Hkv=2, D=128, ctx_lens=[L], trees=[tree])
    want = oracle_mod.verify_attn_case(case)
    node = N // 2
    page, slot = int(case.page_table[0, (L + node) // 16]), (L + node) % 16
    case.k_pool[page, :, slot, 7] = np.array([bad], np.float16).view(np.uint16)[0]
    got, step = _run(case)
    sees = np.zeros(N, bool)
    for i in range(N):
        j = i
        while j >= 0 and j != node:
            j = int(tree[j])
        sees[i] = j == node
    assert sees.any() and not sees.all()
    assert_close(got[:, ~sees], want[:, ~sees], case.dtype, f"{bad} plan={step.plan.as_dict()}")
    if np.isnan(bad):
        assert np.isnan(got[:, sees]).all()


@pytest.mark.parametrize("N,G", [(6, 4), (60, 4), (40, 8)])     # row groups of at most four tiles: two key groups
def test_bf16_reference_overflow_redo(oracle_mod, N, G):
    """bf16 storage keeps the softmax reference of a split frozen at the maxima of its first keys.
    A later score more than ~100 (log2 units) above it overflows 2^(x - m); the row sum shows it
    and the split is redone with the exact loop.  Here a few late prefix keys of every split are
    64 times longer than the rest (an exact change of exponent in bf16), which puts some row's
    score more than 104 above everything in the first 64 keys of that split -- checked below on
    the host, so that the redo is known to be on the path -- and the result must still be the
    oracle's."""
    r = _rng(5100 + N)
    L, C = 9000, 2048
    case = W.make_case("bf16_redo", 930 + N, dtype=W.DT_BF16, Hq=2 * G, Hkv=2, D=128, ctx_lens=[L],
                       trees=[W.random_tree(N, 6, r)])
    hot = [C + 700, 2 * C + 1500, 3 * C + 100, 4 * C + 300]        # one per split but the first; never in a split's first 64 keys
    for pos in hot:
        page = int(case.page_table[0, pos // 16])
        row = W.widen(case.k_pool[page, :, pos % 16, :], W.DT_BF16) * 64.0
        case.k_pool[page, :, pos % 16, :] = W.store(row.astype(np.float32), W.DT_BF16)
    # host check of the premise, from the stored values: x = scale * log2(e) * q.k in float64
    q = W.widen(case.q[0], W.DT_BF16)                                # [N, Hq, D]
    c = case.scale * 1.4426950408889634
    for pos in hot:
        first = np.arange(pos // C * C, pos // C * C + 64)
        pages = case.page_table[0, first // 16]
        k_first = W.widen(case.k_pool[pages, :, first % 16, :], W.DT_BF16)          # [64, Hkv, D]
        k_hot = W.widen(case.k_pool[int(case.page_table[0, pos // 16]), :, pos % 16, :], W.DT_BF16)
        over = -np.inf
        for h in range(case.Hq):
            x_first = c * np.einsum("nd,kd->nk", q[:, h], k_first[:, h // G])     # [N, 64]
            x_hot = c * q[:, h] @ k_hot[h // G]                                    # [N]
            over = max(over, float((x_hot - x_first.max(axis=1)).max()))
        assert over > 104.0, f"the case does not overflow the frozen reference of the split of key {pos}: {over:.1f}"
    want = oracle_mod.verify_attn_case(case)
    for split in (C, 0):                                  # the split size the premise was checked for, and the library's own
        got, step = _run(case, split_tokens=split)
        assert_close(got, want, case.dtype, f"N={N} G={G} split={split} plan={step.plan.as_dict()}")


def test_graph_capture_replays_match_eager(oracle_mod):
    """No entry point allocates, clears memory or synchronises, so a verify step can be captured
    in a HIP graph.  The graph is replayed several times with new queries and lengths in the
    same buffers, with eager work and synchronisations in between; every replay must equal the
    eager result on the same inputs."""
    r = _rng(606)
    ctx = [1500, 40, 700]
    case = W.make_case("graph", 61, dtype=W.DT_BF16, Hq=16, Hkv=4, D=128, ctx_lens=ctx,
                       trees=[W.random_tree(12, 4, r) for _ in ctx])
    step = VerifyStep(case)
    B.owl_verify_attn_init(step.desc)                     # one-time kernel attributes, outside the capture
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            step.run()
    torch.cuda.synchronize()
    q0 = step.q.clone()
    for rep in range(4):
        if rep:                                           # new inputs in place: scaled queries, shorter contexts
            step.q.copy_((q0.view(torch.bfloat16).float() * (1.0 + 0.25 * rep)).to(torch.bfloat16).view(torch.int16))
            step.ctx_lens.copy_(torch.tensor([1500 - 100 * rep, 40, 700 - 300 * (rep % 2)], dtype=torch.int32))
        torch.cuda.synchronize()
        step.out.fill_(float("nan"))
        graph.replay()
        got = step.result().copy()
        step.out.fill_(float("nan"))
        step.run()                                        # eager, same buffers
        want = step.result().copy()
        assert step.dev_status() == 0
        assert np.array_equal(got, want), f"replay {rep}"
    # and the first replay's inputs were the seeded case: against the oracle too
    step.q.copy_(q0)
    step.ctx_lens.copy_(torch.tensor(ctx, dtype=torch.int32))
    torch.cuda.synchronize()
    graph.replay()
    assert_close(step.result(), oracle_mod.verify_attn_case(case), case.dtype, "graph replay")


def test_ragged_flags_bad_counts():
    case = W.make_case("ragged_bad", 77, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[300, 200],
                       trees=[W.chain_tree(5) for _ in range(2)])
    step = VerifyStep(case)
    nd = torch.tensor([9, -1], dtype=torch.int32, device=step.device)
    B.owl_verify_attn_ragged(step.desc, step.q, step.k, step.v, step.page_table, step.ctx_lens,
                             step.tree_parent, nd, step.out, step.workspace, step.status)
    got = step.result()
    assert step.dev_status() & B.OWL_DEV_BAD_NDRAFT
    assert np.isfinite(got).all() and (got[1] == 0).all()            # 9 -> 5 nodes, -1 -> none


@pytest.mark.parametrize("split", [0, 128])
@pytest.mark.parametrize("counts,lens,flags", [
    ([5, -1], [300, 200], B.OWL_DEV_BAD_NDRAFT), ([-1, 5], [300, 200], B.OWL_DEV_BAD_NDRAFT), ([-1, -1], [300, 200], B.OWL_DEV_BAD_NDRAFT),
    ([5, 6], [300, 200], B.OWL_DEV_BAD_NDRAFT), ([5, 0], [300, -7], B.OWL_DEV_BAD_CTX_LEN), ([0, 5], [301, 200], B.OWL_DEV_BAD_CTX_LEN),
    ([5, 0], [300, 200], 0)])
def test_ragged_flags_every_entry_out_of_range(counts, lens, flags, split):
    """An entry out of range is reported whether or not it leaves its sequence anything to scan, whichever sequence it
    belongs to, with a caller-chosen and a library-chosen split size."""
    case = W.make_case("ragged_bad", 77, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[300, 200],
                       trees=[W.chain_tree(5) for _ in range(2)])
    step = VerifyStep(case, split_tokens=split)
    step.ctx_lens = torch.tensor(lens, dtype=torch.int32, device=step.device)
    nd = torch.tensor(counts, dtype=torch.int32, device=step.device)
    B.owl_verify_attn_ragged(step.desc, step.q, step.k, step.v, step.page_table, step.ctx_lens,
                             step.tree_parent, nd, step.out, step.workspace, step.status)
    got = step.result()
    assert step.dev_status() == flags
    for b, n in enumerate(counts):
        assert np.isfinite(got[b]).all() and (got[b, max(0, n):] == 0).all()


# ---------------------------------------------------------------------------
# a single sequence much shorter than the length the plan was made for
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("L,planned", [(0, 131072), (100, 131072), (3000, 131072), (40000, 65536), (5000, 5000), (4999, 5000)])
def test_context_shorter_than_planned(oracle_mod, L, planned):
    """The plan is sized by max_ctx_len; the kernels re-cut a shorter lone sequence into the
    same number of splits.  Same result either way."""
    case = W.make_case("short_ctx", 500 + L % 97, dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[L],
                       trees=[W.random_tree(14, 4, _rng(L + 1))])
    want = oracle_mod.verify_attn_case(case)
    # the page table has to cover the planned length: pad its row (the extra entries are never read)
    import dataclasses
    cols = (planned + case.N + 15) // 16
    table = np.zeros((1, cols), dtype=np.int32)
    table[:, :case.page_table.shape[1]] = case.page_table
    wide = dataclasses.replace(case, page_table=table, max_pages_per_seq=cols)
    got, step = _run(wide, max_ctx_len=planned)
    assert_close(got, want, case.dtype, f"L={L} planned={planned} plan={step.plan.as_dict()}")
    exact, _ = _run(case)
    assert_close(got, exact.astype(np.float64), case.dtype, "planned-for-longer vs planned-exactly")


@pytest.mark.parametrize("dtype,D,G,N,frac,gain", [
    (W.DT_BF16, 128, 8, 13, 0.0, 1.0),        # 104 rows: seven tiles, the fourth pair has one
    (W.DT_BF16, 128, 8, 15, 0.05, 8.0),       # 120 rows: eight tiles, the last one half empty
    (W.DT_BF16, 64, 4, 32, 0.0, 1.0),         # 128 rows, exactly eight tiles
    (W.DT_F16, 128, 4, 26, 0.0007, 40.0),     # a frozen reference that overflows: the piece is redone
    (W.DT_F16, 64, 8, 16, 0.05, 8.0),         # the guarded reference
])
def test_two_tiles_a_pair_of_wavefronts(oracle_mod, dtype, D, G, N, frac, gain):
    """Seven and eight row tiles, planned for long shares: pairs of wavefronts hold two tiles each, split the steps of a
    stage and hand each other a tile at the end.  The lengths are short (none, one stage, ragged ends, several stages), the
    announced length is what makes the plan choose this layout."""
    import dataclasses
    lens, planned = [0, 3000, 64, 1, 63, 700, 128, 5001], 131072
    trees = [W.random_tree(N, 5, _rng(N + 10 * b)) for b in range(len(lens))]
    case = W.make_case("pairs", 870 + N, dtype=dtype, Hq=4 * G, Hkv=4, D=D, ctx_lens=lens, trees=trees, outlier_frac=frac, outlier_gain=gain)
    table = np.zeros((len(lens), (planned + N + 15) // 16), dtype=np.int32)
    table[:, :case.page_table.shape[1]] = np.maximum(case.page_table, 0)
    wide = dataclasses.replace(case, page_table=table, max_pages_per_seq=table.shape[1])
    got, step = _run(wide, max_ctx_len=planned)
    plan = step.plan.as_dict()
    assert plan["row_tiles"] in (7, 8) and plan["row_groups"] == 1 and plan["tiles_per_wave"] == 2, plan
    assert_close(got, oracle_mod.verify_attn_case(case), case.dtype, f"plan={plan}")


def _announced(case, planned):
    """The case with a page table wide enough for ``planned`` tokens; the entries behind the sequences hold -1."""
    import dataclasses
    table = np.full((case.B, (planned + case.N + 15) // 16), -1, dtype=np.int32)
    table[:, :case.page_table.shape[1]] = case.page_table
    return dataclasses.replace(case, page_table=table, max_pages_per_seq=table.shape[1])


def _close_to_oracle(oracle_mod, case, got, what):
    """All rows, or forty of them where all would keep the oracle busy for long."""
    if int(case.ctx_lens.sum()) * case.N * case.Hq > 2e7:
        rows = sample_rows(case, 40, seed=5, always=[(0, 0, 0), (case.B - 1, case.N - 1, case.Hq - 1)])
        assert np.isfinite(got).all(), what
        assert_close(np.stack([got[b, i, h] for b, i, h in rows]), oracle_mod.verify_attn_case(case, rows=rows), case.dtype, what)
    else:
        assert_close(got, oracle_mod.verify_attn_case(case), case.dtype, what)


@pytest.mark.parametrize("dtype,D,G,N,Hkv,lens,split,flags,groups", [
    (W.DT_BF16, 128, 8, 13, 4, [0, 3000, 64, 1, 63, 700, 128, 5001], 0, B.OWL_FLAG_FP32_PARTIALS, 1),
    (W.DT_F16, 64, 4, 30, 4, [0, 3000, 64, 1, 63, 700, 128, 5001], 0, B.OWL_FLAG_FP32_PARTIALS, 1),
    (W.DT_BF16, 128, 8, 31, 2, [20000, 16353, 16354, 0, 500, 1], 16384, 0, 2),     # a caller's splits, two groups of eight tiles
    (W.DT_BF16, 64, 16, 60, 1, [2900], 0, 0, 8),                                    # eight groups, the last of four tiles
    (W.DT_F16, 128, 16, 60, 1, [100], 0, 0, 8),
    (W.DT_F16, 64, 4, 32, 8, [131040], 0, 0, 1),                                    # a lone sequence as long as announced
    (W.DT_BF16, 64, 4, 32, 8, [131039], 0, 0, 1),
])
def test_pairs_of_wavefronts_by_other_routes(oracle_mod, dtype, D, G, N, Hkv, lens, split, flags, groups):
    """Pairs with two tiles each and fp32 partials, a caller's split size, several row groups, and lone sequences whose page
    list and parents are asked for along with the length."""
    planned = 131040 if lens[0] > 130000 else 131072
    case = W.make_case("pairs", 40 + N + len(lens), dtype=dtype, Hq=Hkv * G, Hkv=Hkv, D=D, ctx_lens=lens,
                       trees=[W.random_tree(N, 5, _rng(N + 10 * b)) for b in range(len(lens))])
    got, step = _run(_announced(case, planned), max_ctx_len=planned, split_tokens=split, flags=flags)
    plan = step.plan.as_dict()
    assert (plan["row_groups"], plan["tiles_per_wave"]) == (groups, 2) and plan["row_tiles"] <= 8 * groups, plan
    _close_to_oracle(oracle_mod, case, got, f"plan={plan}")


@pytest.mark.parametrize("split", [0, 1024])
@pytest.mark.parametrize("dtype,L", [(W.DT_BF16, 0), (W.DT_BF16, 100), (W.DT_F16, 9001), (W.DT_BF16, 31999), (W.DT_BF16, 32000)])
def test_three_tiles_and_a_length_short_of_the_announced(oracle_mod, dtype, L, split):
    """The three-tile kernel puts the page list that a lone sequence would have if it were as long as announced, and the
    parents, into LDS before it knows the length.  Shorter sequences have other windows, and entries of -1 in the list."""
    planned = 32000
    case = W.make_case("three", 300 + L % 89, dtype=dtype, Hq=64, Hkv=8, D=128, ctx_lens=[L], trees=[W.hybrid_tree(32, 8, _rng(L + 3))])
    got, step = _run(_announced(case, planned), max_ctx_len=planned, split_tokens=split)
    plan = step.plan.as_dict()
    assert (plan["row_groups"], plan["tiles_per_wave"]) == (1, 3), plan
    _close_to_oracle(oracle_mod, case, got, f"L={L} plan={plan}")


@pytest.mark.parametrize("split", [0, 1024])
@pytest.mark.parametrize("entry,bad", [(0, -1), (63, 10 ** 6), (1100, -7), (2002, 10 ** 6)])
def test_three_tiles_and_a_page_out_of_the_pool(oracle_mod, entry, bad, split):
    """One wavefront finds the entry in its part of the list asked for ahead and reads the list again: the flag is set, and the
    rest of the result is that of a table with page 0 in the entry's place."""
    import dataclasses
    L = 32000
    case = W.make_case("three_bad", 77, dtype=W.DT_BF16, Hq=64, Hkv=8, D=128, ctx_lens=[L], trees=[W.hybrid_tree(32, 8, _rng(5))])
    table = case.page_table.copy()
    table[0, entry] = bad
    step = VerifyStep(dataclasses.replace(case, page_table=table), split_tokens=split)
    assert step.plan.as_dict()["tiles_per_wave"] == 3
    step.run()
    got = step.result()
    assert step.dev_status() == B.OWL_DEV_BAD_PAGE
    table = table.copy()
    table[0, entry] = 0
    _close_to_oracle(oracle_mod, dataclasses.replace(case, page_table=table), got, f"entry {entry} = {bad}")


# ---------------------------------------------------------------------------
# the largest shapes the entry point takes
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("name,kw", [
    # 64 drafted nodes x 8 query heads per KV head = 512 rows = 32 row tiles: two row groups of 24 + 8 tiles
    ("n64_g8_tree", dict(dtype=W.DT_BF16, Hq=16, Hkv=2, D=128, ctx_lens=[20000], N=64, depth=8)),
    # the same with fp16 storage and head_dim 64
    ("n64_g8_f16_d64", dict(dtype=W.DT_F16, Hq=16, Hkv=2, D=64, ctx_lens=[9000, 1], N=64, depth=8)),
    # 16 query heads on ONE KV head (multi-query attention), 24 row tiles exactly: three tiles on every wave
    ("mqa_g16_n24", dict(dtype=W.DT_BF16, Hq=16, Hkv=1, D=128, ctx_lens=[15000], N=24, depth=6)),
    # no grouping at all (Hq = Hkv), the deepest chain the mask word holds
    ("mha_chain64", dict(dtype=W.DT_BF16, Hq=4, Hkv=4, D=128, ctx_lens=[5000, 33], N=64, depth=None)),
    # a forest of 64 roots: every node sees only itself among the drafts
    ("forest64", dict(dtype=W.DT_BF16, Hq=8, Hkv=2, D=128, ctx_lens=[3000], N=64, depth=0)),
])
def test_largest_shapes_every_element(oracle_mod, name, kw):
    r = _rng(sum(map(ord, name)))                      # a fixed seed per case
    N, depth = kw.pop("N"), kw.pop("depth")
    def tree():
        if depth is None:
            return W.chain_tree(N)
        if depth == 0:
            return np.full(N, -1, np.int32)
        return W.random_tree(N, depth, r)
    case = W.make_case(name, 7000 + N, trees=[tree() for _ in kw["ctx_lens"]], **kw)
    want = oracle_mod.verify_attn_case(case)
    for split in (0, 1024):
        got, step = _run(case, split_tokens=split)
        assert_close(got, want, case.dtype, f"{name} split={split} plan={step.plan.as_dict()}")


# ---------------------------------------------------------------------------
# one GPU's share of a model whose KV heads are spread over several GPUs
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("name,Hkv,G,N,L,groups,split,groups_at_split", [
    ("70b_over_8_gpus", 1, 8, 40, 24000, 5, 1472, 5),     # 20 row tiles on one KV head: five row groups of four tiles
    ("70b_over_4_gpus", 2, 8, 40, 24000, 5, 512, 3),      # two KV heads; with 47 splits: three groups of seven tiles
    ("70b_over_4_gpus_b", 2, 8, 40, 24000, 5, 256, 2),    # with 94 splits: two groups of ten (two tiles per wave)
    ("8b_over_8_gpus", 1, 4, 60, 12000, 4, 320, 4),       # 15 tiles: 4 + 4 + 4 + 3
    ("wide_on_one_head", 1, 8, 64, 6000, 8, 1472, 8),     # 32 tiles on one head of a short context: eight groups
])
def test_few_kv_heads_use_row_groups(oracle_mod, name, Hkv, G, N, L, groups, split, groups_at_split):
    """With one or two KV heads the splits alone cannot give every compute unit a workgroup: the rows
    are cut into row groups (workgroups that read the same split).  Every element against the oracle,
    with the library's own plan and with a forced split size that does not divide the context."""
    r = _rng(sum(map(ord, name)))
    case = W.make_case(name, 8100 + N, dtype=W.DT_BF16, Hq=Hkv * G, Hkv=Hkv, D=128, ctx_lens=[L],
                       trees=[W.random_tree(N, 8, r)], outlier_frac=0.05)
    want = oracle_mod.verify_attn_case(case)
    got, step = _run(case)
    assert step.plan.row_groups == groups, step.plan.as_dict()
    assert_close(got, want, case.dtype, f"{name} plan={step.plan.as_dict()}")
    got, step = _run(case, split_tokens=split)
    assert step.plan.row_groups == groups_at_split, step.plan.as_dict()
    assert_close(got, want, case.dtype, f"{name} split={split} plan={step.plan.as_dict()}")


# ---------------------------------------------------------------------------
# a context near the upper end: one million tokens, pools beyond 2^31 bytes
# ---------------------------------------------------------------------------
def test_million_token_context(oracle_mod):
    """64-bit addressing of the pool (beyond 2^31 bytes), 68 splits per KV head, page ids above 2^16."""
    L = 1_100_003
    case = W.make_case("ctx_1m", 4242, dtype=W.DT_BF16, Hq=16, Hkv=8, D=128, ctx_lens=[L],
                       trees=[W.random_tree(10, 4, _rng(3))])
    assert case.k_pool.nbytes > 2**31
    got, step = _run(case)
    rows = sample_rows(case, 10, seed=9, always=[(0, 0, 0), (0, case.N - 1, case.Hq - 1)])
    want = oracle_mod.verify_attn_case(case, rows=rows)
    sub = np.stack([got[b, i, h] for b, i, h in rows])
    assert_close(sub, want, case.dtype, f"plan={step.plan.as_dict()}")
    assert np.isfinite(got).all()
