"""GPU parity of the acceptance-only sweep (gr_accept_sweep) against the CPU checker's
acceptance_sweep: alpha*(k, n) over a grid of top-k sizes and draft counts, element by element."""
import numpy as np
import pytest
import torch

from paper_2511_15898_amd import binding as gr, workloads as W

pytestmark = pytest.mark.gpu
ABS_TOL = 1e-5          # spec tolerance on alpha*


def _sweep(p, q, ks, ns, max_k=gr.GR_MAX_SUPPORT):
    dev = torch.device("cuda:0")
    B, V = p.shape
    h = gr.gr_create(B, V, max_k=max_k)
    try:
        acc, st = gr.gr_accept_sweep(h, torch.from_numpy(p).to(dev), torch.from_numpy(q).to(dev), ks, ns)
        torch.cuda.synchronize()
        return acc.cpu().numpy(), st.cpu().numpy()
    finally:
        gr.gr_destroy(h)


def _check(p, q, ks, ns, rows, acc):
    from oracle import gr_oracle as G
    worst = 0.0
    for b in rows:
        want = G.acceptance_sweep(p[b], q[b], ks, ns)
        d = float(np.abs(acc[b] - want).max())
        assert d < ABS_TOL, (b, d, acc[b], want)
        worst = max(worst, d)
    return worst


def test_small_config_every_row_every_cell():
    wl = W.small()
    ks, ns = [1, 2, 7, 32, 100, 256], [1, 2, 3, 4, 8, 16, 64]
    acc, st = _sweep(wl.p, wl.q, ks, ns)
    assert np.all(st == 0)
    _check(wl.p, wl.q, ks, ns, range(wl.B), acc)
    assert np.all(np.diff(acc, axis=2) >= -1e-6)            # nondecreasing in n
    assert np.all(acc[:, 0, :] <= acc[:, 0, :1] + 1e-6)     # one-token support: a single token is certain, more drafts add nothing


def test_large_vocab_full_size_sampled_rows_and_consistency_with_solve():
    """BASELINE's large-vocabulary batch at full size: sampled rows against the checker, every row
    for monotonicity, and the (k, n) cell of the bench configuration against gr_solve's alpha*."""
    wl = W.large_vocab()
    ks, ns = [8, 32, 128], [1, 2, 4, 8]
    acc, st = _sweep(wl.p, wl.q, ks, ns)
    assert np.all(st == 0)
    rows = list(range(0, wl.B, 23))
    _check(wl.p, wl.q, ks, ns, rows, acc)
    assert np.all(np.diff(acc, axis=2) >= -1e-6)
    dev = torch.device("cuda:0")
    h = gr.gr_create(wl.B, wl.V)
    try:
        a, _ = gr.gr_solve(h, torch.from_numpy(wl.p).to(dev), torch.from_numpy(wl.q).to(dev), wl.n, wl.k, 1e-4)
        torch.cuda.synchronize()
        assert np.abs(a.cpu().numpy() - acc[:, ks.index(wl.k), ns.index(wl.n)]).max() < 1e-6
    finally:
        gr.gr_destroy(h)


@pytest.mark.parametrize("B,V", [(1, 8), (3, 1001), (5, 4099), (2, 255)])
def test_ragged_shapes_zeros_and_small_supports(B, V):
    rng = np.random.default_rng(B * 100 + V)
    p = rng.dirichlet(np.full(V, 0.3), size=B).astype(np.float32)
    q = rng.dirichlet(np.full(V, 0.3), size=B).astype(np.float32)
    q[:, 5:] *= (rng.random((B, V - 5)) < 0.5)              # exact zeros in q: supports smaller than k
    p[:, ::3] = 0.0                                         # p = 0 where q > 0 ranks first
    p = (p / p.sum(1, keepdims=True)).astype(np.float32); q = (q / q.sum(1, keepdims=True)).astype(np.float32)
    ks, ns = [1, 3, 64, 256], [1, 2, 5, 10]
    acc, st = _sweep(p, q, ks, ns)
    assert np.all(st == 0)
    _check(p, q, ks, ns, range(B), acc)


def test_identical_rows_accept_everything_and_bad_rows_are_flagged():
    rng = np.random.default_rng(3)
    p = rng.dirichlet(np.full(500, 0.2), size=4).astype(np.float32)
    q = p.copy()
    q[2, 7] = np.nan                                        # bad row
    p[3] *= 0.5                                             # row sum far from 1
    ks, ns = [256], [1, 4]
    acc, st = _sweep(p, q, ks, ns)
    assert list(st) == [0, 0, 3, 3]
    assert np.all(np.isnan(acc[2:]))
    # p = q over a support of at most 256 tokens out of 500: the top-k draft differs from p, so compare with the checker
    _check(p, q, ks, ns, [0, 1], acc)
    # a top-k that covers the whole support of p = q accepts with certainty
    p2 = np.zeros((2, 300), np.float32); p2[:, :100] = rng.dirichlet(np.full(100, 0.5), size=2)
    acc2, st2 = _sweep(p2, p2.copy(), [128], [1, 3])
    assert np.all(st2 == 0) and np.abs(acc2 - 1.0).max() < 1e-6


def test_argument_checks_and_handle_state():
    dev = torch.device("cuda:0")
    wl = W.small(B=4)
    p = torch.from_numpy(wl.p).to(dev); q = torch.from_numpy(wl.q).to(dev)
    h = gr.gr_create(4, wl.V)
    try:
        for ks, ns in (([0], [2]), ([257], [2]), ([8], [0]), ([8], [65]), ([8] * 9, [2]), ([8], [2] * 17), ([], [2])):
            with pytest.raises(gr.GrError) as e:
                gr.gr_accept_sweep(h, p, q, ks, ns)
            assert e.value.code == gr.GR_EINVAL
        gr.gr_solve(h, p, q, wl.n, wl.k, 1e-4)
        gr.gr_accept_sweep(h, p, q, [8], [2])
        with pytest.raises(gr.GrError) as e:                # the sweep took the handle's selection scratch
            gr.gr_verify(h, torch.from_numpy(wl.drafts).to(dev), torch.from_numpy(wl.uniforms).to(dev))
        assert e.value.code == gr.GR_ESTATE
        torch.cuda.synchronize()
    finally:
        gr.gr_destroy(h)


@pytest.mark.parametrize("seed", [1, 2])
def test_random_grids(seed):
    """Seeded random shapes, generators, exact zeros and grids (top-k sizes 1..256, draft counts 1..64)."""
    rng = np.random.default_rng(9000 + seed)
    for case in range(30):
        B = int(rng.integers(1, 7))
        V = int(rng.integers(2, 3000)) if case % 10 else int(rng.integers(20000, 140000))
        ss = int(rng.integers(1e6))
        gen = int(rng.integers(0, 3))
        if gen == 0:
            wl = W.llm_shaped(B=B, V=V, n=2, k=0, temperature=(0.3, 2.0), near_identical_frac=0.2, seed_sub=ss)
        elif gen == 1:
            wl = W.small(B=B, V=V, n=2, k=0, seed_sub=ss)
        else:
            wl = W.tiny(B=B, V=V, n=2, seed_sub=ss)
        p, q = wl.p.copy(), wl.q.copy()
        if rng.random() < 0.4:
            zq = rng.random(q.shape) < rng.choice([0.05, 0.5, 0.9]); zq[np.arange(B), q.argmax(1)] = False; q[zq] = 0
            zp = rng.random(p.shape) < 0.1; zp[np.arange(B), p.argmax(1)] = False; p[zp] = 0
            q = (q / q.sum(1, keepdims=True, dtype=np.float32)).astype(np.float32)
            p = (p / p.sum(1, keepdims=True, dtype=np.float32)).astype(np.float32)
        ks = [int(x) for x in rng.integers(1, 257, size=int(rng.integers(1, 9)))]
        ns = [int(x) for x in rng.integers(1, 65, size=int(rng.integers(1, 17)))]
        acc, st = _sweep(np.ascontiguousarray(p), np.ascontiguousarray(q), ks, ns)
        assert np.all(st == 0), (seed, case)
        _check(p, q, ks, ns, range(B), acc)


def test_top_k_sizes_up_to_the_whole_vocabulary():
    """Sec. 7, first experiment: the acceptance study runs k from 10 to V.  Grids that reach beyond GR_MAX_SUPPORT
    run on the HBM-resident ordering; every cell against the checker on mid-size rows, cells at or below
    GR_MAX_SUPPORT also against the streaming route, and acceptance must not fall when k grows at n = 1...
    (it need not be monotone in k for n > 1, so only the checker decides there)."""
    wl = W.llm_shaped(B=12, V=5000, n=4, k=0, seed_sub=71)
    ks, ns = [10, 100, 256, 1000, 4999, 0], [1, 2, 4, 8, 16]
    acc, st = _sweep(wl.p, wl.q, ks, ns, max_k=0)
    assert np.all(st == 0)
    _check(wl.p, wl.q, ks, ns, range(wl.B), acc)
    small, _ = _sweep(wl.p, wl.q, [10, 100, 256], ns)
    assert np.abs(small - acc[:, :3, :]).max() < 2e-6
    assert np.all(np.diff(acc, axis=2) >= -1e-6)
    with pytest.raises(gr.GrError) as e:                  # a handle without the workspace refuses the large grid
        _sweep(wl.p, wl.q, ks, ns)
    assert e.value.code == gr.GR_EINVAL
    # rows with exact zeros in q and a top-k above the number of positive entries
    q = wl.q.copy(); q[:, ::3] = 0.0; q = (q / q.sum(1, keepdims=True, dtype=np.float32)).astype(np.float32)
    acc, st = _sweep(wl.p, q, [300, 2000, 0], [2, 5], max_k=0)
    _check(wl.p, q, [300, 2000, 0], [2, 5], range(wl.B), acc)


def test_top_k_sizes_up_to_the_whole_vocabulary_at_full_width():
    """Two rows of the large-vocabulary configuration, k up to V = 128256 (the checker orders 128256 tokens per k)."""
    wl = W.large_vocab(B=2)
    ks, ns = [128, 1000, 10000, 0], [2, 8]
    acc, st = _sweep(wl.p, wl.q, ks, ns, max_k=0)
    assert np.all(st == 0)
    _check(wl.p, wl.q, ks, ns, range(wl.B), acc)


@pytest.mark.parametrize("V,ns", [(8192, [7, 1, 64, 7, 2]), (8193, [16, 16, 3]), (12289, list(range(16, 0, -1)))])
def test_draft_counts_in_any_order_on_both_workgroup_sizes(V, ns):
    """Draft counts unsorted and repeated come back in the caller's order; vocabularies on both sides of the large
    workgroup's threshold, top-k sizes that leave whole waves without a token of the support.  Same bound as above."""
    wl = W.llm_shaped(B=3, V=V, n=4, k=0, temperature=(0.5, 1.5), near_identical_frac=0.3, seed_sub=V)
    ks = [0, 3, 257, V - 1]
    acc, st = _sweep(wl.p, wl.q, ks, ns, max_k=0)
    assert np.all(st == 0)
    _check(wl.p, wl.q, ks, ns, range(wl.B), acc)


@pytest.mark.parametrize("V", [1001, 5000, 8192, 8193, 12289])
def test_grids_that_end_below_half_the_vocabulary(V):
    """The ranks by q of a support of at most half the vocabulary come from its own tokens: a largest top-k size on both
    sides of V / 2, many equal q across the sizes' ends (ties by token id), and rows of which most q are zero."""
    wl = W.llm_shaped(B=4, V=V, n=2, k=0, temperature=(0.5, 1.5), seed_sub=V)
    p, q = wl.p.copy(), wl.q.copy()
    q[1] = np.round(q[1] * (4.0 * V)) + 1.0                          # few distinct values
    q[2, np.random.default_rng(V).random(V) < 0.6] = 0.0
    q[3] = 1.0
    q = (q / q.sum(1, keepdims=True, dtype=np.float64)).astype(np.float32)
    for ks in ([10, 300], [300, V // 2 - 1, 64], [V // 2, 17], [V // 2 + 1, 257]):
        acc, st = _sweep(p, q, ks, [1, 2, 8], max_k=0)
        assert np.all(st == 0)
        _check(p, q, ks, [1, 2, 8], range(4), acc)
    acc, st = _sweep(p[2:3], q[2:3], [0, 300], [1, 2, 8], max_k=0)     # no top-k: the zeros leave a support below V / 2
    assert np.all(st == 0)
    _check(p[2:3], q[2:3], [0, 300], [1, 2, 8], [0], acc)


@pytest.mark.parametrize("V", [257, 511, 4097, 12290, 20001])
def test_rows_that_take_the_bins_to_their_ends(V):
    """What the bins of the ratio have to resolve: a draft that is the target up to noise (one bin, cut again and again), equal rows, rows of
    two ratios, flat drafts (the thresholds lie among equal q, more of them than one list holds), masked targets and ratios many
    octaves apart, rows that begin anywhere (V odd).  F is found to 1e-13; the bound is that of a float32 result."""
    from oracle import gr_oracle as G
    rng = np.random.default_rng(V)
    base = rng.dirichlet(np.full(V, 0.4)) + 1e-12
    p = np.stack([base] * 7); q = p.copy()
    q[0] *= np.exp(0.01 * rng.standard_normal(V))                       # draft close to the target
    q[1] *= 1.0 + 1e-7 * rng.standard_normal(V)                         # the target up to the rounding of float32
    q[3] = np.where(rng.random(V) < 0.5, 2.0, 0.7) * p[3]               # two ratios
    q[4] = 1.0                                                          # flat: every threshold among equal q
    p[5, rng.random(V) < 0.3] = 0.0; q[5, rng.random(V) < 0.3] = 0.0    # masked tokens on both sides
    p[6] = np.exp(-60.0 * rng.random(V)); q[6] = np.exp(-60.0 * rng.random(V))
    p = (p / p.sum(1, keepdims=True)).astype(np.float32); q = (q / q.sum(1, keepdims=True)).astype(np.float32)
    ks, ns = [0, 1, 2, 255, V - 1, V // 2, 100, 100], [1, 2, 3, 16, 64]
    acc, st = _sweep(p, q, ks, ns, max_k=0)
    assert np.all(st == 0)
    for b in range(len(p)):
        want = G.acceptance_sweep(p[b], q[b], ks, ns)
        assert np.abs(acc[b] - want).max() <= 2e-7, (b, acc[b], want)    # two roundings of a value up to 1 to float32
    again, _ = _sweep(p, q, ks, ns, max_k=0)
    assert np.array_equal(acc, again)


@pytest.mark.parametrize("V,positive", [(2047, 2047), (2048, 2048), (2049, 2049), (2050, 2050), (6000, 2049), (20001, 2049)])
def test_rows_with_about_as_many_tokens_as_are_kept_at_hand(V, positive):
    """Supports on both sides of the 2048 tokens that the later rounds find at hand, drafts close enough to the target that there are
    such rounds; zeros among the tokens or none.  Bound: two roundings of a value up to 1 to float32."""
    from oracle import gr_oracle as G
    rng = np.random.default_rng(V + positive)
    base = rng.dirichlet(np.full(V, 2.0), size=6) + 1e-9
    p, q = base.copy(), base.copy()
    for b, near in enumerate([1e-2, 1e-4, 1e-6, 0.0, 0.3, 1.0]):
        q[b] *= np.exp(near * rng.standard_normal(V))
        q[b, rng.permutation(V)[positive:]] = 0.0
    p = (p / p.sum(1, keepdims=True)).astype(np.float32); q = (q / q.sum(1, keepdims=True)).astype(np.float32)
    assert np.all((q > 0).sum(1) == positive)
    ks, ns = [0, positive, positive - 1, 300, 20], [1, 2, 5, 16]
    acc, st = _sweep(p, q, ks, ns, max_k=0)
    assert np.all(st == 0)
    for b in range(len(p)):
        want = G.acceptance_sweep(p[b], q[b], ks, ns)
        assert np.abs(acc[b] - want).max() <= 2e-7, (b, acc[b], want)


@pytest.mark.parametrize("V,gap", [(128256, 16), (128256, 20), (131077, 24)])
def test_small_acceptances_of_targets_and_drafts_apart(V, gap):
    """Half of the tokens for the target, half for the draft, `gap` nats apart: acceptances of 1e-6 to 1e-11, which hang on the sums of many
    tokens too small to be whole in the kernel's units.  Bound: the acceptance's rounding to float32 and, in float64, four roundings for each of n
    factors Q and of the difference from 1."""
    rng = np.random.default_rng(gap)
    wide = np.longdouble
    p, q = np.empty((3, V), np.float32), np.empty((3, V), np.float32)
    for b in range(3):
        t, d, half = rng.gumbel(size=V), rng.gumbel(size=V), rng.random(V) < 0.5
        t[half] -= gap; d[~half] -= gap
        p[b], q[b] = np.exp(t) / np.exp(t).sum(), np.exp(d) / np.exp(d).sum()
    ks, ns = [0, V // 2, 5000], [1, 3, 8]
    acc, st = _sweep(p, q, ks, ns, max_k=0)
    assert np.all(st == 0)
    for b in range(3):
        total = p[b].sum(dtype=wide)
        for a, k in enumerate(ks):
            ids = np.argsort(-q[b], kind="stable")[:k or V]
            order = ids[np.argsort(-q[b, ids].astype(np.float64) / p[b, ids].astype(np.float64), kind="stable")]
            P = np.cumsum(p[b, order].astype(wide)) / total
            Q = np.cumsum(q[b, order].astype(wide)); Q /= Q[-1]
            for c, n in enumerate(ns):
                want = 1.0 + min(wide(0.0), (P - Q ** n).min())
                assert abs(acc[b, a, c] - want) <= 2.0 ** -24 * want + (4 * n + 8) * 2.0 ** -53, (b, k, n, acc[b, a, c], want)
