"""gr_solve_verify (solve and verification in one launch) against gr_solve followed by gr_verify, through the C ABI:
the same kernels' arithmetic on the same policy, so acceptance probability, status, token and accepted flag are
compared bit for bit.  The two-call path is the one the other GPU tests hold against the CPU checker.  Cases: every
configuration that fits the LDS-resident path, rows that fall back to sampling from p (cap on |T|, iteration cap),
bad rows, draws that leave the drafts (uniforms near 1 walk the residual tokens), a support above GR_MAX_SUPPORT
(which keeps the two steps inside the call), a ragged tiny vocabulary, nine to sixteen drafts, and rows given as
logits (gr_solve_logits_verify against gr_solve_logits + gr_verify)."""
import numpy as np
import pytest

from paper_2511_15898_amd import workloads as W

pytestmark = pytest.mark.gpu


def _both(wl, tol, uniforms=None, drafts=None, p=None, **cfg):
    import torch
    from paper_2511_15898_amd import binding as gr
    dev = torch.device("cuda:0")
    pt = torch.from_numpy(wl.p if p is None else p).to(dev); qt = torch.from_numpy(wl.q).to(dev)
    d = torch.from_numpy(wl.drafts if drafts is None else drafts).to(dev)
    u = torch.from_numpy(wl.uniforms if uniforms is None else uniforms).to(dev)
    h = gr.gr_create(wl.B, wl.V, max_k=wl.k, max_n=wl.n, **cfg)
    try:
        acc, st = gr.gr_solve(h, pt, qt, wl.n, wl.k, tol)
        tok, ok = gr.gr_verify(h, d, u)
        two = [x.clone() for x in (acc, st, tok, ok)]
        one = gr.gr_solve_verify(h, pt, qt, wl.n, wl.k, tol, d, u)
        one = [x.clone() for x in one]
        tok2, ok2 = gr.gr_verify(h, d, u)              # the handle keeps the policy as after gr_solve
        torch.cuda.synchronize()
    finally:
        gr.gr_destroy(h)
    names = ("accept_prob", "status", "token", "accepted")
    for name, a, b in zip(names, two, one):
        if name == "accept_prob":
            assert torch.equal(a.view(torch.int32), b.view(torch.int32)), name      # NaN of a bad row included
        else:
            assert torch.equal(a, b), name
    assert torch.equal(tok2, two[2]) and torch.equal(ok2, two[3])
    return {n_: x.cpu().numpy() for n_, x in zip(names, one)}


def test_small_and_llm_shaped_and_large():
    for wl, tol in ((W.small(), 1e-6), (W.llm_shaped(seed_sub=3), 1e-6), (W.large_vocab(), 1e-4)):
        out = _both(wl, tol)
        assert np.all(out["status"] == 0)
        assert np.all((out["token"] >= 0) & (out["token"] < wl.V))
        assert 0 < out["accepted"].sum() <= wl.B


def test_draws_that_leave_the_drafts_walk_the_other_tokens():
    wl = W.large_vocab(B=64, seed_sub=7)
    rng = np.random.default_rng(11)
    u = (1.0 - rng.random(wl.B) * 0.004).astype(np.float32)               # the top of the CDF: where residual tokens sit
    u = np.minimum(u, np.float32(0.99999994))
    out = _both(wl, 1e-4, uniforms=u)
    assert (out["accepted"] == 0).sum() >= 3              # most slices leave little beyond the drafts
    wl = W.llm_shaped(B=48, V=777, n=3, k=16, seed_sub=8)                 # ragged V, one short tile
    out = _both(wl, 1e-6, uniforms=np.full(wl.B, 0.999, np.float32))
    assert (out["accepted"] == 0).sum() >= 1


def test_rows_that_fall_back_to_p_and_bad_rows():
    wl = W.large_vocab(B=32, seed_sub=9)
    p = wl.p.copy()
    p[3, 17] = np.nan                                                     # a bad row: token -1, accepted 0
    p[5] *= 0.5                                                           # row sum off by more than 1e-3
    out = _both(wl, 1e-6, p=p, max_T=8)                                   # most rows exceed the cap on |T|
    assert out["status"][3] == 3 and out["status"][5] == 3 and out["token"][3] == -1 and out["accepted"][5] == 0
    assert (out["status"] == 1).sum() >= 8                                # GR_ROW_TRUNC_CAP
    out = _both(wl, 1e-6, max_iter=2)                                     # iteration cap
    assert (out["status"] == 2).sum() >= 8                                # GR_ROW_ITER_CAP
    bad = wl.drafts.copy(); bad[1, 0] = wl.V + 5; bad[2, 1] = -1          # a draft outside the vocabulary
    out = _both(wl, 1e-4, drafts=bad)
    assert out["token"][1] == -1 and out["token"][2] == -1


def test_large_support_keeps_two_steps_and_many_drafts():
    wl = W.llm_shaped(B=8, V=5000, n=4, k=600, seed_sub=12)               # support above GR_MAX_SUPPORT: HBM-resident path
    out = _both(wl, 1e-4)
    assert np.all(out["status"] != 3)
    wl = W.llm_shaped(B=24, V=4096, n=12, k=48, seed_sub=13)              # the kernel for nine to sixteen drafts
    out = _both(wl, 1e-5)
    assert np.all(out["status"] == 0)


def test_rows_given_as_logits():
    import torch
    from paper_2511_15898_amd import binding as gr
    dev = torch.device("cuda:0")
    for wl, tol, two_temps in ((W.small(keep_logits=True), 1e-6, False), (W.large_vocab(B=64, seed_sub=21, keep_logits=True), 1e-4, True),
                               (W.llm_shaped(B=6, V=3000, n=3, k=500, seed_sub=22, keep_logits=True), 1e-4, False)):   # the last: HBM-resident support
        tl = torch.from_numpy(wl.meta["target_logits"]).to(dev); dl = torch.from_numpy(wl.meta["draft_logits"]).to(dev)
        T = torch.from_numpy(wl.meta["temps"].astype(np.float32)).to(dev)
        Td = (T * 1.25) if two_temps else None
        d = torch.from_numpy(wl.drafts).to(dev)                 # drawn from the float32 q: a draft that the logits' top-k does not
        u = torch.from_numpy(wl.uniforms).to(dev)               # hold gives token -1 on both paths alike
        h = gr.gr_create(wl.B, wl.V, max_k=wl.k, max_n=wl.n)
        try:
            acc, st = gr.gr_solve_logits(h, tl, dl, T, wl.n, wl.k, tol, draft_temperature=Td)
            tok, ok = gr.gr_verify(h, d, u)
            two = [x.clone() for x in (acc, st, tok, ok)]
            one = [x.clone() for x in gr.gr_solve_logits_verify(h, tl, dl, T, wl.n, wl.k, tol, d, u, draft_temperature=Td)]
            torch.cuda.synchronize()
        finally:
            gr.gr_destroy(h)
        for name, a, b in zip(("accept_prob", "status", "token", "accepted"), two, one):
            assert torch.equal(a.view(torch.int32) if name == "accept_prob" else a, b.view(torch.int32) if name == "accept_prob" else b), name
        assert int((one[1] == 0).sum()) >= wl.B // 2 and int((one[2] >= 0).sum()) >= wl.B // 2


@pytest.mark.parametrize("n,k,V,logits", [(1, 20, 300, False), (2, 256, 600, False), (3, 33, 1024, True), (4, 64, 1025, False), (5, 200, 700, False),
                                          (8, 128, 2000, True), (8, 9, 333, False)])
def test_batches_on_both_workgroup_sizes(n, k, V, logits):
    """Batches of more than 256, 320 or 448 rows, by the draft count, run two smaller workgroups to a compute unit: the same rows in one batch of
    460 and in halves.  The routed masses are summed over other waves, so programs agree to their stopping measure (1e-8), far inside 1e-6."""
    import torch
    from paper_2511_15898_amd import binding as gr
    B = 460
    wl = W.llm_shaped(B=B, V=V, n=n, k=k, temperature=(0.5, 1.5), near_identical_frac=0.2, seed_sub=2000 + V)
    dev = torch.device("cuda:0")
    p, q = torch.from_numpy(wl.p).to(dev), torch.from_numpy(wl.q).to(dev)
    drafts, u = torch.from_numpy(wl.drafts).to(dev), torch.from_numpy(wl.uniforms).to(dev)
    temp = torch.ones(B, device=dev)
    h = gr.gr_create(B, V, max_k=k, max_n=n)
    def run(rows):
        if logits:
            gr.gr_solve_logits(h, p[rows].log().contiguous(), q[rows].log().contiguous(), temp[rows], n, k, 1e-4)
        else:
            gr.gr_solve(h, p[rows].contiguous(), q[rows].contiguous(), n, k, 1e-4)
        pi, given = gr.gr_policy_slice(h, drafts[rows].contiguous(), V)
        one = (gr.gr_solve_verify(h, p[rows].contiguous(), q[rows].contiguous(), n, k, 1e-4, drafts[rows].contiguous(), u[rows].contiguous()))
        return (pi, given) + tuple(one)
    try:
        whole = [x.cpu().numpy() for x in run(slice(0, B))]
        halves = [np.concatenate([a.cpu().numpy(), b.cpu().numpy()]) for a, b in zip(run(slice(0, 230)), run(slice(230, B)))]
    finally:
        gr.gr_destroy(h)
    pi, given, acc, st, tok, ok = zip(whole, halves)
    assert np.array_equal(*st) and np.array_equal(*acc)
    assert np.abs(pi[0] - pi[1]).max() < 1e-6 and np.abs(given[0] - given[1]).max() < 1e-6
    assert (tok[0] != tok[1]).sum() <= 1 and (ok[0] != ok[1]).sum() <= 1      # a uniform on an edge


@pytest.mark.parametrize("n,k,V", [(2, 12, 64), (3, 12, 64), (4, 12, 64), (8, 12, 64), (4, 0, 300)])
def test_programs_that_take_long_in_large_batches(n, k, V):
    """A tolerance that no evaluation meets: every row with a program of a batch of 460 is left to the second launch, with large workgroups, which goes on
    from its best weights through the step's budget and the finite differences to the cap.  Its weights must be those of rows solved to 1e-12 in
    batches of 230.  Bound: w answers to its target R as R / (P - R) does, P the token's draw probability: 1 + w times the measure, summed over the
    tokens that move with it, for which a thousandfold is allowed at the least.  A cap of 12 evaluations is reached in the first launch."""
    from dataclasses import replace
    from parity_util import run_gpu
    B = 460
    wl = W.small(B=B, V=V, n=n, k=k, seed_sub=n + 12)
    part = lambda rows: replace(wl, B=230, p=wl.p[rows], q=wl.q[rows], drafts=wl.drafts[rows], uniforms=wl.uniforms[rows])
    def run(w, **how):
        out = run_gpu(w, 1e-5 if k else 0.05, want_slice=False, export_rows=range(w.B), **how)   # a whole row's programs would end above the cap
        if "rows" in out:
            for name in ("order", "block", "weight"):
                out[name] = np.zeros((w.B, V))
                for b, r in out["rows"].items():
                    out[name][b, : len(r[name])] = r[name]
            del out["rows"]
        return out
    def both(**how):
        first, second = run(part(slice(0, 230)), **how), run(part(slice(230, B)), **how)
        return {name: np.concatenate([first[name], second[name]]) for name in first}
    solved, out = both(rel_tol=1e-12), run(wl, rel_tol=1e-17, max_iter=200)
    fine = solved["status"] == 0
    ran = fine & (solved["iterations"] > 0)
    assert ran.sum() >= B // 2
    long = ran & (out["status"] == 2)                          # the measure of a small program can come out 0 exactly
    assert long.sum() >= 0.9 * ran.sum() and np.all(out["status"][fine & ~long] == 0) and np.all(out["iterations"][long] >= 200)
    assert np.array_equal(out["accept_prob"], solved["accept_prob"]) and np.array_equal(out["support"], solved["support"])
    for b in np.flatnonzero(ran):
        kk = out["support"][b]
        assert np.array_equal(out["order"][b, :kk], solved["order"][b, :kk]) and np.array_equal(out["block"][b, :kk], solved["block"][b, :kk])
        w, want = out["weight"][b, :kk], solved["weight"][b, :kk]
        assert np.array_equal(w > 0, want > 0) and np.abs(w[want > 0] / want[want > 0] - 1.0).max() < 1e-12 * max(1e3, 1.0 + want.max()), b
    short, halves = run(wl, rel_tol=1e-17, max_iter=12), both(rel_tol=1e-17, max_iter=12)
    assert np.mean((short["status"] == halves["status"]) & (short["iterations"] == halves["iterations"])) >= 0.9      # a measure of exactly 0 again
