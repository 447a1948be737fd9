"""The reduced Newton step at the edges of its layout: programs of fewer tokens than the eight whose couplings it computes, of one
more, of one and of two tokens per lane of the stepping wave, at the smallest and largest draft count of every kernel; and how
many evaluations it takes (the fixed-point iteration that stood here needed twice as many on these rows)."""
import numpy as np
import pytest

from parity_util import compare_rows, run_gpu
from paper_2511_15898_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("k", [2, 7, 8, 9, 10, 16, 17, 64, 65, 72])
def test_sizes_around_the_step_s_layout(n, k):
    wl = W.small(B=4, V=512, n=n, k=k, seed_sub=100 * n + k)
    out = run_gpu(wl, 1e-6)
    compare_rows(wl, out, range(wl.B), 1e-6)
    assert np.all(out["status"] == 0) and out["iterations"].max() <= 24, out["iterations"]


@pytest.mark.parametrize("n, most, mean_most", [(2, 24, 7.0), (4, 14, 5.5), (8, 12, 5.0), (16, 14, 5.0)])
def test_evaluations_of_the_step(n, most, mean_most):
    wl = W.llm_shaped(B=256, V=8000, n=n, k=128, temperature=(0.5, 1.5), near_identical_frac=0.1, seed_sub=900 + n)
    out = run_gpu(wl, 1e-4, want_slice=False)
    assert np.mean(out["status"] == 0) > 0.99
    ev = out["iterations"][out["status"] == 0]
    assert ev.max() <= most and ev.mean() <= mean_most, (int(ev.max()), float(ev.mean()))


@pytest.mark.parametrize("n", [2, 4, 8, 9, 16])
def test_the_finite_differences_stay_at_the_solution(n):
    """A tolerance that no evaluation meets: the step's budget of 120 + m evaluations ends, and the damped Newton iteration with a
    finite-difference Jacobian goes on from its best point to the iteration cap, on the evaluator and the order of tokens that the
    step uses.  The rows end at the cap; their weights must be those of rows solved to 1e-12 (a target's saturation amplifies that
    at most a thousandfold on these rows)."""
    wl = W.small(B=6, V=64, n=n, k=12, seed_sub=n + 12)
    solved = run_gpu(wl, 1e-5, rel_tol=1e-12)
    out = run_gpu(wl, 1e-5, rel_tol=1e-17, max_iter=200)
    assert np.all(solved["status"] == 0) and solved["iterations"].max() < 60          # the step alone
    ran = solved["iterations"] > 0                         # rows with a program
    assert ran.sum() >= 4 and np.all(out["status"][ran] == 2) and np.all(out["iterations"][ran] >= 200), out["iterations"]
    assert np.array_equal(out["order"], solved["order"]) and np.array_equal(out["block"], solved["block"])
    w, want = out["weight"][ran], solved["weight"][ran]
    kk = out["support"][ran]
    for b in range(len(kk)):
        some = want[b, : kk[b]] > 0
        assert np.array_equal(w[b, : kk[b]] > 0, some)
        assert np.abs(w[b, : kk[b]][some] / want[b, : kk[b]][some] - 1.0).max() < 1e-9, b


def test_rows_that_held_the_step_up():
    """Rows found among fifteen million random ones (golden/stubborn_rows.json): a token that saturates, whose step without a bound kept
    all others from theirs; slow modes of blocks without slack, which a secant pair ends; a secant step gone astray, halved twenty
    times; light tokens that meet only one another, and an acceptance near 0, where the fixed-point step is the better one.  Four of
    them ended at the cap after 1000 evaluations, the others took 41 to 788; the mixed iteration that stood here 2 to 57."""
    import json
    import os
    rows = json.load(open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "stubborn_rows.json")))
    took = []
    for i, r in enumerate(rows):
        p, q = np.array([r["p"]], np.float32), np.array([r["q"]], np.float32)
        wl = W._finish("stubborn", p, q, r["n"], r["k"], np.random.default_rng(i))
        out = run_gpu(wl, r["tol"])
        compare_rows(wl, out, [0], r["tol"])
        assert out["status"][0] == 0, (i, out["iterations"])
        took.append(int(out["iterations"][0]))
    assert max(took) <= 80 and np.mean(took) <= 32, took
