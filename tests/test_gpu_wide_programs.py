"""Programs whose targets, and so their weights, lie many decades apart: the step is taken in float32, the weights and the
stopping measure are not."""
import numpy as np
import pytest

from parity_util import compare_rows, run_gpu
from paper_2511_15898_amd import workloads as W

pytestmark = pytest.mark.gpu


def _one_block(V, n, tiny):
    """Rows that are one outer block over the whole vocabulary (F >= 0 throughout and F(V) = 0 exactly: every sum is dyadic), the
    first token's target `tiny` and its draw mass small enough for F(1) > 0."""
    p, q = np.full((len(tiny), V), 1.0 / V), np.full((len(tiny), V), 1.0 / V)
    for b, t in enumerate(tiny):
        first = 2.0 ** -8
        while first ** n > 0.25 * t:
            first *= 0.5
        q[b, 1] += q[b, 0] - first; q[b, 0] = first
        p[b, 1] += p[b, 0]; p[b, 0] = t
    rng = np.random.default_rng(V + n)
    wl = W._finish("block", p.astype(np.float32), q.astype(np.float32), n, 0, rng)
    return wl


def _check_weights(wl, out, tol):
    """Every row solved, its weights those of the checker: both stop at 1e-8 of the targets or closer, and a program's weights
    answer to its targets at most a hundredfold here."""
    from oracle import gr_oracle as G
    compare_rows(wl, out, range(wl.B), tol)
    for b in range(wl.B):
        sol = G.solve_row(wl.p[b], wl.q[b], wl.n, wl.k, tol=tol, max_T=128)
        assert out["status"][b] == sol.status == 0 and out["h_size"][b] == sol.h, (b, out["status"][b])
        w = out["weight"][b, : len(sol.order)]
        assert np.array_equal(out["order"][b, : len(sol.order)], sol.order) and np.all((w > 0) == (sol.w > 0))
        some = sol.w > 0
        assert np.abs(w[some] / sol.w[some] - 1.0).max() < 1e-6, (b, w, sol.w)


@pytest.mark.parametrize("V", [16, 32])
def test_a_step_that_is_not_a_number_is_not_taken(V):
    """Weights 37 to 40 decades apart without slack, where the couplings overflow float32.  The fixed-point iteration that is taken
    in place of such a step needs no more than a few evaluations here; the finite differences took a thousand and gave up."""
    wl = _one_block(V, 16, [1e-38, 1e-39, 1e-41])
    out = run_gpu(wl, 1e-7)
    _check_weights(wl, out, 1e-7)
    assert out["iterations"].max() <= 24, out["iterations"]
