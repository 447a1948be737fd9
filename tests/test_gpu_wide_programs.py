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


def _check_weights(wl, out, tol, token=None):
    """Every row solved, its weights those of the checker: both stop at 1e-8 of the targets or closer, and a program's weights
    answer to its targets at most a hundredfold here.  token [B]: of this token alone, where others take nearly all of the probability
    that they are drawn, or none but what no weight moves (such weights answer without a bound)."""
    from oracle import gr_oracle as G
    compare_rows(wl, out, range(wl.B), tol)
    for b in range(wl.B):
        sol = G.solve_row(wl.p[b], wl.q[b], wl.n, wl.k, tol=tol, max_T=128)
        assert out["status"][b] == sol.status == 0 and out["h_size"][b] == sol.h, (b, out["status"][b])
        w = out["weight"][b, : len(sol.order)]
        assert np.array_equal(out["order"][b, : len(sol.order)], sol.order) and np.all((w > 0) == (sol.w > 0))
        some = sol.w > 0 if token is None else (sol.order == token[b]) & (sol.w > 0)
        assert np.all(np.abs(w[some] / sol.w[some] - 1.0) < 1e-6), (b, w, sol.w)


@pytest.mark.parametrize("V", [16, 32])
def test_a_step_that_is_not_a_number_is_not_taken(V):
    """Weights 37 to 40 decades apart without slack, where the couplings overflow float32.  The fixed-point iteration that is taken
    in place of such a step needs no more than a few evaluations here; the finite differences took a thousand and gave up."""
    wl = _one_block(V, 16, [1e-38, 1e-39, 1e-41])
    out = run_gpu(wl, 1e-7)
    _check_weights(wl, out, 1e-7)
    assert out["iterations"].max() <= 24, out["iterations"]


@pytest.mark.parametrize("n", [8, 9, 12, 16])
@pytest.mark.parametrize("V", [8, 16, 32, 64])
def test_couplings_of_light_tokens_stay_finite(V, n):
    """The weight of a coupling at a node grows with the node's place, which is the inverse of the lightest weight: as infinity it met
    factors that had vanished, and no token had Newton's step.  Rows ended at the cap after 1000 evaluations, or took up to 22 on
    fixed-point steps."""
    wl = _one_block(V, n, [1e-30, 1e-35, 1e-37, 1e-38, 1e-39, 1e-41, 1e-44])
    out = run_gpu(wl, 1e-7)
    _check_weights(wl, out, 1e-7, np.ones(wl.B, int))       # not the light token's: its share of tuples that it fills alone takes four cumulants
    assert out["iterations"].max() <= 10, out["iterations"]


def _favoured(V, k, n, gaps):
    """Rows whose draft likes one token best that the target all but excludes: its target logit lies `gap` below the largest."""
    rng = np.random.default_rng(1000 * V + 10 * k + n)
    t = 2.0 * rng.gumbel(size=(len(gaps), V))
    d = 0.8 * t + rng.normal(size=t.shape)
    token = []
    for b, gap in enumerate(gaps):
        x = int(rng.integers(V))
        token.append(x)
        t[b, x] = t[b].max() - gap
        d[b, x] = d[b].max() + 0.5
    t, d = t.astype(np.float32), d.astype(np.float32)
    return W._finish("favoured", W._softmax32(t.astype(np.float64)), W._softmax32(d.astype(np.float64)), n, k, rng,
                     {"target_logits": t, "draft_logits": d, "temps": np.ones(len(gaps)), "token": np.array(token)})


@pytest.mark.parametrize("V, k, n", [(40, 6, 2), (40, 8, 4), (12, 7, 8), (64, 0, 9), (64, 0, 16)])
def test_a_light_token_that_comes_first_does_not_steer_the_step(V, k, n):
    """Programs that list a token of tiny target first: those of up to eight tokens (decreasing q) and a token above 0.3 of the draw
    mass with more than eight drafts.  With that token held the step was rounding: 37 to 316 evaluations."""
    wl = _favoured(V, k, n, [40, 50, 60, 65, 70, 75, 80])
    out = run_gpu(wl, 1e-5)
    _check_weights(wl, out, 1e-5, wl.meta["token"])
    assert out["iterations"].max() <= 24, out["iterations"]


@pytest.mark.parametrize("V, k, n", [(64, 0, 2), (64, 0, 9), (512, 64, 4), (300, 100, 8), (40, 6, 2), (40, 6, 16)])
def test_a_token_too_light_for_the_step_s_float32(V, k, n):
    """Target gaps up to the last float32 probability and, as logits, beyond it (a token banned by its logit): the reciprocal of such
    a token's row overflowed, and the step of every token with it.  60 to 480 evaluations."""
    from test_gpu_logits import _compare, _drafts_from_logits, _run_logits
    wl = _favoured(V, k, n, [84, 88, 92, 98, 103, 106, 110, 200])
    out = run_gpu(wl, 1e-5)
    _check_weights(wl, out, 1e-5, wl.meta["token"])
    assert out["iterations"].max() <= 24, out["iterations"]
    drafts = _drafts_from_logits(wl, range(wl.B), 3)
    out = _run_logits(wl, 1e-5, drafts)
    _compare(wl, out, range(wl.B), 1e-5, drafts)
    assert np.all(out["status"] == 0) and out["iterations"].max() <= 24, out["iterations"]
