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
