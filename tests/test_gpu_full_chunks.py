"""Supports above 256 tokens at the edges of the scan's tiles (2048 ranks) and of the chunks that gather and scatter, with row
counts that leave some of the chunk kernels' workgroups without a row: alpha* on every row, everything else on sampled rows."""
import numpy as np
import pytest

from paper_2511_15898_amd import workloads as W
from parity_util import check_alpha_all_rows, compare_rows, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [5, 66])
@pytest.mark.parametrize("V", [257, 2047, 2048, 2049, 4097])
def test_rows_at_tile_edges(B, V):
    wl = W.llm_shaped(B=B, V=V, n=3, k=0, seed_sub=1300 + V)
    rows = sorted({0, B // 2, B - 1})
    out = run_gpu(wl, 1e-3, export_rows=rows)
    check_alpha_all_rows(wl, out)
    stats = compare_rows(wl, out, rows, 1e-3)
    assert stats["rows"] == len(rows)


@pytest.mark.parametrize("V", [2048, 2049, 9001])
def test_flat_rows_end_above_the_cap(V):
    """Dirichlet rows whose truncation sets hold thousands of tokens: the count alone ends them."""
    wl = W.tiny(B=4, V=V, n=2)
    out = run_gpu(wl, 1e-4, export_rows=range(wl.B))
    check_alpha_all_rows(wl, out)
    compare_rows(wl, out, range(wl.B), 1e-4)
    assert np.all(out["status"] != 0)


@pytest.mark.parametrize("V", [65536, 65537, 73729])
def test_rows_on_both_sort_tiles(V):
    """Rows up to and above the length that takes the sort's longer tiles, with a last tile of one token."""
    wl = W.llm_shaped(B=2, V=V, n=2, k=0, seed_sub=1400 + V)
    out = run_gpu(wl, 1e-3, export_rows=range(wl.B))
    check_alpha_all_rows(wl, out)
    compare_rows(wl, out, range(wl.B), 1e-3)


@pytest.mark.parametrize("V", [1000, 1023, 1024, 1025, 1033])
def test_sums_of_the_ranks_that_one_wave_adds(V):
    """Rows up to the length that one wave adds alone, and above it: supports that end in and behind its last lane."""
    wl = W.llm_shaped(B=3, V=V, n=3, k=0, seed_sub=1500 + V)
    out = run_gpu(wl, 1e-3, export_rows=range(wl.B))
    check_alpha_all_rows(wl, out)
    compare_rows(wl, out, range(wl.B), 1e-3)


@pytest.mark.parametrize("B, V, top", [(3, 301, 290), (2, 1025, 513), (2, 8192, 300), (2, 8192, 0), (63, 8193, 0), (64, 8193, 4097), (66, 8193, 4096),
                                       (2, 12289, 0), (1, 65537, 0)])
def test_grids_on_both_sides_of_the_short_rows(B, V, top):
    """Rows that gather for themselves and rows that have it done, supports above and up to half of the vocabulary, row counts on both
    sides of the one from which a row's chunks share an XCD, and draft masses that tie at the ends of the supports."""
    import torch
    from oracle import gr_oracle as G
    from paper_2511_15898_amd import binding as gr
    rng = np.random.default_rng(B * V + top)
    wl = W.llm_shaped(B=B, V=V, n=2, k=0, seed_sub=1600 + V)
    p, q = wl.p, wl.q.copy()
    q[:, rng.permutation(V)[: V // 3]] = np.float32(0.5 / V)          # many equal entries: ties go to the lower id
    q = (q / q.sum(1, keepdims=True, dtype=np.float64)).astype(np.float32)
    ks, ns = [5, 200, 257, top], [1, 3, 7]
    dev = torch.device("cuda:0")
    h = gr.gr_create(B, V, max_k=top)
    try:
        acc, st = gr.gr_accept_sweep(h, torch.from_numpy(p).to(dev), torch.from_numpy(q).to(dev), ks, ns)
        torch.cuda.synchronize()
        acc, st = acc.cpu().numpy(), st.cpu().numpy()
    finally:
        gr.gr_destroy(h)
    assert np.all(st == 0)
    for b in sorted({0, B // 2, B - 1}):
        assert np.abs(acc[b] - G.acceptance_sweep(p[b], q[b], ks, ns)).max() < 1e-5, b
