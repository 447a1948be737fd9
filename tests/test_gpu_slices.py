"""A row's tokens shared among up to 32 workgroups: batches and supports on both sides of every limit on the number of slices,
slices that end inside a tile, rows given as probabilities and as logits."""
import numpy as np
import pytest
import torch

from paper_2511_15898_amd import binding as gr, workloads as W

pytestmark = pytest.mark.gpu


# slices: 32 of 2 tiles, 31 and a ragged last tile, 16 by the support, 8 by the support, one slice (3 tiles), 2 slices of 2 tiles, unaligned rows
@pytest.mark.parametrize("B,V,k", [(1, 65536, 64), (2, 63000, 64), (3, 65600, 65), (3, 70001, 256), (2, 3072, 33), (2, 3073, 33), (2, 40003, 7)])
def test_every_number_of_slices(B, V, k):
    from oracle import gr_oracle as G
    rng = np.random.default_rng(V + k)
    target = 4.0 * rng.gumbel(size=(B, V)); draft = 0.8 * target + rng.normal(size=(B, V))
    target, draft = target.astype(np.float32), draft.astype(np.float32)
    target[0, V - 1] = target[0].max() + 1.0                # the largest target in the last slice: every sum is rescaled to it
    dev = torch.device("cuda:0")
    soft = lambda x: torch.softmax(torch.from_numpy(x).double(), 1).float()
    p, q = soft(target), soft(draft)
    n, ks, ns = 3, [1, max(2, k // 2), k], [1, 3, 8]
    h = gr.gr_create(B, V, max_k=k, max_n=n)
    try:
        acc, st = gr.gr_solve(h, p.to(dev), q.to(dev), n, k, 1e-4)
        temp = torch.ones(B, device=dev)
        acc_lg, st_lg = gr.gr_solve_logits(h, torch.from_numpy(target).to(dev), torch.from_numpy(draft).to(dev), temp, n, k, 1e-4)
        grid, st_grid = gr.gr_accept_sweep(h, p.to(dev), q.to(dev), ks, ns)
        torch.cuda.synchronize()
        acc, acc_lg, grid = acc.cpu().numpy(), acc_lg.cpu().numpy(), grid.cpu().numpy()
        assert st.max() < gr.GR_ROW_BAD and st_lg.max() < gr.GR_ROW_BAD and not st_grid.any()
    finally:
        gr.gr_destroy(h)
    for b in range(B):
        want = G.acceptance_sweep(p[b].numpy(), q[b].numpy(), ks, ns)
        assert np.abs(grid[b] - want).max() < 1e-5
        # alpha* of the solve is the grid's cell of n drafts; from logits it differs by the float32 rounding of p and q (6e-8 each, n of them)
        assert abs(acc[b] - want[2, 1]) < 1e-5 and abs(acc_lg[b] - want[2, 1]) < 1e-5
