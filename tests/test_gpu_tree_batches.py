"""A level of a walk is one batch of rows picked from the tree, each with its own draft count: counts on both sides of the
solve kernels' degrees, rows that no vector load can take, and supports that still go by count."""
import numpy as np
import pytest

from paper_2511_15898_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,L,V,k", [(9, 3, 515, 24), (5, 4, 1022, 40), (16, 2, 400, 12), (3, 3, 701, 300)])
def test_walks_with_mixed_draft_counts(K, L, V, k):
    from oracle import tree_walk as TW
    from test_gpu_tree_walk import _walk_gpu
    S = 8
    p, q, paths, u = W.draft_tree(S=S, K=K, L=L, V=V, k=k, seed_sub=700 + K)
    for a in range(K):                                     # one row per level for all paths, tokens among its largest: long walks with several drafts
        p[:, a], q[:, a] = p[:, 0], q[:, 0]
        for l in range(L):
            paths[:, a, l] = q[:, 0, l].argsort(axis=1)[:, -1 - (a + l) % 3]
    tokens, length, accepted, fallbacks = _walk_gpu(p, q, paths, u, k, 1e-5)
    compared = 0
    for s in range(S):
        out, nacc, fb, edge = TW.tree_walk([[p[s, a, l] for l in range(L)] for a in range(K)],
                                           [[q[s, a, l] for l in range(L)] for a in range(K)], paths[s], u[s], k, 1e-5, max_T=128)
        if edge < 1e-5:
            continue
        compared += 1
        assert list(tokens[s, :length[s]]) == out and accepted[s] == nacc and fallbacks[s] == fb, (s, tokens[s], out)
    assert compared >= S - 2


@pytest.mark.parametrize("S,K,L,V,k", [(90, 4, 4, 300, 24), (257, 2, 3, 261, 12), (40, 16, 3, 300, 16), (70, 4, 3, 300, 24), (60, 7, 3, 301, 20)])
def test_walks_of_several_levels_to_a_batch(S, K, L, V, k):
    """Trees on both sides of what one batch takes (512 nodes, 256 of a later level), some in batches of more rows than the handle has and than
    the chip has compute units (390 nodes of 3 or 4 paths at most, of 5 to 7 too): the same walks taken node by node, every step a tree of one level with the
    paths that are left.  A token may differ where the uniform falls on an edge of the distribution."""
    import torch
    from paper_2511_15898_amd import binding as gr
    rng = np.random.default_rng(S)
    first = rng.integers(0, 2, (S, K, L))                   # every path one of two at each level: nodes of several paths at all levels
    seed = np.zeros((S, K, L), np.int64)
    for l in range(1, L):
        seed[:, :, l] = seed[:, :, l - 1] * 2 + first[:, :, l - 1] + 1
    noise = rng.gumbel(size=(S, 1 << L, V)) * 4.0
    draft = 0.8 * noise + rng.standard_normal(noise.shape)
    soft = lambda x: (lambda e: e / e.sum(-1, keepdims=True))(np.exp(x - x.max(-1, keepdims=True)))
    at = np.arange(S)[:, None, None], seed
    p, q = soft(noise)[at].astype(np.float32), soft(draft)[at].astype(np.float32)
    paths = np.argsort(-q, axis=-1)[..., :2]
    paths = np.take_along_axis(paths, first[..., None], -1)[..., 0].astype(np.int32)
    u = rng.random((S, L)).astype(np.float32)
    dev = torch.device("cuda:0")
    P, Q = torch.from_numpy(p).to(dev), torch.from_numpy(q).to(dev)
    h = gr.gr_create(S, V, max_k=k, max_n=K)
    try:
        tokens, length, accepted, fallbacks = gr.gr_tree_walk(h, P, Q, paths, u, k, 1e-4)
        differ = 0
        for s in range(0, S, 3):
            active, out, nacc = list(range(K)), [], 0
            for l in range(L):
                rows = [P[s, active, l][None, :, None], Q[s, active, l][None, :, None]]
                t, n, a, _ = gr.gr_tree_walk(h, rows[0].contiguous(), rows[1].contiguous(), paths[s, active, l][None, :, None], u[s, l].reshape(1, 1), k, 1e-4)
                out.append(int(t[0, 0])); nacc += int(a[0])
                if not a[0]:
                    break
                active = [x for x in active if paths[s, x, l] == t[0, 0]]
            differ += list(tokens[s, :length[s]]) != out or accepted[s] != nacc
            assert np.all(tokens[s, length[s]:] == -1) and length[s] - accepted[s] in (0, 1)
        assert differ <= 1, differ
    finally:
        gr.gr_destroy(h)
