"""A level of a walk is one batch of rows picked from the tree, each with its own draft count: counts on both sides of the
solve kernels' degrees, rows that no vector load can take, and supports that still go by count."""
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
