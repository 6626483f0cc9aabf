"""kd-trees over given vectors (written over a blob's own) against the oracle,
bit for bit: one point, sizes at and beside a whole subtree of 2,048, leaves
so small that a subtree has more segments than are reduced at once, ties in
every dimension, and spreads at and above what a 32-bit sort key holds."""
import numpy as np
import pytest

from oracle import ffo

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,C,leaf,top", [
    (1, 1, 3, 8, 50), (5, 1, 1, 2, 50), (64, 32, 3, 8, 1 << 20), (64, 32, 3, 2, (1 << 20) + 1), (45, 45, 1, 2, 1 << 26),
    (41, 50, 3, 2, 3), (49, 42, 3, 2, 1000), (128, 96, 3, 2, 40000), (128, 96, 1, 64, 2), (97, 61, 3, 3, 1),
])
def test_kdtree_of_given_vectors(W, H, C, leaf, top):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_05151_amd import ff
    print("kdtree vectors", W, H, C, leaf, top, flush=True)
    rho, N = 3, W * H
    rng = np.random.default_rng(W * H + leaf)
    V = rng.integers(-top, top, (N, 9 * C), endpoint=top > 1).astype(np.int32)   # top 1: only -1 and 0
    V[0, 0], V[N - 1, 0] = -top, top - 1   # the widest spread in every tree
    d = ff.ff_desc_init(W, H, C, 0, 4, (rho,))
    blob = torch.zeros(d.bytes, dtype=torch.uint8, device="cuda")
    rows = ff.blob_views(d, blob)["wht"][rho].view(N, -1)
    rows[:, :9 * C] = torch.from_numpy(V).cuda()
    nn = ff.ff_tree_nodes(N, leaf)
    nd, ns = (torch.empty(nn, dtype=torch.int32, device="cuda") for _ in range(2))
    perm = torch.empty(N, dtype=torch.int32, device="cuda")
    prm = ff.ff_default_params(k=0, leaf=leaf)
    ws = torch.empty(ff.ff_match_workspace_bytes(d, d, rho, prm), dtype=torch.uint8, device="cuda")
    ff.ff_build_kdtree(d, blob, rho, leaf, nd, ns, perm, ws)
    torch.cuda.synchronize()
    rnd, rns, rperm = ffo.kdtree_build(V, leaf)
    assert np.array_equal(nd.cpu().numpy(), rnd)
    assert np.array_equal(ns.cpu().numpy()[rnd >= 0], rns[rnd >= 0])
    assert np.array_equal(perm.cpu().numpy(), rperm)
