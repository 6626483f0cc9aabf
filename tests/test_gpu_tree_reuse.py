"""A kd-tree left in the workspace by ff_match_field_tree seeds a later call of
another depth and another number of sweeps and searches as the call's own tree
does: the tree's place depends on neither."""
import sys

import numpy as np
import pytest

from synth import pairs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("built,used", [
    (dict(k=3, n_prop=4, n_rs=3), dict(k=2, n_prop=1, n_rs=1)),
    (dict(k=0, n_prop=0, n_rs=0), dict(k=3, n_prop=4, n_rs=3)),
    (dict(k=1, n_prop=3, n_rs=0), dict(k=3, n_prop=20, n_rs=2)),
])
def test_tree_of_another_schedule(built, used):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_05151_amd import ff
    print("tree reuse", built, used, flush=True)
    sys.stdout.flush()
    W, H, r = 97, 71, 8
    p = pairs.layered_pair(seed=900, W=W, H=H, nlayers=2)
    d = ff.ff_desc_init(W, H, 3, 3, 4, (r,))
    blobs = []
    for img in (p.img1, p.img2):
        b = torch.empty(d.bytes, dtype=torch.uint8, device="cuda")
        ff.ff_compute_descriptors(d, torch.from_numpy(np.ascontiguousarray(img)).cuda(), b)
        blobs.append(b)
    size = max(ff.ff_match_workspace_bytes(d, d, r, ff.ff_default_params(**kw)) for kw in (built, used))

    def match(ws, **kw):
        F = torch.empty((H, W), dtype=torch.int32, device="cuda")
        C = torch.empty_like(F)
        ff.ff_match_field(d, blobs[0], d, blobs[1], r, ff.ff_default_params(seed=3, **used, **kw), None, F, C, ws)
        torch.cuda.synchronize()
        assert ff.ff_read_status(ws) == 0
        return F.cpu().numpy(), C.cpu().numpy()

    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    ref = match(ws)
    ws = torch.full((size,), 0xA5, dtype=torch.uint8, device="cuda")
    ff.ff_match_field_tree(d, blobs[0], d, blobs[1], r, ff.ff_default_params(**built), ws)
    for _ in range(2):   # the tree outlives the call that used it
        got = match(ws, use_kdtree=2)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])


@pytest.mark.parametrize("src,dst", [((97, 71), (97, 71)), ((97, 71), (70, 51)), ((97, 71), (40, 33)), ((131, 90), (9, 5))])
def test_source_larger_than_target(src, dst):
    """The second grid buffer inside the tree's scratch, partly past its end and
    almost wholly past it: against the oracle, with the call's own tree, with one
    left by ff_match_field_tree (used twice), and without a workspace."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import ffo
    from paper_1508_05151_amd import ff
    print("source larger", src, dst, flush=True)
    sys.stdout.flush()
    r, k = 6, 2
    p = pairs.layered_pair(seed=901, W=src[0], H=src[1], nlayers=2)
    img2 = np.ascontiguousarray(p.img2[:dst[1], :dst[0]])
    d, blobs = [], []
    for img in (p.img1, img2):
        e = ff.ff_desc_init(img.shape[1], img.shape[0], 3, k, 4, (r,))
        b = torch.empty(e.bytes, dtype=torch.uint8, device="cuda")
        ff.ff_compute_descriptors(e, torch.from_numpy(np.ascontiguousarray(img)).cuda(), b)
        d.append(e)
        blobs.append(b)
    oF, oC = ffo.match_field(ffo.Desc(p.img1, k, 4, (r,)), ffo.Desc(img2, k, 4, (r,)), r, k=k, seed=3)
    F = torch.empty((src[1], src[0]), dtype=torch.int32, device="cuda")
    C = torch.empty_like(F)
    prm = ff.ff_default_params(k=k, seed=3)

    def same():
        torch.cuda.synchronize()
        return np.array_equal(F.cpu().numpy(), oF) and np.array_equal(C.cpu().numpy(), oC)

    ws = torch.full((ff.ff_match_workspace_bytes(d[0], d[1], r, prm),), 0xA5, dtype=torch.uint8, device="cuda")
    ff.ff_match_field(d[0], blobs[0], d[1], blobs[1], r, prm, None, F, C, ws)
    assert same() and ff.ff_read_status(ws) == 0
    ws.fill_(0xA5)
    ff.ff_match_field_tree(d[0], blobs[0], d[1], blobs[1], r, prm, ws)
    for _ in range(2):
        ff.ff_match_field(d[0], blobs[0], d[1], blobs[1], r, ff.ff_default_params(k=k, seed=3, use_kdtree=2), None, F, C, ws)
        assert same() and ff.ff_read_status(ws) == 0
    ff.ff_match_field_noalloc(d[0], blobs[0], d[1], blobs[1], r, prm, None, F, C)
    assert same()
