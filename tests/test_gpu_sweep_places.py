"""Batches whose sweeps have more tiles than the chip has places for their
workgroups, at radii with an instance of their own and at others, and the same
fields one by one (a third as many workgroups, other visits and revisits, the
instance without the second radius): the same bytes; at one radius against the
oracle."""
import sys

import numpy as np
import pytest

from oracle import ffo
from synth import pairs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("radii,n,oracle", [((5,), 6, True), ((8, 6), 8, False), ((8, 5), 10, False)])
def test_more_tiles_than_places(radii, n, oracle):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_05151_amd import ff
    print("sweep places", radii, n, flush=True)
    sys.stdout.flush()
    W, H, k = 320, 240, 1
    tiles = ((W + 30) // 16) * (H // 16) * n   # of the finest level
    assert tiles > 2048 if radii == (8, 6) else tiles // len(radii) > 1280
    p = pairs.layered_pair(seed=910, W=W, H=H, nlayers=3)
    d = ff.ff_desc_init(W, H, 3, k, 4, radii)
    b1, b2 = (torch.empty(d.bytes, dtype=torch.uint8, device="cuda") for _ in range(2))
    ff.ff_compute_descriptors(d, torch.from_numpy(np.ascontiguousarray(p.img1)).cuda(), b1)
    ff.ff_compute_descriptors(d, torch.from_numpy(np.ascontiguousarray(p.img2)).cuda(), b2)
    prm = ff.ff_default_params(k=k)
    out = [(torch.empty((H, W), dtype=torch.int32, device="cuda"), torch.empty((H, W), dtype=torch.int32, device="cuda"))
           for _ in range(n)]
    jobs = [ff.make_job(d, b1, d, b2, radii[i % len(radii)], F, C, 1, i, 31, k=k) for i, (F, C) in enumerate(out)]
    ws = torch.full((ff.ff_match_batch_workspace_bytes(jobs, prm),), 0xA5, dtype=torch.uint8, device="cuda")
    ff.ff_match_batch(jobs, prm, ws)
    torch.cuda.synchronize()
    assert ff.ff_read_status(ws) == 0
    for i, (F, C) in enumerate(out):
        r = radii[i % len(radii)]
        one = ff.ff_default_params(k=k, field_id=1, pair_id=i, seed=31)
        w1 = torch.full((ff.ff_match_workspace_bytes(d, d, r, one),), 0xA5, dtype=torch.uint8, device="cuda")
        F1, C1 = torch.empty_like(F), torch.empty_like(C)
        ff.ff_match_field(d, b1, d, b2, r, one, None, F1, C1, w1)
        torch.cuda.synchronize()
        assert ff.ff_read_status(w1) == 0
        assert torch.equal(F, F1) and torch.equal(C, C1), i
    if oracle:
        oF, oC = ffo.match_field(ffo.Desc(p.img1, k, 4, radii), ffo.Desc(p.img2, k, 4, radii), radii[0], seed=31, field_id=1,
                                 pair_id=n - 1, k=k)
        assert np.array_equal(out[-1][0].cpu().numpy(), oF) and np.array_equal(out[-1][1].cpu().numpy(), oC)
