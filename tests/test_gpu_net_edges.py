"""The proposal network's kernels at the sizes where a tile or a piece ends: one
pixel per row, rows one pixel over and under 16 and 32 outputs, odd inputs
(a last row or column without its neighbour at stride 2), rows of several
whole pieces, and images that do not start on a word.  Forward output and
gradient against the float64 oracle, with every ReLU clearly active, so that
the bound is two bf16 ulps of each element's magnitude (2^-6)."""
import numpy as np
import pytest

from oracle import ffo
from oracle import net_oracle as N
from test_gpu_net import Q, _batch, _clear_labels, _dev, _say, _theta_active

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _unaligned(a):
    """The same bytes on the device, starting one byte off a word."""
    flat = torch.empty(a.size + 1, dtype=torch.uint8, device="cuda")
    flat[1:] = torch.from_numpy(np.ascontiguousarray(a)).cuda().reshape(-1)
    return flat[1:].view(a.shape)


@pytest.mark.parametrize("B,W,H,aligned", [
    (1, 8, 8, True), (3, 9, 17, True), (1, 130, 33, True), (1, 126, 31, False), (2, 264, 24, True), (1, 1030, 16, True),
    (2, 61, 40, False),
])
def test_forward_and_gradient_at_tile_edges(B, W, H, aligned):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1508_05151_amd import ff
    _say("net edges", B, W, H, aligned)
    i1, i2, _ = _batch(130, B, W, H)
    x = N.input_tensor(i1, i2)
    th = _theta_active(7, x)
    th64 = th.astype(np.float64)
    out, acts = N.forward(th64, x, keep=True)
    lab, lab_px = _clear_labels(np.random.default_rng(W + H), out)
    lab[0, 0, 0], lab_px[0, 0, 0] = ffo.pack(np.array(640), np.array(-640)), (640 / Q, -640 / Q)   # at least one label
    put = _dev if aligned else _unaligned
    g1, g2 = put(i1), put(i2)
    net = ff.ProposalNet(th, subpel=Q)
    flow = torch.empty(out.shape, dtype=torch.float32, device="cuda")
    prop = net.forward(g1, g2, flow_out=flow)
    loss, g = net.gradient(g1, g2, _dev(lab))
    torch.cuda.synchronize()
    got = flow.cpu().numpy().astype(np.float64)
    assert (np.abs(got - out) <= 2.0 ** -6 * N.forward_magnitude(th64, acts)).all()
    assert np.array_equal(prop.cpu().numpy(), N.proposal_q(got, Q))
    rloss, gout = N.masked_l1(out, lab_px)
    rg, mag = N.backward(th64, acts, gout, magnitude=True)
    assert abs(float(loss.item()) - rloss) <= 1e-4 * max(rloss, 1.0)
    g = g.cpu().numpy().astype(np.float64)
    assert (np.abs(g - rg) <= 2.0 ** -6 * mag + 1e-30).all(), float((np.abs(g - rg) / np.maximum(mag, 1e-30)).max())
