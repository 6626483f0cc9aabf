"""The PCA of the SIFT colours against NumPy in float64 on the same vectors:
the eigen-decomposition (tridiagonal form, correction step, and the Jacobi
solver for covariances whose eigenvalues coincide) and the projection, at row
counts off the kernels' steps and at channel counts around their tile of 16.

Bounds, from the arithmetic: the covariance's entries are sums of products
below 1 with a relative rounding of n eps / sqrt(n) at most 1e-13 for the n
here; eigenvalues move by at most the matrix' change (Weyl) and the solvers'
own 128 eps, so 1e-12 of the largest; the basis is orthonormal to the same.
A code may differ by one where 1024 (d - mean) . basis lies within 1e-7 of a
half (the sum of 128 terms below 1024, rounded to 53 bits, is within 1e-10)."""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _texture(w, h, seed):
    g = np.random.default_rng(seed).standard_normal((h, w))
    ky, kx = np.fft.fftfreq(h)[:, None] * h, np.fft.rfftfreq(w)[None, :] * w
    t = np.fft.irfft2(np.fft.rfft2(g) / np.maximum(np.hypot(kx, ky), 1.0), s=(h, w))
    t = (t - t.min()) / max(float(t.max() - t.min()), 1e-9)
    return np.round(255 * t).astype(np.uint8)


def _pca(L1, L2, S):
    from paper_1508_05151_amd import ff
    (h1, w1), (h2, w2) = L1.shape, L2.shape
    c1 = torch.empty((h1, w1, S), dtype=torch.int16, device="cuda")
    c2 = torch.empty((h2, w2, S), dtype=torch.int16, device="cuda")
    d1 = torch.empty((h1, w1, 128), dtype=torch.float32, device="cuda")
    d2 = torch.empty((h2, w2, 128), dtype=torch.float32, device="cuda")
    pca = torch.empty(2 * 128 + 128 * 128, dtype=torch.float64, device="cuda")
    ws = torch.full((ff.ff_sift_workspace_bytes(w1, h1, w2, h2),), 0xFF, dtype=torch.uint8, device="cuda")
    ff.ff_sift_colors(torch.from_numpy(L1).cuda(), torch.from_numpy(L2).cuda(), S, c1, c2, ws, pca=pca, desc1=d1,
                      desc2=d2)
    torch.cuda.synchronize()
    p = pca.cpu().numpy()
    v = np.concatenate([d.cpu().numpy().reshape(-1, 128) for d in (d1, d2)]).astype(np.float64)
    codes = np.concatenate([c.cpu().numpy().reshape(-1, S) for c in (c1, c2)])
    return v, p[:128], p[128:256], p[256:].reshape(128, 128), codes


@pytest.mark.parametrize("w1,h1,w2,h2,S", [(64, 40, 64, 40, 18), (61, 37, 50, 43, 16), (33, 17, 33, 19, 17),
                                          (97, 31, 20, 90, 32), (250, 131, 249, 130, 1)])
def test_pca_and_codes(w1, h1, w2, h2, S):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("pca", w1, h1, w2, h2, S, flush=True)
    sys.stdout.flush()
    v, mean, ev, U, codes = _pca(_texture(w1, h1, w1 + S), _texture(w2, h2, h2 + S), S)
    m = v.mean(0)
    C = v.T @ v / len(v) - np.outer(m, m)
    want = np.linalg.eigvalsh(C)[::-1]
    assert np.abs(mean - m).max() <= 1e-13
    assert np.abs(ev - want).max() <= 1e-12 * want[0]
    assert np.abs(U.T @ U - np.eye(128)).max() <= 1e-12
    assert np.abs(U.T @ C @ U - np.diag(ev)).max() <= 1e-12 * want[0]
    assert np.all(U[np.abs(U).argmax(0), np.arange(128)] > 0)
    x = 1024.0 * ((v - mean) @ U[:, :S])
    off = np.abs(codes - np.clip(np.rint(x), -2047, 2047))
    near_half = np.abs(x - np.floor(x) - 0.5) < 1e-7
    assert np.all((off == 0) | ((off == 1) & near_half))


def test_pca_of_degenerate_covariances():
    """No vectors but zero, and fewer distinct vectors than dimensions: the
    eigenvalues, and a basis that spans the vectors, from the Jacobi solver."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("pca degenerate", flush=True)
    flat = np.full((21, 34), 90, np.uint8)
    v, mean, ev, U, codes = _pca(flat, flat, 5)
    assert not v.any() and not ev.any() and not codes.any()
    step = np.repeat((np.arange(40) >= 20).astype(np.uint8) * 120 + 40, 1)[None, :].repeat(24, 0)
    v, mean, ev, U, codes = _pca(np.ascontiguousarray(step), flat, 12)
    m = v.mean(0)
    C = v.T @ v / len(v) - np.outer(m, m)
    want = np.maximum(np.linalg.eigvalsh(C)[::-1], 0)
    assert np.abs(ev - want).max() <= 1e-12 * want[0]
    r = int((want > 1e-9 * want[0]).sum())
    assert 0 < r < 128
    assert np.abs(U[:, :r].T @ U[:, :r] - np.eye(r)).max() <= 1e-10
    assert np.abs((v - m) - (v - m) @ U[:, :r] @ U[:, :r].T).max() <= 1e-3
