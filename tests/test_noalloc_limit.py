"""What ff_match_field_noalloc accepts fits its static array: its size limit
(checked before the pointers, so null ones tell accepted from refused) against
ff_match_workspace_bytes, for sources as large as the target and much larger,
trees of few and many nodes, and the most sweeps a call can have."""
import ctypes as C

import pytest

# the array: FF_NOALLOC_SCRATCH_BYTES and 2 KB for each of 5 levels x 64 sweeps
WORDS = 5 * 64 * 2048


@pytest.fixture(scope="module")
def ff():
    from paper_1508_05151_amd import ff
    return ff


def _accepted(ff, src, dst, p):
    rc = ff.lib().ff_match_field_noalloc(C.byref(src), None, C.byref(dst), None, 8, C.byref(p), None, None, None, None,
                                         None)
    assert rc in (-1, -2)
    return rc == -1


@pytest.mark.parametrize("leaf,k,n_prop,use_kdtree", [(8, 3, 4, 1), (2, 4, 64, 1), (3, 0, 1, 1), (64, 4, 64, 1), (8, 4, 4, 0)])
def test_accepted_fits(ff, leaf, k, n_prop, use_kdtree):
    p = ff.ff_default_params(leaf=leaf, k=k, n_prop=n_prop, n_rs=min(3, n_prop), use_kdtree=use_kdtree)
    seen = set()
    for W, H in [(2048, 2048), (8191, 512), (6313, 485), (1600, 1000), (1280, 720), (8191, 128)]:
        src = ff.ff_desc_init(W, H, 1, k, 1, (8,))
        for w in (1, 37, 200, 500, 700, 800, 900, 1000, 1100, 1156, 1200, 1300, 1400, 1700, 2048):
            dst = ff.ff_desc_init(w, w, 1, k, 1, (8,))
            ok = _accepted(ff, src, dst, p)
            seen.add(ok)
            if ok:
                assert ff.ff_match_workspace_bytes(src, dst, 8, p) <= ff.NOALLOC_SCRATCH_BYTES + WORDS, (W, H, w)
    assert seen == ({True, False} if use_kdtree else {True})


def test_common_sizes_are_accepted(ff):
    p = ff.ff_default_params()
    for W, H in [(1024, 436), (1242, 375), (1280, 720), (1600, 1000)]:
        d = ff.ff_desc_init(W, H, 3, 3, 4, (8,))
        assert _accepted(ff, d, d, p), (W, H)
    d = ff.ff_desc_init(1920, 1080, 3, 3, 4, (8,))
    assert not _accepted(ff, d, d, p)
