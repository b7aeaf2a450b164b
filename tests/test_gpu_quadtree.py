"""Image quadtree by contrast on the GPU (Eq. 10, Algorithm 1) against the oracle: the same leaves
(sorted), contrast within FP32 rounding, on images of several sizes (odd, thin, and the 640x480 and
1200x680 frame sizes of the paper's RGB-D data) at several thresholds and minimum sizes."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mrh():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2511_21459_amd as mrh

    return mrh


def _image(rng, h, w, patch=8, noise=25.0):
    smooth = rng.integers(0, 256, (h // patch + 2, w // patch + 2, 3)).repeat(patch, 0).repeat(patch, 1)[:h, :w]
    return np.clip(smooth + rng.normal(0, noise, (h, w, 3)), 0, 255).astype(np.uint8)


CASES = [(37, 53, 300.0, 3, 8), (64, 48, 800.0, 2, 4), (100, 7, 50.0, 1, 8), (480, 640, 400.0, 4, 16),
         (680, 1200, 250.0, 8, 32), (480, 640, 1e9, 4, 16), (480, 640, 0.0, 1, 16)]


def test_quadtree_matches_oracle(mrh):
    rng = np.random.default_rng(1)
    qt = mrh.Quadtree(1200, 680)
    for h, w, thr, mn, patch in CASES:
        announce(f"quadtree {w}x{h} threshold {thr} min {mn}")
        img = _image(rng, h, w, patch)
        want, wc, near = oracle.quadtree(img, thr, mn)
        assert near == 0
        leaves, con = qt.build(torch.from_numpy(img).cuda(), thr, mn)
        got = leaves.cpu().numpy()
        gc = con.cpu().numpy().astype(np.float64)
        go, oo = np.lexsort(got.T[::-1]), np.lexsort(want.T[::-1])
        assert np.array_equal(got[go], want[oo]), (w, h, thr, len(got), len(want))
        assert np.allclose(gc[go], wc[oo], rtol=1e-5, atol=1e-3)
        print(w, h, thr, mn, "leaves", len(got))
    qt.close()


def test_quadtree_small_buffer(mrh):
    import ctypes

    announce("quadtree buffer too small")
    img = torch.from_numpy(_image(np.random.default_rng(2), 64, 64)).cuda()
    qt = mrh.Quadtree(64, 64)
    leaves, _ = qt.build(img, 100.0, 2)
    L = mrh._lib.load()
    buf = torch.empty((2, 4), dtype=torch.int32, device="cuda")
    n = ctypes.c_int64()
    st = L.mrh_quadtree_build(qt._h, ctypes.c_void_p(img.data_ptr()), 64, 64, 100.0, 2, ctypes.c_void_p(buf.data_ptr()),
                              None, 2, ctypes.byref(n))
    assert st == -5 and n.value == leaves.shape[0] > 2
    assert L.mrh_quadtree_build(qt._h, ctypes.c_void_p(img.data_ptr()), 65, 64, 100.0, 2, None, None, 0, ctypes.byref(n)) == -1
    assert L.mrh_quadtree_build(qt._h, ctypes.c_void_p(img.data_ptr()), 64, 64, 100.0, 0, None, None, 0, ctypes.byref(n)) == -1
    qt.close()


# (height, width, min size): sides of 40 and 41, subtree roots at every depth (0 .. 8) and without
# pixels, and both sides of the line beyond which tables of the whole image are used
SUBTREES = [(1, 1, 1), (1, 8, 1), (40, 40, 1), (41, 40, 1), (5, 40, 1), (80, 81, 1), (161, 33, 2), (321, 319, 1), (10, 640, 1),
            (640, 1, 1), (81, 641, 1), (80, 641, 1), (641, 200, 3), (170, 1300, 2), (2600, 330, 5), (700, 5200, 9)]


@pytest.mark.parametrize("h,w,mn", SUBTREES)
def test_quadtree_subtrees(mrh, h, w, mn):
    announce(f"quadtree subtrees {w}x{h}")
    img = _image(np.random.default_rng(h * 7919 + w), h, w, 8 if h * w < 100000 else 64, 12.0)
    qt = mrh.Quadtree(w, h)
    dev = torch.from_numpy(img).cuda()
    for thr in (0.0, 200.0) if h * w < 300000 else (300.0,):
        want, wc, near = oracle.quadtree(img, thr, mn)
        assert near == 0
        leaves, con = qt.build(dev, thr, mn)
        got, gc = leaves.cpu().numpy(), con.cpu().numpy()
        go, oo = np.lexsort(got.T[::-1]), np.lexsort(want.T[::-1])
        assert np.array_equal(got[go], want[oo]), (thr, len(got), len(want))
        # the contrast is an FP64 quotient of exact sums, rounded once to FP32
        assert np.allclose(gc[go], wc[oo], rtol=1e-6, atol=1e-6)
    qt.close()


# (height, width, min size): on both sides of the line between the two forms where subtree roots lie at depth
# 7 (2.5 million pixels), either side the longer, and beyond depth 7
@pytest.mark.parametrize("h,w,mn", [(977, 2561, 6), (976, 2561, 6), (2561, 977, 6), (650, 5120, 6), (1000, 5121, 9)])
def test_quadtree_large_images(mrh, h, w, mn):
    announce(f"quadtree large {w}x{h}")
    img = _image(np.random.default_rng(h + w), h, w, 64, 12.0)
    qt = mrh.Quadtree(w, h)
    want, wc, near = oracle.quadtree(img, 300.0, mn)
    assert near == 0
    leaves, con = qt.build(torch.from_numpy(img).cuda(), 300.0, mn)
    got, gc = leaves.cpu().numpy(), con.cpu().numpy()
    go, oo = np.lexsort(got.T[::-1]), np.lexsort(want.T[::-1])
    assert np.array_equal(got[go], want[oo]), (len(got), len(want))
    assert np.allclose(gc[go], wc[oo], rtol=1e-6, atol=1e-6)
    qt.close()


@pytest.mark.parametrize("h,w", [(40, 40), (640, 640), (97, 203)])
def test_quadtree_extreme_values(mrh, h, w):
    """Channels of 0 and 255 only, the largest sums that a subtree holds."""
    announce(f"quadtree of 0 and 255, {w}x{h}")
    rng = np.random.default_rng(w)
    for img in (np.full((h, w, 3), 255, np.uint8), np.where(rng.random((h, w, 3)) < 0.97, 255, 0).astype(np.uint8)):
        qt = mrh.Quadtree(w, h)
        want, wc, near = oracle.quadtree(img, 10.0, 1)
        assert near == 0
        leaves, con = qt.build(torch.from_numpy(img).cuda(), 10.0, 1)
        got, gc = leaves.cpu().numpy(), con.cpu().numpy()
        go, oo = np.lexsort(got.T[::-1]), np.lexsort(want.T[::-1])
        assert np.array_equal(got[go], want[oo])
        assert np.allclose(gc[go], wc[oo], rtol=1e-6, atol=1e-6)
        qt.close()
