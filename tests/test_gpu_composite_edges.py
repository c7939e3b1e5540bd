"""Compositing at the edges of its rounds and lists, against the FP64 oracle.

The backward works on lists of sixteen records a 4x4 block, in rounds of 128 (64 at 8x8 tiles), and the forward on
rounds of one or two records per thread: tile lists around those sizes, views that end inside a block, and Gaussians
that take every branch of a pair (opacities that clamp, needle-thin conics, faint ones that only skip).  The bars are
those of the other parity tests.
"""
import numpy as np
import pytest

from paper_2411_02703_amd import scenes
from test_gpu_parity import check_grads, check_images, grad_reference, run_gpu

import oracle

pytestmark = pytest.mark.gpu


def _scene(n, mixed):
    """n Gaussians that nearly all reach every tile of one 19x11 view."""
    sc = scenes.random_scene(7000 + n, n, 19, 11, sh_degree=1, views=1, log_scale_mu=-0.9, zrange=(3.0, 6.0))
    rng = np.random.default_rng(n)
    if mixed:
        sc.opacity[:] = rng.choice([6.0, 0.5, -3.0], n).astype(np.float32)        # clamped, ordinary, faint
        sc.log_scales[rng.uniform(size=n) < 0.3] = np.array([0.5, -6.0, -6.0], np.float32)  # needles
    else:
        sc.opacity[:] = -3.0                                                       # long lists that do not stop
    return sc


@pytest.mark.parametrize("tile", [(16, 16), (16, 8), (8, 8), (32, 8)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 127, 128, 129, 257])
def test_lists_around_the_round_sizes_match_the_oracle(gpu_lib, n, tile):
    for mixed in (False, True):
        sc = _scene(n, mixed)
        for seg in (-1, 64):
            print("edges", n, tile, mixed, seg, flush=True)
            out = run_gpu(sc, tile=tile, targets=True, fused=True, seg=seg)
            L, ref, exc, _, scale = grad_reference(sc.params(), 1, sc.cams, tgt_rgb=sc.tgt_rgb, tgt_depth=sc.tgt_depth)
            np.testing.assert_allclose(out["loss"], L, rtol=1e-5)
            check_grads(out["grads"], ref, exc, f"n={n} {tile} mixed={mixed} seg={seg}", scale=scale)
            if seg < 0:
                img = oracle.forward(32, sc.params(), 1, sc.cams)
                out["cams"] = sc.cams
                check_images(out, img, img["near"], f"n={n} {tile}")


@pytest.mark.parametrize("size", [(184, 712, 1), (256, 512, 1), (128, 128, 8)])  # 2047, 2048 and 8 x 256 tiles of 8x8
@pytest.mark.parametrize("n", [31, 32, 33, 70])
def test_forward_kernel_of_whole_tiles_by_frame_and_list_size(gpu_lib, n, size):
    w, h, views = size
    sc = scenes.random_scene(7100 + n, n, w, h, sh_degree=1, views=views, log_scale_mu=0.3, zrange=(3.0, 6.0))
    sc.opacity[:] = -2.0
    L, ref, exc, _, scale = grad_reference(sc.params(), 1, sc.cams, tgt_rgb=sc.tgt_rgb, tgt_depth=sc.tgt_depth)
    for seg in (-1, 64):
        print("frame", n, size, seg, flush=True)
        out = run_gpu(sc, tile=(8, 8), targets=True, fused=True, seg=seg)
        np.testing.assert_allclose(out["loss"], L, rtol=1e-5)
        check_grads(out["grads"], ref, exc, f"n={n} {size} seg={seg}", scale=scale)


@pytest.mark.parametrize("sizes", [[(336, 272)], [(341, 275), (16, 17)], [(400, 300), (5, 400), (200, 150)]])
def test_ssim_over_more_tiles_than_blocks(gpu_lib, sizes):
    """1071 tiles and channels and more over at most 1024 blocks, aligned and ragged; bounds as for few tiles (a moment
    is a sum of 121 terms in FP32 either way)."""
    import torch

    from paper_2411_02703_amd import binding as B

    cams = [scenes.identity_camera(0.8 * w, 0.8 * w, w / 2, h / 2, w, h) for w, h in sizes]
    for i, c in enumerate(cams):
        c.weight = 1.0 / (i + 1)
    total = sum(w * h for w, h in sizes)
    rng = np.random.default_rng(total)
    x, y = (rng.uniform(size=3 * total).astype(np.float32) for _ in range(2))
    fr = B.Frame(10, cams)
    g, loss = torch.empty(3 * total, device="cuda"), torch.zeros(64, device="cuda")
    print("ssim", sizes, flush=True)
    B.gs_ssim(fr, torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda(), 0.2, g, loss)
    want, gref = oracle.ssim_loss(x, y, cams, 0.2)
    np.testing.assert_allclose(float(loss[0].item()), want, rtol=1e-5)
    rms = np.sqrt((gref ** 2).mean())
    assert np.all(np.abs(g.cpu().numpy().astype(np.float64) - gref) <= 1e-4 * (np.abs(gref) + rms))
