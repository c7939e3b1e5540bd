"""Who runs the forward of the backward's whole tiles, by frame size (2047 and 2048 tiles) and list length (0, 1, 7, 8 and
more records): the kernel of the segments' sums, which hands the upstream gradient over, or the backward's own.  In loss mode
and with image gradients, with work items a workgroup and taken from a counter, against the FP64 oracle.  The frame's memory
is filled with NaN first, so that a state slot or a loss word that nobody writes shows."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes
from paper_2411_02703_amd.step import GaussianModel
from test_gpu_parity import check_grads, grad_reference

pytestmark = pytest.mark.gpu


def _scene(n, w, h, empty):
    """n Gaussians that cover the first view, and a second view of `empty` pixels a side that sees none."""
    sc = scenes.random_scene(7300 + n, n, w, h, sh_degree=1, views=1, fx=200.0, log_scale_mu=1.8, log_scale_sigma=0.1,
                              zrange=(3.0, 6.0))
    sc.means[:, :2] *= 0.1
    sc.opacity[:] = -2.0
    away = scenes.Camera(np.eye(3), np.array([0.0, 0.0, -100.0]), 40.0, 40.0, empty / 2, empty / 2, empty, empty, 0.5)
    sc.cams = [sc.cams[0], away]
    sc.cams[0].weight = 0.5
    sc.tgt_rgb, sc.tgt_depth = scenes.uniform_targets(7400 + n, sc.cams, (3.0, 6.0), 0.5)
    return sc


def _run(sc, lens, seg, persistent, images):
    model = GaussianModel(sc.params(), sc.sh_degree)
    fr = B.Frame(model.n, sc.cams, B.default_opts(tile_w=8, tile_h=8, seg_len=seg, persistent=persistent), int(lens.sum()) + 64)
    fr.block.fill_(255)
    B.gs_project(model.ps, fr)
    assert B.gs_bin_tiles(fr, sync_count=True) == lens.sum()
    rng = B.frame_tensor(fr, "tile_range", 2 * fr.f.n_tiles, torch.int32).view(-1, 2).cpu().numpy()
    assert np.array_equal(rng[:, 1] - rng[:, 0], lens)
    out = {}
    if images is None:
        B.gs_render_bwd(model.ps, fr, None, model.gs, tgt_rgb=torch.as_tensor(sc.tgt_rgb).cuda(),
                        tgt_depth=torch.as_tensor(sc.tgt_depth).cuda())
        out["loss"] = float(B.frame_tensor(fr, "loss", 1, torch.float32).item())
    else:
        g = [torch.as_tensor(a).cuda() for a in images]
        B.gs_render_bwd(model.ps, fr, None, model.gs, g_rgb=g[0], g_depth=g[1], g_vis=g[2])
    out["grads"] = {k: v.cpu().numpy() for k, v in model.g.items()}
    return out


@pytest.mark.parametrize("size", [(264, 496, 8), (184, 712, 8), (256, 512, 24)])  # 2046 + 1, 2047 + 1 and 2048 + 9 tiles
@pytest.mark.parametrize("n", [1, 7, 8, 9, 33, 70])
def test_whole_tiles_by_frame_and_list_size(gpu_lib, n, size):
    w, h, empty = size
    sc = _scene(n, w, h, empty)
    lens = np.concatenate([np.full((w // 8) * (h // 8), n), np.zeros((empty // 8) ** 2, int)])
    P = sc.total_pixels
    rng = np.random.default_rng(n)
    images = tuple(rng.normal(size=m * P).astype(np.float32) for m in (3, 1, 1))
    for g in (None, images):
        kw = dict(tgt_rgb=sc.tgt_rgb, tgt_depth=sc.tgt_depth) if g is None else dict(g_rgb=g[0], g_depth=g[1], g_vis=g[2])
        L, ref, exc, _, scale = grad_reference(sc.params(), 1, sc.cams, **kw)
        for seg, persistent in ((-1, 0), (64, 0), (64, 1)):
            print("whole", n, size, seg, persistent, g is None, flush=True)
            out = _run(sc, lens, seg, persistent, g)
            if g is None:
                np.testing.assert_allclose(out["loss"], L, rtol=1e-5)
            check_grads(out["grads"], ref, exc, f"n={n} {size} seg={seg} persistent={persistent} loss={g is None}", scale=scale)
