"""The backward at its own edges: the stop rule at every transmittance of a list, and image gradients that are not finite."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes
from paper_2411_02703_amd.step import GaussianModel

pytestmark = pytest.mark.gpu


def _frame(model, cams, **opts):
    fr = B.Frame(model.n, cams, B.default_opts(**opts))
    B.gs_project(model.ps, fr)
    n = B.gs_bin_tiles(fr, sync_count=True)
    assert n <= fr.capacity
    return fr


def _stack(n, seed):
    """n Gaussians one behind the other, all centred on the pixel (9, 6) of a 19x11 view: there every alpha is the opacity."""
    rng = np.random.default_rng(seed)
    cam = scenes.identity_camera(16.0, 16.0, 9.5, 6.5, 19, 11)
    p = dict(means=np.zeros((n, 3), np.float32), log_scales=np.full((n, 3), -1.0, np.float32),
             quats=scenes.random_quats(rng, n), opacity=rng.uniform(-4.5, -2.2, n).astype(np.float32),
             sh=rng.uniform(0.2, 1.0, (n, 1, 3)).astype(np.float32))
    p["means"][:, 2] = np.linspace(3.0, 6.0, n)
    return p, [cam]


@pytest.mark.parametrize("tile", [(16, 16), (8, 8)])
@pytest.mark.parametrize("n", [16, 150])
def test_the_backward_stops_at_the_forwards_pair(gpu_lib, n, tile):
    """t_min at the transmittance behind each record and one ulp above it: the record counts, or ends the pixel.  The
    products are formed in list order in FP32, as the forward forms them, so the expected last record is exact."""
    params, cams = _stack(n, n)
    model = GaussianModel(params, 0)
    o = B.frame_tensor(_frame(model, cams, tile_w=tile[0], tile_h=tile[1]), "rec", n * 12, torch.float32).view(n, 12)[:, 3]
    o = o.cpu().numpy()
    T = np.cumprod((np.float32(1) - o).astype(np.float32), dtype=np.float32)  # left to right
    pick = range(n) if n <= 16 else [0, 14, 15, 16, 30, 31, 32, 47, 62, 63, 64, 65, 79, 95, 100, 111, 126, 127, 128, 129, 144, 149]
    px = 6 * 19 + 9
    for k in pick:
        for t_min, count in ((T[k], k + 1), (np.nextafter(T[k], np.float32(1)), k)):
            print("stop", n, tile, k, count, flush=True)
            fr = _frame(model, cams, tile_w=tile[0], tile_h=tile[1], t_min=float(t_min), seg_len=-1)
            rgb, depth, vis = fr.empty_images()
            B.gs_render_fwd(fr, rgb, depth, vis)
            w, t = np.float32(0), np.float32(1)
            for j in range(count):
                w, t = w + o[j] * t, t * (np.float32(1) - o[j])
            assert vis[px].item() == w  # the forward composites `count` records
            g = torch.zeros_like(rgb)
            g[px::19 * 11] = 1.0
            for fwd in (None, (rgb, depth, vis)):
                model.zero_grad()
                B.gs_render_bwd(model.ps, fr, fwd, model.gs, g_rgb=g, g_depth=torch.zeros_like(depth),
                                g_vis=torch.zeros_like(vis))
                hit = (model.g["sh"].view(n, -1) != 0).all(dim=1).cpu().numpy()
                assert hit[:count].all() and not hit[count:].any(), (k, count, np.flatnonzero(hit))


@pytest.mark.parametrize("field", ["g_rgb", "g_depth", "g_vis"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf"), 3e38])
@pytest.mark.parametrize("tile,seg", [((16, 16), -1), ((8, 8), -1), ((16, 8), 64)])
def test_a_gradient_that_is_not_finite_reaches_the_contributing_records_only(gpu_lib, tile, seg, value, field):
    """Records whose pixels all have ordinary gradients get the gradient that they get with 0 at the other pixels (up to
    the order of the float sums), whatever stands there."""
    n, w, h = 400, 40, 24
    rng = np.random.default_rng(5)
    sc = scenes.random_scene(77, n, w, h, log_scale_mu=-2.4, zrange=(3.0, 6.0))
    sc.sh[:] = rng.uniform(0.2, 1.0, sc.sh.shape)  # (no clamped colour)
    sc.opacity[: n // 8] = 6.0  # clamped alphas, which take the other form of the walk
    model = GaussianModel(sc.params(), 0)
    fr = _frame(model, sc.cams, tile_w=tile[0], tile_h=tile[1], seg_len=seg)
    img = fr.empty_images()
    B.gs_render_fwd(fr, *img)

    def grads(fwd, **g):
        model.zero_grad()
        B.gs_render_bwd(model.ps, fr, fwd, model.gs, **g)
        return {k: v.view(n, -1).cpu().numpy().astype(np.float64) for k, v in model.g.items()}

    bad = [5 * w + 7, 17 * w + 30, 23 * w + 39]
    base = dict(g_rgb=torch.randn(3 * w * h, device="cuda"), g_depth=torch.randn(w * h, device="cuda"),
                g_vis=torch.randn(w * h, device="cuda"))
    zero = {k: torch.zeros_like(v) for k, v in base.items()}
    one = zero["g_rgb"].clone()
    for c in range(3):
        for p in bad:
            one[c * w * h + p] = 1.0
    touched = (grads(img, **dict(zero, g_rgb=one))["sh"] != 0).any(axis=1)
    assert 0 < touched.sum() < n // 2
    clean = {k: v.clone() for k, v in base.items()}
    for k, v in clean.items():
        for p in bad:
            v.view(-1, w * h)[:, p] = 0.0
    dirty = {k: v.clone() for k, v in clean.items()}
    for p in bad:
        dirty[field].view(-1, w * h)[:, p] = value
    for fwd in (img, None):
        print("not finite", tile, seg, value, field, fwd is None, flush=True)
        want, got = grads(fwd, **clean), grads(fwd, **dirty)
        for k in want:
            a, b = want[k][~touched], got[k][~touched]
            rms = np.sqrt((want[k] ** 2).mean())
            assert np.isfinite(b).all(), (k, int((~np.isfinite(b)).any(axis=1).sum()))
            assert np.abs(a - b).max() <= 1e-4 * rms, k
        if not np.isfinite(value):
            reached = np.any([~np.isfinite(got[k]).all(axis=1) for k in got], axis=0)
            assert reached[touched & (sc.opacity < 4.0)].all()
