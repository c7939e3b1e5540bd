"""Map expansion by as many points as a grid of one dimension has no threads for."""
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes

pytestmark = pytest.mark.gpu

KEYS = {"means": 3, "log_scales": 3, "quats": 4, "opacity": 1, "sh": 3}


def _expand(points, colours, cam, vis):
    """Rows of an empty map of degree 0 after gs_expand."""
    n = points.shape[0]
    sets = []
    for _ in range(3):
        d = {k: torch.empty((n, w) if w > 1 else (n,), device="cuda") for k, w in KEYS.items()}
        d["sh"] = d["sh"].view(n, 1, 3)
        sets.append(d)
    added = torch.zeros(1, dtype=torch.int64, device="cuda")
    opts = B.gs_expand_opts(0.5, 0.2, 0.05, 0.4, 0.1, 1)
    B.gs_expand(*[B.params_struct(d, 0) for d in sets], 0, points, colours, cam, vis, opts, added)
    torch.cuda.synchronize()
    a = int(added.item())
    return a, {k: v[:a].clone() for k, v in sets[0].items()}


def test_2_to_the_28_points(gpu_lib):
    """All but the last 3000 points lie where the map already explains the image and are left out: the result is that of
    the 3000 alone, bit for bit."""
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("needs 90 GiB of free device memory")
    M, some = 1 << 28, 3000
    cam = scenes.identity_camera(40.0, 40.0, 32.0, 24.0, 64, 48)
    vis = torch.zeros(64 * 48, device="cuda")
    vis[24 * 64 + 32] = 1.0
    g = torch.Generator(device="cuda").manual_seed(3)
    pts = torch.zeros((M, 3), device="cuda")
    pts[:, 2] = 5.0  # the pixel (32, 24)
    pts[-some:] = torch.rand((some, 3), generator=g, device="cuda") * 3.0 + torch.tensor([0.5, -1.5, 3.0], device="cuda")
    rgb = torch.full((M, 3), 0.25, device="cuda")
    print("expand", M, flush=True)
    want_n, want = _expand(pts[-some:].contiguous(), rgb[-some:].contiguous(), cam, vis)
    n, got = _expand(pts, rgb, cam, vis)
    assert n == want_n and 1000 < n <= some
    for k in KEYS:
        assert torch.equal(got[k], want[k]), k
    del pts, rgb
    torch.cuda.empty_cache()
