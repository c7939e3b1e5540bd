"""Map maintenance at the edges of its blocks, searches and key ranges: rows move bit for bit, new ones match the oracle."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes

import oracle

pytestmark = pytest.mark.gpu
SHAPES = dict(means=(3,), log_scales=(3,), quats=(4,), opacity=(), sh=None)


def _set(n, deg, shift, rng=None):
    """One parameter set whose arrays start `shift` floats behind a 16-byte boundary."""
    out = {}
    for k, s in SHAPES.items():
        s = ((deg + 1) ** 2, 3) if s is None else s
        size = n * int(np.prod(s, dtype=np.int64))
        t = torch.full((size + 4,), -7.0, device="cuda")[shift:shift + size]
        if rng is not None:
            t.copy_(torch.as_tensor(rng.standard_normal(size).astype(np.float32)))
        out[k] = t.view(n, *s)
    return out


@pytest.mark.parametrize("shift_in,shift_out", [(0, 0), (1, 0), (0, 2), (3, 3)])
@pytest.mark.parametrize("n,deg", [(1, 3), (255, 0), (256, 3), (257, 2), (511, 1), (140_001, 0), (5000, 3),
                                   (16_383, 0), (16_384, 1), (16_385, 2)])
def test_pruned_and_reordered_rows_move_bit_for_bit(gpu_lib, n, deg, shift_in, shift_out):
    rng = np.random.default_rng(n + deg)
    sets = [_set(n, deg, shift_in, rng) for _ in range(3)]
    outs = [_set(n, deg, shift_out) for _ in range(3)]
    ins = [B.params_struct(d, deg) for d in sets]
    to = [B.params_struct(d, deg) for d in outs]
    perm = torch.empty(n, dtype=torch.int32, device="cuda")
    print("order", n, deg, shift_in, shift_out, flush=True)
    B.gs_spatial_order(*ins, *to, perm)
    want = oracle.spatial_order(sets[0]["means"].cpu().numpy())
    assert np.array_equal(perm.cpu().numpy(), want)
    idx = torch.as_tensor(want.astype(np.int64)).cuda()
    for a, b in zip(sets, outs):
        for k in a:
            assert torch.equal(b[k], a[k][idx]), k
    n_kept = torch.zeros(1, dtype=torch.int64, device="cuda")
    for tau in (0.5, 0.05, 0.999):
        print("prune", n, deg, shift_in, shift_out, tau, flush=True)
        kept = oracle.prune(sets[0]["opacity"].cpu().numpy(), tau)
        for d in outs:
            for t in d.values():
                t.fill_(-7.0)
        B.gs_prune(*ins, tau, *to, n_kept)
        assert int(n_kept.item()) == kept.size
        idx = torch.as_tensor(kept.astype(np.int64)).cuda()
        for a, b in zip(sets, outs):
            for k in a:
                assert torch.equal(b[k][: kept.size], a[k][idx]), k
                assert bool((b[k][kept.size:] == -7.0).all()), k


@pytest.mark.parametrize("n_map,n_pts,cap,kind", [(0, 1, 1, "scan"), (1, 3, 1, "scan"), (70, 17, 2, "scan"),
                                                  (3000, 1023, 1, "crowd"), (3000, 1025, 3, "crowd"),
                                                  (257, 2049, 2, "copies"), (500, 4100, 1, "scan"),
                                                  (200, 600, 5, "edge"), (100, 300, 40, "far")])
def test_expansion_counts_and_neighbours_match_the_oracle(gpu_lib, n_map, n_pts, cap, kind):
    """Voxels crowded by the map or by copies of a point, key stretches of one and more keys, cells at the ends of the
    key range and neighbours in later rings or beyond them; log-scales within FP32 rounding (1e-5 on a log)."""
    rng = np.random.default_rng(n_map + n_pts)
    pts = rng.uniform(-2, 2, (n_pts, 3))
    mm = rng.uniform(-2, 2, (n_map, 3))
    voxel, cell = 0.1, 0.2
    if kind == "crowd":
        mm[: n_map * 2 // 3] = 0.55 + rng.uniform(0, 0.02, (n_map * 2 // 3, 3))
        pts[::3] = 0.5 + rng.uniform(0, 0.3, pts[::3].shape)
    elif kind == "copies":
        pts[:] = pts[rng.integers(0, 40, n_pts)]
    elif kind == "edge":  # the key range ends at 104.8576 with this cell
        cell = 1e-4
        pts = 104.8574 + rng.uniform(0, 6e-4, (n_pts, 3))
        pts[::2, 1:] *= -1
    elif kind == "far":
        cell = 0.01
        pts = pts * 0.05 + rng.integers(0, 2, (n_pts, 1)) * 30.0
    pts, mm = pts.astype(np.float32), mm.astype(np.float32)
    rgb = rng.uniform(0, 1, (n_pts, 3)).astype(np.float32)
    cam = scenes.random_scene(1, 1, 32, 24, views=1).cams[0]
    vis = np.zeros((24, 32), np.float32)
    kept, ref = oracle.expand(pts, rgb, cam, vis, 0.5, mm, voxel=voxel, cap=cap, init_opacity=0.1, sh_degree=1)
    sets = [_set(n_map + n_pts, 1, 0) for _ in range(3)]
    sets[0]["means"][:n_map] = torch.as_tensor(mm).cuda()
    n_added = torch.zeros(1, dtype=torch.int64, device="cuda")
    print("expand", n_map, n_pts, cap, kind, flush=True)
    B.gs_expand(*[B.params_struct(d, 1) for d in sets], n_map, torch.as_tensor(pts).cuda(), torch.as_tensor(rgb).cuda(),
                cam, torch.as_tensor(vis.reshape(-1)).cuda(), B.gs_expand_opts(0.5, 0.2, voxel, cell, 0.1, cap), n_added)
    a = int(kept.sum())
    assert int(n_added.item()) == a
    got = {k: t[n_map:n_map + a].cpu().numpy() for k, t in sets[0].items()}
    assert np.array_equal(got["means"], pts[kept])
    np.testing.assert_allclose(got["log_scales"], ref["log_scales"], rtol=0, atol=1e-5)
    assert np.array_equal(got["quats"], ref["quats"].astype(np.float32))
    np.testing.assert_allclose(got["opacity"], ref["opacity"], rtol=1e-6)
    np.testing.assert_allclose(got["sh"], ref["sh"], rtol=1e-6, atol=1e-7)
    for d in sets[1:]:
        for k, t in d.items():
            assert not bool(t[n_map:n_map + a].any()) and bool((t[:n_map] == -7.0).all()), k
    for d in sets:
        for k, t in d.items():
            assert bool((t[n_map + a:] == -7.0).all()), k
