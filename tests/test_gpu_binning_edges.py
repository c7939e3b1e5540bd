"""Binning around the sizes of its running sums (blocks of 256 items, groups of 64 blocks) and with records of every width,
bit for bit from the GPU's own records, twice from one projection."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes
from paper_2411_02703_amd.step import GaussianModel
from test_gpu_parity import gpu_records

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,views,tile,mu,size", [(1, 1, (8, 8), 0.5, (64, 48)), (255, 2, (16, 16), -2.0, (96, 72)),
                                                  (257, 6, (16, 8), -2.0, (96, 72)),
                                                  (16_384, 1, (16, 16), -2.5, (96, 72)),
                                                  (16_385, 5, (32, 8), -2.5, (96, 72)),
                                                  (700, 2, (8, 8), 0.5, (512, 384)),      # hundreds of tiles a record
                                                  (3000, 1, (8, 8), -1.6, (512, 384)),    # around 32 tiles a record
                                                  (70_000, 3, (16, 16), -3.0, (160, 120))])
def test_binning_is_bit_exact_from_gpu_records(gpu_lib, n, views, tile, mu, size):
    sc = scenes.random_scene(4000 + n, n, *size, sh_degree=0, views=views, log_scale_mu=mu)
    model = GaussianModel(sc.params(), 0)
    capacity = 8192 if n < 256 else 6_000_000  # (the sorts of a small capacity run in one block)
    fr = B.Frame(model.n, sc.cams, B.default_opts(tile_w=tile[0], tile_h=tile[1]), capacity)
    print("bin", n, views, tile, flush=True)
    B.gs_project(model.ps, fr)
    for sync in (False, True):
        B.gs_bin_tiles(fr, sync_count=sync)
        total, flags = B.gs_read_counters(fr)
        rec, rect, vis = gpu_records(fr, n, views)
        rk, rv, lo, hi = oracle.bin_records(rect, np.ascontiguousarray(rec[:, 2]).view(np.uint32), vis.astype(np.int32),
                                            n, sc.cams, *tile)
        assert flags == 0 and total == len(rk)
        keys, vals = B.sorted_pairs(fr, total)
        assert np.array_equal(keys.cpu().numpy().view(np.uint32), (rk >> np.uint64(32)).astype(np.uint32))
        assert np.array_equal(vals.cpu().numpy().astype(np.int64), rv)
        r4 = rect.astype(np.int64)
        area = np.where(vis, (r4[:, 1] - r4[:, 0] + 1) * (r4[:, 3] - r4[:, 2] + 1), 0)
        per = area.reshape(views, n).sum(0)
        first = B.frame_tensor(fr, "inst_first", n, torch.int32).cpu().numpy()
        assert np.array_equal(first, np.cumsum(per) - per)
