"""The radix sort around its tile sizes, its changes of kernel (8192 keys) and of tile size (2^19 keys) and with keys that
load its digits unevenly, against a stable argsort, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["equal", "descending", "two", "random"])
@pytest.mark.parametrize("n", [1, 63, 1024, 1025, 2047, 2048, 2049, 4097, 8192, 8193, (1 << 19) - 1, 1 << 19, (1 << 19) + 1, 65 * 8192,
                               65 * 8192 + 1])
def test_sort_around_the_tile_sizes_is_a_stable_sort(gpu_lib, n, kind):
    rng = np.random.default_rng(n)
    keys = {"equal": lambda: np.full(n, 0xffffffffffffffff, np.uint64),
            "descending": lambda: np.arange(n, 0, -1, dtype=np.uint64) << np.uint64(13),
            "two": lambda: np.where(rng.uniform(size=n) < 0.01, np.uint64(1) << np.uint64(63), np.uint64(255)),
            "random": lambda: rng.integers(0, 1 << 64, n, dtype=np.uint64)}[kind]()
    order = np.argsort(keys, kind="stable")
    for bits in (64, 17):
        kt = torch.as_tensor(keys.view(np.int64)).cuda()
        vt = torch.arange(n, dtype=torch.int32, device="cuda")
        print("sort", n, kind, bits, flush=True)
        B.gs_sort_pairs(kt, vt, bits)
        want = order if bits == 64 else np.argsort(keys & np.uint64((1 << 24) - 1), kind="stable")
        assert np.array_equal(vt.cpu().numpy(), want)
        assert np.array_equal(kt.cpu().numpy().view(np.uint64), keys[want])
