"""64-bit sorts around the sizes where their tiles change from 2048 to 4096 and 8192 keys (2^19, 2^20), in a workspace and in
the static scratch, against a stable argsort, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B

pytestmark = pytest.mark.gpu

A, Z = 1 << 19, 1 << 20


@pytest.mark.parametrize("kind", ["equal", "two", "random"])
@pytest.mark.parametrize("n", [A, A + 1, A + 4096, A + 4097, 3 * A // 2 + 5, Z - 4097, Z - 4096, Z - 1, Z, Z + 1, Z + 8193])
def test_sort_around_the_lines_of_the_tile_size(gpu_lib, n, kind):
    rng = np.random.default_rng(n)
    keys = {"equal": lambda: np.full(n, 0x0123456789abcdef, np.uint64),
            "two": lambda: np.where(rng.uniform(size=n) < 0.01, np.uint64(1) << np.uint64(63), np.uint64(255)),
            "random": lambda: rng.integers(0, 1 << 64, n, dtype=np.uint64)}[kind]()
    for bits in (64, 16):
        part = keys if bits == 64 else keys & np.uint64(0xffff)
        want = np.argsort(part, kind="stable")
        for sort in (B.gs_sort_pairs,) + ((B.gs_sort_pairs_static,) if n <= Z else ()):
            kt = torch.as_tensor(keys.view(np.int64)).cuda()
            vt = torch.arange(n, dtype=torch.int32, device="cuda")
            print("sort", n, kind, bits, sort.__name__, flush=True)
            sort(kt, vt, bits)
            assert np.array_equal(vt.cpu().numpy(), want)
            assert np.array_equal(kt.cpu().numpy().view(np.uint64), keys[want])
