"""The Adam step inside the projection backward at every row length and alignment of its 16-byte words, against the oracle's
Adam on the gradient that the kernel formed (bounds as in the test of the sparse step)."""
import numpy as np
import pytest
import torch

from paper_2411_02703_amd import binding as B
from paper_2411_02703_amd import scenes
from paper_2411_02703_amd.step import BatchedStep, GaussianModel

import oracle

pytestmark = pytest.mark.gpu


def _shifted(model, key, shift):
    """The model's arrays `key` start `shift` floats behind a 16-byte boundary."""
    for d in (model.p, model.m, model.v):
        t = d[key]
        new = torch.empty(t.numel() + 4, device="cuda")[shift:shift + t.numel()].view(t.shape)
        d[key] = new.copy_(t)
    model.ps, model.ms, model.vs = (B.params_struct(d, model.sh_degree) for d in (model.p, model.m, model.v))


@pytest.mark.parametrize("shift", [0, 1, 2])
@pytest.mark.parametrize("n,deg", [(1, 0), (65, 0), (257, 1), (191, 2), (321, 2), (255, 3), (66, 3)])
def test_fused_adam_matches_the_oracle_on_every_row(gpu_lib, n, deg, shift):
    sc = scenes.random_scene(5000 + n, n, 64, 48, sh_degree=deg, views=2, log_scale_mu=-1.5, depth_fraction=0.3)
    if n > 8:
        sc.means[: n // 4, 2] = -3.0  # behind every camera
    for sparse in (False, True):
        model = GaussianModel(sc.params(), deg)
        rng = np.random.default_rng(n)
        for k in model.m:
            model.m[k].copy_(torch.as_tensor(rng.normal(0, 1e-3, tuple(model.m[k].shape)).astype(np.float32)))
            model.v[k].copy_(torch.as_tensor(rng.uniform(1e-6, 1e-4, tuple(model.v[k].shape)).astype(np.float32)))
        _shifted(model, "sh", shift)
        model.set_sparse_adam(sparse)
        before = [{k: t.cpu().numpy().copy() for k, t in d.items()} for d in (model.p, model.m, model.v)]
        st = BatchedStep(model, sc.cams, sc.tgt_rgb, sc.tgt_depth, keep_grads=True)
        print("adam", n, deg, shift, sparse, flush=True)
        st.run_eager()
        torch.cuda.synchronize()
        seen = B.frame_tensor(st.frame, "vis_mask", n, torch.int64).cpu().numpy() != 0
        rows = seen if sparse else np.ones(n, bool)
        g = model.g["sh"].cpu().numpy().reshape(n, -1)
        p0, m0, v0 = (d["sh"].reshape(n, -1) for d in before)
        got = [d["sh"].cpu().numpy().reshape(n, -1) for d in (model.p, model.m, model.v)]
        for c in range(g.shape[1]):
            want = oracle.adam(p0[:, c], g[:, c], m0[:, c], v0[:, c], model.adam.lr[4 if c < 3 else 5], step=1)
            for a, b in zip(got, want):
                np.testing.assert_allclose(a[rows, c], np.asarray(b)[rows], rtol=1e-6, atol=1e-7, err_msg=f"{c} {sparse}")
        for a, b in zip(got, (p0, m0, v0)):
            assert np.array_equal(a[~rows], b[~rows])
