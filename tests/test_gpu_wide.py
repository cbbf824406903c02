"""Global-front plans under both workgroup sizes: eight waves (3D, and 2D batches of up
to 256 RVEs) and four (larger 2D batches, and 3D batches mixed with meshes whose panels
fit LDS) give the same P and A to 1e-9 relative, with equal status and Newton counts."""
import numpy as np
import pytest

from paper_1908_08292_amd import api, rve, workloads

pytestmark = pytest.mark.gpu


def _solve(d, n, r, q, F, prec):
    import torch
    batch, meshes = api.build_batch(d, n, r, q)
    s = api.Solver(batch, keep_state=False)
    s.set_F(F)
    s.solve(opts=rve.default_opts(precision=prec))
    torch.cuda.synchronize()
    out = s.results()
    batch.destroy()
    for m in set(meshes):
        m.destroy()
    return out


@pytest.mark.parametrize("d,sizes,extra", [(2, (44, 45), 250), (3, (5, 6, 7), 1)])
@pytest.mark.parametrize("prec", [0, 1])
def test_eight_and_four_waves_agree(d, sizes, extra, prec):
    B = 9
    n = np.resize(np.array(sizes, np.int32), B)
    F = workloads.draw_F(np.random.default_rng(61 + d), B, d, 0.08)
    r, q = np.full(B, 0.3), np.full(B, 10.0)
    print(f"case wide {d}d {sizes} prec={prec}", flush=True)
    wide = _solve(d, n, r, q, F, prec)
    # 2D: past 256 RVEs; 3D: beside an RVE of 3^3 (panels in LDS)
    n2 = np.concatenate([n, np.full(extra, sizes[0] if d == 2 else 3, np.int32)])
    pad = lambda x: np.concatenate([x, np.repeat(x[:1], extra, axis=0)])
    four = _solve(d, n2, pad(r), pad(q), pad(F), prec)
    assert np.all(wide["status"] == 0) and np.all(four["status"] == 0)
    if prec == 0:
        assert np.array_equal(wide["iters"], four["iters"][:B])
    for k in ("P", "A"):
        for b in range(B):
            e = np.linalg.norm(wide[k][b] - four[k][b]) / np.linalg.norm(four[k][b])
            assert e < 1e-9, (k, b, e)
