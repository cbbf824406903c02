"""2D meshes at both ends of what lives in LDS, against the oracle (P to 1e-8 and A to 1e-6
relative, equal Newton counts in FP64): fronts in global memory (periodic, 44 x 44 on) in
workgroups of eight waves and, beside a mesh whose panels are in LDS, of four; and panels
in LDS of the largest meshes under linear displacements (up to 64 x 64)."""
import numpy as np
import pytest

import oracle
from paper_1908_08292_amd import api, rve, workloads

pytestmark = pytest.mark.gpu


def _solve(n, bc, prec, threads, panels, flags=0):
    """The batch of sizes n, its path checked, against the oracle on every RVE."""
    import torch
    B = len(n)
    wl = workloads.rve2d(B, seed=4700 + n[0])
    batch, meshes = api.build_batch(2, n, wl.radius, wl.ratio, bc=bc)
    assert batch.launches(prec)[:, :3].tolist() == [[B, panels, threads]]
    s = api.Solver(batch)
    s.set_F(wl.F)
    print(f"case 2d n={n} bc={bc} prec={prec} threads={threads} flags={flags}", flush=True)
    s.solve(opts=rve.default_opts(precision=prec, flags=flags))
    torch.cuda.synchronize()
    out = s.results()
    w, off = s.w.cpu().numpy(), batch.state_offsets
    batch.destroy()
    for m in set(meshes):
        m.destroy()
    for b in range(B):
        with oracle.bc(bc):
            ref = oracle.rve_solve(2, int(n[b]), oracle.phase_by_centroid(2, int(n[b]), wl.radius[b]),
                                   oracle.two_phase_lame(wl.ratio[b]), wl.F[b])
        assert out["status"][b] == ref["status"] == 0, (b, n[b])
        if prec == rve.PREC_FP64:
            assert out["iters"][b] == ref["iters"], (b, n[b])
        else:
            assert abs(int(out["iters"][b]) - ref["iters"]) <= 1, (b, n[b])
        eP = np.linalg.norm(out["P"][b] - ref["P"]) / np.linalg.norm(ref["P"])
        eA = np.linalg.norm(out["A"][b] - ref["A"]) / np.linalg.norm(ref["A"])
        print(f"  n={n[b]} P {eP:.1e} A {eA:.1e}", flush=True)
        assert eP <= 1e-8 and eA <= 1e-6, (b, n[b], eP, eA)
        assert np.all(np.isfinite(w[off[b]:off[b + 1]]))


@pytest.mark.parametrize("prec", [rve.PREC_FP64, rve.PREC_FP32_IR])
@pytest.mark.parametrize("flags", [0, rve.FLAG_DIRECT_TANGENT])
def test_global_fronts_eight_waves(prec, flags):
    _solve([44, 45, 48], 0, prec, 512, 0, flags)


@pytest.mark.parametrize("prec", [rve.PREC_FP64, rve.PREC_FP32_IR])
@pytest.mark.parametrize("flags", [0, rve.FLAG_DIRECT_TANGENT])
def test_global_fronts_four_waves_beside_panels(prec, flags):
    _solve([44, 45, 48, 7, 33, 43], 0, prec, 256, 3, flags)


@pytest.mark.parametrize("prec", [rve.PREC_FP64, rve.PREC_FP32_IR])
def test_largest_panels_under_linear_displacements(prec):
    _solve([47, 56, 64], 1, prec, 256, 3)
