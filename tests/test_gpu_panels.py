"""2D plans whose front panels live in LDS, over the sizes where their pieces change:
single fronts, every panel width modulo the 16-column block and the 8-column product
step, wave fronts only with all update matrices in LDS (n <= 8 or so), subtrees fused
per wave, workgroup fronts alone, and both tails of the size range; both couplings and
precisions, mixed in one batch, against the oracle (FP64: P to 1e-8 and A to 1e-6
relative with equal Newton counts, as everywhere in the parity tests)."""
import numpy as np
import pytest

import oracle
from paper_1908_08292_amd import api, rve, workloads

pytestmark = pytest.mark.gpu

SIZES = (2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 13, 15, 16, 17, 20, 23, 27, 31, 32, 37, 43)


@pytest.mark.parametrize("bc", [0, 1])
@pytest.mark.parametrize("prec", [0, 1])
def test_mixed_sizes_match_the_oracle(bc, prec):
    torch = pytest.importorskip("torch")
    n = np.array([k for k in SIZES if not (bc == 1 and k == 2)] * 3, np.int32)
    B = len(n)
    F = workloads.draw_F(np.random.default_rng(77 + bc), B, 2, 0.12)
    r = np.random.default_rng(78).uniform(0.15, 0.35, B)
    batch, meshes = api.build_batch(2, n, r, np.full(B, 10.0), bc=bc)
    s = api.Solver(batch)
    s.set_F(F)
    print(f"case mixed sizes bc={bc} prec={prec}", flush=True)
    s.solve(opts=rve.default_opts(precision=prec))
    torch.cuda.synchronize()
    out = s.results()
    with oracle.bc(bc):
        for b in range(0, B):
            if b >= len(SIZES) and n[b] > 20:
                continue  # the large ones once
            ref = oracle.rve_solve(2, int(n[b]), oracle.phase_by_centroid(2, int(n[b]), r[b]),
                                   oracle.two_phase_lame(10.0), F[b])
            assert out["status"][b] == 0 and ref["status"] == 0, (b, n[b])
            eP = np.linalg.norm(out["P"][b] - ref["P"]) / np.linalg.norm(ref["P"])
            eA = np.linalg.norm(out["A"][b] - ref["A"]) / np.linalg.norm(ref["A"])
            assert eP < 1e-8 and eA < 1e-6, (b, n[b], eP, eA)
            if prec == 0:
                assert out["iters"][b] == ref["iters"], (b, n[b])
    batch.destroy()
    for m in set(meshes):
        m.destroy()
