"""How a batch is launched: RVEs whose panels take more than half of a CU's LDS do not
cost the others their second workgroup per CU, whether they run in one launch (few
others) or in two, and the split changes no result."""
import numpy as np
import pytest

from paper_1908_08292_amd import api, rve, workloads

pytestmark = pytest.mark.gpu

HALF_LDS = 80 * 1024


def _batch(n, seed):
    n = np.asarray(n, np.int32)
    batch, meshes = api.build_batch(2, n, np.full(len(n), 0.27), np.full(len(n), 8.0))
    s = api.Solver(batch, keep_state=False)
    s.set_F(workloads.draw_F(np.random.default_rng(seed), len(n), 2, 0.1))
    return batch, s, meshes


def _done(batch, meshes):
    batch.destroy()
    for m in set(meshes):
        m.destroy()


@pytest.mark.parametrize("n,large", [([16] * 14288 + [33], 1), ([48] * 512 + [40] * 8, 8), ([24] * 1024 + [40] * 256, 256)])
@pytest.mark.parametrize("prec", [0, 1])
def test_many_smaller_rves_keep_two_workgroups_per_cu(n, large, prec):
    print(f"case launches {n[0]} x {len(n) - large} + {n[-1]} x {large} prec={prec}", flush=True)
    batch, s, meshes = _batch(n, 5)
    rows = batch.launches(prec)
    assert rows[:, 0].tolist() == [large, len(n) - large]
    assert rows[0, 1] == large and rows[0, 3] > HALF_LDS
    assert rows[1, 3] <= HALF_LDS and np.all(rows[:, 2] == 256)
    _done(batch, meshes)


def test_few_smaller_rves_share_the_launch():
    for n in ([16] * 3000 + [40], [40] * 300, [8] * 64, [48] * 200 + [40] * 8):
        batch, s, meshes = _batch(n, 6)
        assert batch.launches().shape[0] == 1, n[0]
        _done(batch, meshes)


@pytest.mark.parametrize("prec", [0, 1])
def test_split_batch_gives_what_its_parts_give(prec):
    """Bitwise: the whole batch, eager and replayed from a graph, one launch (static
    workspace) and a subset list in any order, against the parts as batches of their own."""
    import torch
    n = [16] * 2400 + [33, 35, 16] * 100
    o = rve.default_opts(precision=prec)
    print(f"case launches split parts prec={prec}", flush=True)
    batch, s, meshes = _batch(n, 7)
    assert batch.launches(prec)[:, 0].tolist() == [200, 2500]
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        s.solve(opts=o, stream=st.cuda_stream)
    torch.cuda.synchronize()
    whole = [t.clone() for t in (s.P, s.A, s.status, s.iters)]
    assert int((whole[2] != 0).sum()) == 0
    F = s.F.view(-1, 4).cpu().numpy()
    for sel in (np.array(n) == 16, np.array(n) > 16):
        part, meshes2 = api.build_batch(2, np.array(n, np.int32)[sel], np.full(sel.sum(), 0.27), np.full(sel.sum(), 8.0))
        p = api.Solver(part, keep_state=False)
        p.set_F(F[sel])
        p.solve(opts=o)
        torch.cuda.synchronize()
        idx = torch.as_tensor(np.nonzero(sel)[0], device="cuda")
        for got, want, w in ((p.P, whole[0], 4), (p.A, whole[1], 16), (p.status, whole[2], 1), (p.iters, whole[3], 1)):
            assert torch.equal(got.view(-1, w), want.view(-1, w)[idx])
        _done(part, meshes2)

    def clear():
        for t in (s.P, s.A):
            t.fill_(7.0)
        for t in (s.status, s.iters):
            t.fill_(-5)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        s.solve(opts=o, stream=st.cuda_stream)
    for _ in range(3):
        clear()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip((s.P, s.A, s.status, s.iters), whole))
    del g
    clear()
    batch.solve(s.F, s.P, s.A, None, s.status, s.iters, opts=o, static=True)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip((s.P, s.A, s.status, s.iters), whole))
    clear()
    pick = np.random.default_rng(8).permutation(len(n))[:150].astype(np.int32)
    idx = torch.as_tensor(np.concatenate([pick, np.full(50, -1, np.int32)]), device="cuda")
    cnt = torch.tensor([170], dtype=torch.int32, device="cuda")
    batch.solve_subset(idx, cnt, s.F, s.P, s.A, None, s.status, s.iters, opts=o)
    torch.cuda.synchronize()
    hit = torch.zeros(len(n), dtype=torch.bool, device="cuda")
    hit[torch.as_tensor(pick.astype(np.int64), device="cuda")] = True
    for got, want, w, rest in ((s.P, whole[0], 4, 7.0), (s.A, whole[1], 16, 7.0), (s.status, whole[2], 1, -5),
                               (s.iters, whole[3], 1, -5)):
        assert torch.equal(got.view(-1, w)[hit], want.view(-1, w)[hit])
        assert bool((got.view(-1, w)[~hit] == rest).all())
    _done(batch, meshes)


@pytest.mark.parametrize("d,n,threads", [(2, 6, 256), (2, 44, 512), (3, 4, 256), (3, 5, 512)])
def test_autotune_returns_the_workgroup_size_that_ran(d, n, threads):
    import torch
    F = workloads.draw_F(np.random.default_rng(9), 4, d, 0.05)
    mesh = rve.Mesh(d, n, rve.two_phase_lame(8.0), radius=0.27)
    print(f"case autotune {d}d n={n}", flush=True)
    try:
        t = rve.autotune(mesh, torch.tensor(F.reshape(-1), device="cuda"))
        assert t["threads"] == threads
        batch = rve.Batch([mesh] * 4)
        assert batch.launches()[:, 2].tolist() == [threads]
        batch.destroy()
    finally:
        rve.tuning_reset(d, n)
        mesh.destroy()
