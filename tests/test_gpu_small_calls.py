"""The tilings the library picks for small single calls (every tile of a launch
resident at once): each entry of its list is reached by one grid size, ragged
against the tile, with one shot or several, both tops, equal and unequal grid
spacings.  Gathers and snapshots equal those of 128 x 64
tiles at time block 4 bit for bit (the same update expression); gradients
equal the FP64 oracle's to relative L2 <= 1e-4, the bar of every propagation
test, and those of 128 x 64 tiles at time block 3 bit for bit.  A tuning the caller sets is never replaced."""
import numpy as np
import pytest

import oracle
from paper_2605_30541_amd import sgwave
from paper_2605_30541_amd.sgwave import Geometry, Plan, Shots
from test_gpu_gradient import _og, gpu_gradient, rel_l2
from test_gpu_sweep import run

pytestmark = pytest.mark.gpu

EXPLICIT = dict(variant=2, tile_x=128, tile_z=64, time_block=4)


# padded cells nz + 2 nbl (free top: nz + nbl) by nx + 2 nbl, over 256 CUs
@pytest.mark.parametrize("nz,nx,nbl,nshot", [
    (5, 3, 0, 1), (8, 9, 0, 2), (64, 128, 20, 1), (65, 129, 20, 2), (81, 107, 9, 3), (131, 257, 17, 1),
    (200, 300, 40, 1), (301, 501, 40, 1), (361, 563, 40, 1), (441, 719, 40, 1), (521, 901, 40, 1),
    (300, 500, 40, 3)])
@pytest.mark.parametrize("top", [sgwave.SG_TOP_FREE, sgwave.SG_TOP_ABSORBING], ids=["free", "absorbing"])
@pytest.mark.parametrize("dz", [10.0, 8.0], ids=["square", "unequal"])
def test_small_forward_equals_wide_tiles(nz, nx, nbl, nshot, top, dz):
    rng = np.random.default_rng(nz + nx)
    nt = 85                                     # 84 steps: not a multiple of 5 or of 8
    g = Geometry(nz=nz, nx=nx, dz=dz, dx=10.0, dt=8e-4, nt=nt, nbl=nbl, top=top, vmax_hint=3000.0,
                 snap_every=23, snap_count=3)
    v = rng.uniform(1800.0, 3000.0, (nz, nx)).astype(np.float32)
    at = lambda n: np.stack([rng.uniform(0, (nz - 1) * dz, n), rng.uniform(0, (nx - 1) * 10.0, n)], 1)
    src, rec = at(nshot), np.concatenate([at(40), [[0.0, 0.0], [(nz - 1) * dz, (nx - 1) * 10.0]]])
    wl = np.stack([oracle.ricker(35.0 + k, g.dt, nt, t0=0.012) for k in range(nshot)])
    a = run(g, v, src, rec, wl, {})
    b = run(g, v, src, rec, wl, EXPLICIT)
    for k in range(2):
        assert np.any(b[k] != 0)
        assert np.array_equal(a[k], b[k])


# the list's entries in turn; then a call too large for any of them
@pytest.mark.parametrize("nz,nx,nbl,nshot,top", [
    (5, 7, 0, 1, sgwave.SG_TOP_FREE), (40, 51, 11, 3, sgwave.SG_TOP_ABSORBING),
    (64, 128, 20, 2, sgwave.SG_TOP_FREE), (200, 300, 40, 1, sgwave.SG_TOP_FREE),
    (301, 501, 40, 1, sgwave.SG_TOP_ABSORBING), (361, 563, 40, 1, sgwave.SG_TOP_FREE),
    (441, 719, 40, 1, sgwave.SG_TOP_FREE), (521, 901, 40, 1, sgwave.SG_TOP_FREE),
    (300, 500, 40, 4, sgwave.SG_TOP_FREE)])
def test_small_gradient_matches_oracle(nz, nx, nbl, nshot, top):
    rng = np.random.default_rng(nz * 1000 + nx)
    nt, hi = 60, np.array([(nz - 1) * 10.0, (nx - 1) * 10.0])
    g = Geometry(nz=nz, nx=nx, dz=10.0, dx=10.0, dt=1e-3, nt=nt, nbl=nbl, top=top, vmax_hint=3000.0)
    v = rng.uniform(1800.0, 3000.0, (nz, nx)).astype(np.float32)
    src = rng.uniform(0, 1, (nshot, 2)) * hi
    near = np.repeat(src, 3, 0) + rng.uniform(-60, 60, (3 * nshot, 2))   # within reach of the 59 levels
    rec = np.clip(near, 0, hi)
    wl = oracle.ricker(40.0, g.dt, nt, t0=0.012)
    resid = rng.standard_normal((nshot, g.nrow, len(rec))).astype(np.float32)
    ref = oracle.gradient(_og(g), v.astype(np.float64), src, wl, rec, resid.astype(np.float64))
    d_ref, _ = oracle.forward(_og(g), v.astype(np.float64), src, wl, rec)
    got, gathers = gpu_gradient(g, v, src, rec, wl, resid, ckpt=13)
    assert np.linalg.norm(d_ref[:, -1]) > 0 and np.linalg.norm(ref) > 0
    assert rel_l2(gathers, d_ref) <= 1e-4
    assert rel_l2(got, ref) <= 1e-4
    # the partial imaging sums cover the same levels whatever the tiling
    for tuning in (dict(variant=2, tile_x=128, tile_z=64, time_block=3), dict(variant=3, tile_x=128, time_block=3)):
        same, _ = gpu_gradient(g, v, src, rec, wl, resid, ckpt=13, tuning=tuning)
        assert np.array_equal(got, same)


def test_set_tunings_stand():
    """The launches the plan counts are those of the time block it was given."""
    import torch
    g = Geometry(nz=64, nx=128, dz=10.0, dx=10.0, dt=1e-3, nt=41, nbl=20, vmax_hint=3000.0)
    v = torch.full((64, 128), 2000.0, device="cuda")
    wl = torch.from_numpy(oracle.ricker(30.0, g.dt, g.nt).astype(np.float32)).cuda()
    got = {}
    for tb in (0, 1, 2, 4, 5, 6):
        plan = Plan(g)
        if tb:
            plan.set_tuning(variant=2, time_block=tb)
        plan.set_profiling(True)
        sgwave.forward(plan, v, Shots([[10.0, 400.0]], [[10.0, 640.0]], wl[None]))
        torch.cuda.synchronize()
        got[tb] = plan.profile()[1]
    assert got == {0: 6, 1: 40, 2: 20, 4: 10, 5: 8, 6: 7}


@pytest.mark.parametrize("nrec", [1, 62, 66, 900])
@pytest.mark.parametrize("tuning", [None, dict(variant=2, tile_x=128, tile_z=64, time_block=3)],
                         ids=["default", "wide"])
def test_gradient_with_few_and_many_nodes_per_tile(nrec, tuning):
    """Receiver nodes per tile on both sides of what the adjoint sums up before
    its first level (256), repeated positions among them."""
    rng = np.random.default_rng(nrec)
    nz, nx, nt = 40, 60, 50
    g = Geometry(nz=nz, nx=nx, dz=10.0, dx=10.0, dt=1e-3, nt=nt, nbl=8, vmax_hint=3000.0)
    v = rng.uniform(1800.0, 3000.0, (nz, nx)).astype(np.float32)
    src = np.array([[200.0, 300.0], [120.0, 250.0]])
    rec = np.stack([rng.uniform(0, (nz - 1) * 10.0, nrec), rng.uniform(0, (nx - 1) * 10.0, nrec)], 1)
    rec[nrec // 2:nrec // 2 + 2] = rec[0]
    wl = oracle.ricker(40.0, g.dt, nt, t0=0.012)
    resid = rng.standard_normal((2, g.nrow, nrec)).astype(np.float32)
    ref = oracle.gradient(_og(g), v.astype(np.float64), src, wl, rec, resid.astype(np.float64))
    got, _ = gpu_gradient(g, v, src, rec, wl, resid, ckpt=12, tuning=tuning)
    assert np.linalg.norm(ref) > 0
    assert rel_l2(got, ref) <= 1e-4


@pytest.mark.parametrize("nz,nx,nshot", [(64, 128, 1), (30, 40, 2), (200, 300, 1), (620, 1001, 4)])
def test_autotuned_calls_are_no_slower_than_the_default(nz, nx, nshot):
    """The autotuner also times the tiling that the default takes for a small
    call; when that is the fastest it reports all zeros, which set the default.
    Gathers stay the same bit for bit."""
    import torch
    g = Geometry(nz=nz, nx=nx, dz=10.0, dx=10.0, dt=1e-3, nt=241, nbl=20, vmax_hint=3000.0)
    v = torch.full((nz, nx), 2500.0, device="cuda")
    wl = torch.from_numpy(oracle.ricker(30.0, g.dt, g.nt).astype(np.float32)).cuda()
    shots = Shots(np.full((nshot, 2), 100.0), np.stack([np.full(nx, 10.0), np.arange(nx) * 10.0], 1), wl[None])
    plan = Plan(g)
    ws = torch.empty(sgwave.sg_forward_workspace_size(plan, nshot, nx), dtype=torch.uint8, device="cuda")

    def run_once(gathers):
        sgwave.sg_forward(plan, v, shots, gathers, None, ws)

    def fastest():
        gathers, times = torch.empty((nshot, g.nrow, nx), device="cuda"), []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            run_once(gathers)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times), gathers

    default, ref = fastest()
    best = sgwave.sg_autotune(plan, v, shots, 64, ws)
    tuned, got = fastest()
    print("%d x %d, %d shots: default %.3f ms, autotuned %.3f ms %s" % (nz, nx, nshot, default, tuned, best), flush=True)
    assert tuned <= 1.1 * default
    assert torch.equal(got, ref)
    plan.set_tuning(**best)
    if not any(best.values()):
        assert plan.get_tuning(nshot)["time_block"] == 4 and fastest()[0] <= 1.1 * default
