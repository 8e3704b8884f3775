"""The gradient's bookkeeping at the sizes where it can go wrong, against the
FP64 oracle (relative L2 <= 1e-4, the bar of every propagation test): the fold
of the padded cells onto the edge cells of the model (models of one or two
rows or columns, no sponge, a sponge wider than the model, both tops, more
shots than one), and checkpoints written in place (the last level on a
checkpoint, one past it, a checkpoint at every level, a spacing longer than
the record)."""
import numpy as np
import pytest

import oracle
from paper_2605_30541_amd import sgwave
from paper_2605_30541_amd.sgwave import Geometry
from test_gpu_gradient import _og, gpu_gradient, rel_l2

pytestmark = pytest.mark.gpu
TOL = 1e-4


def run_case(nz, nx, nbl, top, nt, ckpt, nshot=3, tuning=None):
    rng = np.random.default_rng(nz * 1000 + nx)
    g = Geometry(nz=nz, nx=nx, dz=10.0, dx=10.0, dt=1e-3, nt=nt, nbl=nbl, top=top, vmax_hint=3000.0)
    v = rng.uniform(1800.0, 3000.0, (nz, nx)).astype(np.float32)
    src = np.stack([rng.uniform(0, (nz - 1) * 10.0, nshot), rng.uniform(0, (nx - 1) * 10.0, nshot)], 1)
    rec = np.stack([rng.uniform(0, (nz - 1) * 10.0, 9), rng.uniform(0, (nx - 1) * 10.0, 9)], 1)
    wl = oracle.ricker(40.0, g.dt, g.nt, t0=0.012)
    resid = rng.standard_normal((nshot, g.nrow, 9)).astype(np.float32)
    ref = oracle.gradient(_og(g), v.astype(np.float64), src, wl, rec, resid.astype(np.float64))
    d_ref, _ = oracle.forward(_og(g), v.astype(np.float64), src, wl, rec)
    got, gathers = gpu_gradient(g, v, src, rec, wl, resid, ckpt=ckpt, tuning=tuning)
    print("gradient %.2e gathers %.2e" % (rel_l2(got, ref), rel_l2(gathers, d_ref)), flush=True)
    assert np.linalg.norm(d_ref[:, -1]) > 0 and np.linalg.norm(ref) > 0
    assert rel_l2(gathers, d_ref) <= TOL
    assert rel_l2(gathers[:, -1], d_ref[:, -1]) <= TOL
    assert rel_l2(got, ref) <= TOL


@pytest.mark.parametrize("nz,nx,nbl,top", [
    (1, 30, 5, sgwave.SG_TOP_ABSORBING), (30, 1, 5, sgwave.SG_TOP_ABSORBING), (2, 2, 4, sgwave.SG_TOP_ABSORBING),
    (2, 31, 7, sgwave.SG_TOP_FREE), (31, 2, 40, sgwave.SG_TOP_FREE), (17, 23, 0, sgwave.SG_TOP_ABSORBING),
    (33, 65, 40, sgwave.SG_TOP_FREE), (3, 3, 1, sgwave.SG_TOP_FREE)])
def test_fold_onto_the_edge_cells(nz, nx, nbl, top):
    run_case(nz, nx, nbl, top, nt=40, ckpt=9)


@pytest.mark.parametrize("tuning", [None, dict(variant=3, tile_x=128, tile_z=0, time_block=4)],
                         ids=["tiled", "sweep"])
@pytest.mark.parametrize("nt,ckpt", [(41, 10), (42, 10), (40, 10), (30, 1), (30, 64), (25, 24), (3, 2)])
def test_checkpoints_in_place(nt, ckpt, tuning):
    run_case(21, 37, 6, sgwave.SG_TOP_FREE, nt=max(nt, 3), ckpt=ckpt, tuning=tuning)
