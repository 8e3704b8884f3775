"""Fault's pull of four voxels at a time and the polynomial sinc weights at the
sizes where they can go wrong, against the FP64 oracle at the bar of every
builder test: volumes of one to a few rows per axis (bricks and quads cut short,
rows shorter than the eight taps, one-row y axes), sources beyond every edge,
slips of more than a radian, voxels pulled together and alone in one wave; and
fractions from 0 to just below 1, where whole shifts move the profile exactly."""
import numpy as np
import pytest

from oracle import builder as OB
from paper_2605_30541_amd import sgwave
from test_gpu_builder import TOL, _dev, _host, rel_l2

pytestmark = pytest.mark.gpu


def _case(nz, ny, nx, slip, azimuth):
    """A fault through the middle whose taper covers the volume."""
    ext = np.array([nz, ny, nx]) * 10.0
    return dict(cz=0.5 * ext[0], cy=0.5 * ext[1], cx=0.5 * ext[2], azimuth_deg=azimuth, dip_deg=50.0, radius=700.0,
                slip=slip, direction=1, die_r=600.0, die_strike=1500.0, die_theta_deg=80.0)


@pytest.mark.parametrize("slip,azimuth", [(12.0, 30.0), (90.0, -75.0), (900.0, 10.0)])
@pytest.mark.parametrize("nz,ny,nx", [(1, 9, 70), (3, 4, 64), (4, 5, 65), (5, 2, 63), (13, 3, 9), (9, 6, 7), (8, 8, 8),
                                      (33, 9, 129), (21, 1, 40), (64, 17, 100)])
def test_fault_pull_matches_the_oracle(nz, ny, nx, slip, azimuth):
    p = _case(nz, ny, nx, slip, azimuth)
    rng = np.random.default_rng(nz * 100 + nx)
    V = rng.uniform(1500.0, 4500.0, (nz, ny, nx)).astype(np.float32)
    got = _host(sgwave.fault(_dev(V), 10.0, 10.0, 10.0, p, 1480.0))
    ref = OB.fault(V.astype(np.float64), 10.0, 10.0, 10.0, p, 1480.0)
    (_, _, _), w = OB.fault_source(V.shape, 10.0, 10.0, 10.0, p)
    assert np.count_nonzero(w) > 0.5 * V.size
    assert rel_l2(got, ref) <= TOL


def test_weights_over_the_fraction():
    rng = np.random.default_rng(5)
    nz, nx = 40, 4096
    V = rng.uniform(-1.0, 1.0, (nz, 1, nx)).astype(np.float32)
    frac = np.concatenate([np.linspace(0.0, 1.0, nx - 4), [1e-7, 0.99999994, 3.0, -2.0]]).astype(np.float32)
    shift = frac[None, :]
    got = _host(sgwave.squish(_dev(V), 1.0, _dev(shift)))
    ref = OB.squish(V.astype(np.float64), 1.0, shift.astype(np.float64))
    # 8 weights off by <= 1.2e-7 and 8 roundings of sums below 2.5 (the largest sum of |weights|, 2.1)
    assert np.abs(got - ref).max() <= 8 * 1.2e-7 + 8 * 2.5 * 6e-8
    whole = np.flatnonzero(frac == np.floor(frac))
    for c in whole:
        z = np.clip(np.arange(nz) + int(frac[c]), 0, nz - 1)
        assert np.array_equal(got[:, 0, c], V[z, 0, c])
