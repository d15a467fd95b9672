"""One step per launch with per-vector light cones (complex and per-bond
operators on lattices wider than the row pipeline's): blocks of 64 columns and
their edges, wrapping cones, start sites at corners and block edges, batches of
steps, ragged tiles, invalid sites; against the direct algorithm (1e-12; the
FP32 kernel is the uniform complex one, 2e-5)."""
import itertools

import numpy as np
import pytest

import workloads as W
from tests.gpu_common import gpu_moments, maxdiff

pytestmark = pytest.mark.gpu


def _check(w, N, tile, precision, tol, sites=None):
    op, ee, he = gpu_moments(w, sites=sites, N=N, tile=tile, precision=precision, algorithm=2)
    op.close()
    op, d_ee, d_he = gpu_moments(w, sites=sites, N=N, tile=tile, algorithm=1)
    op.close()
    ok = ~np.isnan(d_ee[:, 0])
    assert np.array_equal(ok, ~np.isnan(ee[:, 0]))
    assert maxdiff(ee[ok], d_ee[ok]) <= tol and maxdiff(he[ok], d_he[ok]) <= tol


@pytest.mark.parametrize("kind", [(True, False, 0.0), (True, True, 1.0 / 16.0), (False, True, 0.0)])
@pytest.mark.parametrize("bcx,bcy", list(itertools.product((0, 1), (0, 1))))
@pytest.mark.parametrize("Lx,Ly", [(193, 90), (256, 70), (257, 65), (320, 33)])
def test_cones_and_blocks(Lx, Ly, bcx, bcy, kind):
    cplx, bond, flux = kind
    for N in (4, 18, 20, 35, 90):  # around a batch of eight steps; the largest wraps or leaves the rule's range
        w = W.small_random(Lx, Ly, N, seed=Lx + N, bc_x=bcx, bc_y=bcy, complex_=cplx, bond=bond, flux=flux, n_sites=70)
        sites = w.start_sites.copy()
        sites[:8] = [0, Lx - 1, Lx * Ly - 1, Lx * (Ly - 1), 63, 64, Lx * (Ly // 2) + 127, -1]
        _check(w, N, 48, 0, 1e-12, sites)
        if not bond:
            _check(w, N, 70, 1, 2e-5, sites)


@pytest.mark.parametrize("kind", [(True, False, 0.0), (True, True, 1.0 / 16.0), (False, True, 0.0)])
@pytest.mark.parametrize("bcx,bcy", list(itertools.product((0, 1), (0, 1))))
@pytest.mark.parametrize("Lx,Ly,N", [(140, 12, 150), (193, 5, 260), (130, 1, 150)])
def test_small_tiles_past_the_cones(Lx, Ly, N, bcx, bcy, kind):
    cplx, bond, flux = kind
    if Ly < 3 and (bcy or flux):
        pytest.skip("periodic y needs three rows")
    w = W.small_random(Lx, Ly, N, seed=N, bc_x=bcx, bc_y=bcy, complex_=cplx, bond=bond, flux=flux, n_sites=40)
    _check(w, N, 40, 0, 1e-12)
