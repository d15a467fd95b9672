"""The general row pipeline: complex order parameters, per-bond hopping and
pairing under moment doubling, and neighbour moments (direct recursion), at
the edges of its lane widths and on wrapping, narrow and one-row lattices.
Doubling against the direct algorithm's one-step kernels (FP64 1e-12, FP32
2e-5 as elsewhere), neighbour moments against the oracle-pinned direct
moments of the same sites and against each other across bonds."""
import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_common import DEV, gpu_moments, maxdiff

pytestmark = pytest.mark.gpu

KINDS = [(True, False, 0.0), (True, True, 0.0), (True, True, 1.0 / 16.0), (False, True, 0.0)]


def _workload(Lx, Ly, N, bcx, bcy, kind, n):
    cplx, bond, flux = kind
    return W.small_random(Lx, Ly, N, seed=Lx + 7 * Ly, bc_x=bcx, bc_y=bcy, complex_=cplx, bond=bond, flux=flux,
                          n_sites=min(n, Lx * Ly))


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 2e-5)])
@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("Lx,Ly,bcx,bcy", [
    (1, 9, 0, 0), (3, 3, 1, 1), (63, 12, 0, 1), (64, 9, 1, 0), (65, 14, 1, 1), (128, 7, 0, 0), (129, 6, 0, 1),
    (192, 5, 1, 0), (40, 61, 1, 1),
])
def test_doubling_matches_direct(Lx, Ly, bcx, bcy, kind, precision, tol):
    for N in (4, 5, 37, 80):
        w = _workload(Lx, Ly, N, bcx, bcy, kind, 150)
        op, ee, he = gpu_moments(w, N=N, tile=150, precision=precision, algorithm=2)
        op.close()
        op, d_ee, d_he = gpu_moments(w, N=N, tile=150, algorithm=1)
        op.close()
        assert maxdiff(ee, d_ee) <= tol and maxdiff(he, d_he) <= tol
        assert np.all(he[:, 0::2] == 0)


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 2e-5)])
@pytest.mark.parametrize("kind", KINDS + [(False, False, 0.0)])
@pytest.mark.parametrize("Lx,Ly,bcx,bcy,N", [
    (4, 3, 1, 1, 1), (4, 3, 1, 1, 2), (4, 3, 0, 0, 3), (64, 3, 1, 0, 20), (65, 5, 0, 1, 33), (1, 7, 0, 0, 18),
    (128, 4, 1, 1, 26), (20, 31, 0, 0, 45),
])
def test_neighbour_moments(Lx, Ly, bcx, bcy, N, kind, precision, tol):
    import paper_1007_1609_amd as P
    w = _workload(Lx, Ly, N, bcx, bcy, kind, Lx * Ly)
    op = P.Operator.from_workload(w, DEV)
    sites = torch.as_tensor(w.start_sites, device=DEV)
    ee, he, nb_ee, nb_he = (t.cpu().numpy() for t in P.chebyshev_moments_nb(op, sites, N, len(w.start_sites), precision))
    op.close()
    op, d_ee, d_he = gpu_moments(w, N=N, tile=len(w.start_sites), algorithm=1)
    op.close()
    assert maxdiff(ee, d_ee) <= tol and maxdiff(he, d_he) <= tol
    x, y = np.arange(Lx * Ly) % Lx, np.arange(Lx * Ly) // Lx
    for axis, (pos, size, bc, step) in enumerate(((x, Lx, bcx, 1), (y, Ly, bcy, Lx))):
        ok = np.ones(Lx * Ly, bool) if bc else pos < size - 1
        i = np.flatnonzero(ok)
        j = np.where(pos[i] < size - 1, i + step, i - (size - 1) * step)
        # <j,e|T_n|i,e> = conj <i,e|T_n|j,e>: T_n of a Hermitian matrix
        assert maxdiff(nb_ee[i, 2 * axis], np.conj(nb_ee[j, 2 * axis + 1])) <= tol
        # sites without a neighbour in this direction have zero rows
        assert np.all(nb_ee[~ok, 2 * axis] == 0) and np.all(nb_he[~ok, 2 * axis] == 0)
    # completeness: sum of squares of step 1's row is 2's doubling moment
    if N > 2:
        nrm = ee[:, 1] ** 2 + np.abs(he[:, 1]) ** 2
        nrm += (np.abs(nb_ee[:, :, 1]) ** 2 + np.abs(nb_he[:, :, 1]) ** 2).sum(axis=1)
        assert maxdiff(2 * nrm - 1, ee[:, 2]) <= 2 * tol


def test_tiles_and_invalid_sites():
    w = _workload(48, 40, 50, 0, 0, KINDS[2], 1920)
    sites = w.start_sites.copy()
    sites[[0, 700, 1919]] = [-1, 1920, 1 << 30]
    op, ee, he = gpu_moments(w, sites=sites, N=50, tile=1024, algorithm=2)
    op.close()
    bad = np.isnan(ee).all(axis=1) & np.isnan(he).all(axis=1)
    assert list(np.flatnonzero(bad)) == [0, 700, 1919]
    op, d_ee, d_he = gpu_moments(w, sites=sites, N=50, tile=700, algorithm=1)
    op.close()
    assert maxdiff(ee[~bad], d_ee[~bad]) <= 1e-12 and maxdiff(he[~bad], d_he[~bad]) <= 1e-12


@pytest.mark.parametrize("precision,tol", [(0, 1e-12), (1, 2e-5)])
@pytest.mark.parametrize("kind", KINDS + [(False, False, 0.0)])
@pytest.mark.parametrize("Lx,bcx", [(8, 0), (8, 1), (33, 1), (100, 0)])
def test_neighbour_moments_of_two_open_rows(Lx, bcx, kind, precision, tol):
    """Two rows, open in y: the lower row has no -y neighbour, the upper no +y
    one, and the row there is stays in its own slot (oracle)."""
    import oracle
    import paper_1007_1609_amd as P
    w = _workload(Lx, 2, 32, bcx, 0, kind, 2 * Lx)
    op = P.Operator.from_workload(w, DEV)
    sites = torch.as_tensor(w.start_sites, device=DEV)
    _, _, nb_ee, nb_he = (t.cpu().numpy() for t in P.chebyshev_moments_nb(op, sites, w.N, len(sites), precision))
    a, b = op.bounds.a, op.bounds.b
    op.close()
    o_ee, o_he = oracle.neighbour_moments(oracle.workload_csr(w, a, b), Lx, 2, bcx, 0, w.start_sites, w.N)
    assert maxdiff(nb_ee, o_ee) <= tol and maxdiff(nb_he, o_he) <= tol


from tests.gpu_common import TOL_MOMENT  # noqa: E402

# Neighbour moments whose passes wrap or close rows, or take two columns a lane,
# with the kinds (index into KINDS, 3 + 1: real uniform) and precisions that the
# library gives to the row pipeline; tests/test_plan_host.py checks that it does.
_ALL = [(k, p) for k in range(5) for p in (0, 1)]
NB_ROUTED = [
    (65, 9, 0, 1, 30, 90, _ALL), (65, 9, 1, 1, 30, 90, _ALL), (128, 10, 1, 1, 30, 90, _ALL), (128, 10, 1, 0, 60, 90, _ALL),
    (64, 12, 1, 0, 60, 90, _ALL), (48, 40, 1, 0, 30, 100, _ALL), (100, 24, 1, 0, 60, 100, _ALL),
    # more rows than two passes' halo
    (48, 40, 0, 1, 12, 100, [(4, 0), (3, 0), (1, 0), (2, 0), (3, 1), (0, 1), (1, 1), (2, 1)]),
    (64, 61, 1, 1, 6, 150, [(3, 1), (1, 1)]),
]


@pytest.mark.parametrize("case,kind,precision", [(c[:6], k, p) for c in NB_ROUTED for k, p in c[6]])
def test_routed_neighbour_moments_match_oracle(case, kind, precision):
    import oracle
    import paper_1007_1609_amd as P
    Lx, Ly, bcx, bcy, n, N = case
    w = _workload(Lx, Ly, N, bcx, bcy, (KINDS + [(False, False, 0.0)])[kind], n)
    sites = w.start_sites.copy()
    sites[:6] = [0, Lx - 1, Lx * Ly - 1, Lx * (Ly - 1), Lx, Lx * Ly - 2]
    op = P.Operator.from_workload(w, DEV)
    out = P.chebyshev_moments_nb(op, torch.as_tensor(sites, device=DEV), N, n, precision)
    ee, he, nb_ee, nb_he = (t.cpu().numpy() for t in out)
    a, b = op.bounds.a, op.bounds.b
    op.close()
    tol = 2e-5 if precision else TOL_MOMENT
    o_ee, o_he = oracle.neighbour_moments(oracle.workload_csr(w, a, b), Lx, Ly, bcx, bcy, sites, N)
    assert maxdiff(nb_ee, o_ee) <= tol and maxdiff(nb_he, o_he) <= tol
    l_ee, l_he = oracle.workload_moments(w, a, b, sites=sites)
    assert maxdiff(ee, l_ee) <= tol and maxdiff(he, l_he) <= tol


# Doubling: (Lx, Ly, bc_x, bc_y, vectors, N, kinds of KINDS in FP64 and FP32 that take the pipeline)
DOUBLING_ROUTED = [
    (1, 9, 0, 0, 9, 80, (0, 1, 3), (0, 1, 3)), (3, 3, 1, 1, 9, 81, (0, 1, 3), (0, 1, 3)), (63, 12, 0, 1, 150, 80, (0, 1, 3), (0, 1, 3)),
    (64, 9, 1, 0, 150, 120, (0, 1, 3), (0,)), (65, 14, 1, 1, 150, 80, (0, 1, 3), (0, 1, 3)), (128, 7, 0, 0, 150, 121, (0, 1, 3), (0,)),
    (129, 6, 0, 1, 150, 80, (), (0, 1, 3)), (40, 61, 1, 1, 150, 121, (0, 1, 3), (0,)), (127, 20, 0, 1, 150, 120, (0, 1, 3), (0, 1, 3)),
    (33, 48, 0, 1, 100, 160, (0, 1, 3), (0, 1, 3)),
]


@pytest.mark.parametrize("case,kind,precision", [(c[:6], k, p) for c in DOUBLING_ROUTED for p in (0, 1) for k in c[6 + p]])
def test_routed_doubling_matches_oracle(case, kind, precision):
    import oracle
    Lx, Ly, bcx, bcy, n, N = case
    w = _workload(Lx, Ly, N, bcx, bcy, KINDS[kind], n)
    op, ee, he = gpu_moments(w, N=N, tile=n, precision=precision, algorithm=2)
    a, b = op.bounds.a, op.bounds.b
    op.close()
    few = slice(None, None, max(1, len(w.start_sites) // 12))
    o_ee, o_he = oracle.workload_moments(w, a, b, sites=w.start_sites[few])
    tol = 2e-5 if precision else TOL_MOMENT
    assert maxdiff(ee[few], o_ee) <= tol and maxdiff(he[few], o_he) <= tol
