"""The observables' own grid at the sizes where it can go wrong: fewer than
three cells per side (one cell then), radii as wide as the simulation cell or
half the periodic box, radii below the mean spacing (more cells than disks
would be asked for), odd disk counts, and the two passes of the Delaunay
neighbours (dilute systems, where all disks take the wide search; denser ones
where some do).  Against the oracle's brute force: counts and neighbour counts
equal, Psi_k within 1e-12 (complex products against atan2, cos and sin)."""
import numpy as np
import pytest

from oracle import delaunay as D
from oracle import oracle as O

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_6948_amd as P
    P.load_library()
    return P


def _system(P, n, eta, cells, sweeps):
    g = P.System(P.make_params(n, eta, 5.0, cells, dir_mode=0 if cells == 1 else 1, seed=5))
    g.sweep(sweeps)
    x, y = g.get_positions()
    return g, x, y, O.params(n, eta, 5.0, cells, dir_mode=0 if cells == 1 else 1), O.box_length(n, 1.0, eta)


# radius as a share of its limit (the cell side; half the box for one cell), or absolute when below 0
CASES = [(7, 0.20, 1, 1.0), (9, 0.30, 1, 0.7), (33, 0.40, 1, 1.0), (33, 0.40, 1, 0.6), (257, 0.62, 1, 0.3),
         (256, 0.70, 4, 1.0), (257, 0.60, 4, 0.4), (1003, 0.45, 6, -1.02), (4099, 0.70, 8, 0.5), (64, 0.05, 4, 0.2)]


@pytest.mark.parametrize("n,eta,cells,share", CASES)
def test_cutoff_psi_and_pairs_match_brute_force(P, n, eta, cells, share):
    g, x, y, p, L = _system(P, n, eta, cells, 1)
    limit = 0.5 * L if cells == 1 else L / cells
    r = -share if share < 0 else max(share * limit, 1.01)
    psi, nb, per = g.measure_psi6(r, per_disk=True)
    opsi, onb, oper = O.psi6(p, x, y, r)
    assert nb == onb
    assert abs(psi - opsi) < TOL and np.max(np.abs(per - oper)) < TOL
    g.gr_accumulate(r, 37)
    counts, samples, ov = g.gr_counts()
    oc, oov = O.pair_histogram(p, x, y, r, 37)
    assert samples == 1 and ov == oov == 0
    np.testing.assert_array_equal(counts, oc)
    # another radius, hence another grid in the same scratch memory
    assert g.measure_psi6(min(1.3, limit))[1] == O.psi6(p, x, y, min(1.3, limit))[1]


@pytest.mark.parametrize("n,eta,cells,sweeps", [(255, 0.71, 1, 1), (64, 0.66, 1, 2), (1003, 0.30, 6, 2), (1003, 0.48, 6, 3),
                                                (1025, 0.55, 8, 3), (4099, 0.62, 8, 3), (10007, 0.71, 12, 1)])
def test_delaunay_matches_triangulation(P, n, eta, cells, sweeps):
    g, x, y, p, L = _system(P, n, eta, cells, sweeps)
    psi, nb, per, cnt = g.measure_psi6_delaunay(0.0, per_disk=True)
    opsi, oper, ocnt = D.psi6_delaunay(x, y, L, L)
    np.testing.assert_array_equal(cnt, ocnt)
    assert nb == 6.0
    assert abs(psi - opsi) < TOL and np.max(np.abs(per - oper)) < TOL
