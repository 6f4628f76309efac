"""The written-out event loop and the tallies at their edges, against the CPU
oracle, bit for bit (positions, digests, per-cell tallies, pressure): chains
whose records fill the lanes once and several times, also where they are undone
from there; reads that wrap around one periodic box, also along the axes, where
the lattice gives exact distance ties; cells whose window of eight bins is wider
than the cell; more cells than one tile of the tallies' sum."""
import math

import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_6948_amd as P
    P.load_library()
    return P


@pytest.mark.parametrize("n,eta,cells,ell,dir_mode,sweeps,reject", [
    (4096, 0.72, 4, 0.5, 1, 3, True),      # undone at walls and frozen disks, or kept
    (4096, 0.74, 4, 2.0, 1, 3, True),      # some 50 lifts a chain: the lanes fill up, the undo log beyond them
    (1024, 0.74, 4, 40.0, 1, 2, False),    # 1,000 events a chain: the lanes fill many times
    (400, 0.70, 1, 20.0, 1, 2, False),     # one periodic cell: reads wrap around the box
    (81, 0.62, 1, 9.0, 0, 3, False),       # the same, few bins, along the axes
    (576, 0.72, 8, 9.0, 1, 3, False),      # cells of 2.9 sigma: windows wider than the cell
    (16900, 0.50, 46, 1.0, 1, 2, False),   # 2,116 cells: the tallies' second tile, a short one
    (36864, 0.50, 64, 1.0, 1, 1, False),   # 4,096 cells: two whole tiles
])
def test_event_loop_edges(P, n, eta, cells, ell, dir_mode, sweeps, reject):
    print(f"[event loop] n={n} eta={eta} C={cells} ell={ell} dir={dir_mode} reject={reject}", flush=True)
    st = O.State(O.params(n, eta, ell, cells, dir_mode=dir_mode, seed=11, boundary=1 if reject else 0), None, None)
    g = P.System(P.make_params(n, eta, ell, cells, dir_mode=dir_mode, seed=11,
                               flags=P.EC_FLAG_REJECT if reject else 0))
    st.run(sweeps)
    g.sweep(sweeps)
    x, y = g.get_positions()
    np.testing.assert_array_equal(g.get_digests(sweeps), np.array(st.digests[-sweeps:], dtype=np.uint64))
    np.testing.assert_array_equal(x, st.x)
    np.testing.assert_array_equal(y, st.y)
    delta, cnt = g.get_cell_tallies()
    np.testing.assert_array_equal(delta, st.acc_delta)
    np.testing.assert_array_equal(cnt, st.acc_cnt)
    z, bp, counts = g.measure_pressure()
    assert (z, bp) == tuple(st.pressure())
    assert math.isfinite(z) and counts["chains"] > 0
    g.close()
