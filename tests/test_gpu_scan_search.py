"""EC_FLAG_SCAN_SEARCH (every event by an exact search over all staged disks) gives the sweeps of the windowed search and
of the CPU oracle, bit for bit."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,eta,cells,ell,reject", [(1024, 0.70, 8, 4.0, False), (576, 0.30, 4, 6.0, False),
                                                    (1024, 0.70, 4, 0.5, True)])
def test_scan_search_gives_the_same_events(n, eta, cells, ell, reject):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_6948_amd as P
    st = O.State(O.params(n, eta, ell, cells, dir_mode=O.DIR_ISO, seed=17, boundary=1 if reject else 0))
    st.run(3)
    for flags in (0, P.EC_FLAG_SCAN_SEARCH):
        g = P.System(P.make_params(n, eta, ell, cells, seed=17, flags=flags | (P.EC_FLAG_REJECT if reject else 0)))
        g.sweep(3)
        x, y = g.get_positions()
        np.testing.assert_array_equal(g.get_digests(3), np.array(st.digests[-3:], dtype=np.uint64))
        np.testing.assert_array_equal(x, st.x)
        np.testing.assert_array_equal(y, st.y)
        delta, cnt = g.get_cell_tallies()
        np.testing.assert_array_equal(delta, st.acc_delta)
        np.testing.assert_array_equal(cnt, st.acc_cnt)
        g.close()
