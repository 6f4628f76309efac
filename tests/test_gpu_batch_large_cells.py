"""Batches whose cells take so much LDS that the wavefronts of a workgroup decide how many fit on a CU: the default
schedule gives every system the trajectory of a run of its own, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1409_6948_amd as P
    P.load_library()
    return P


# (disks, density, cells per side) of the systems: cells of about 12 and 21 KB, of 33, of 45
@pytest.mark.parametrize("systems", [[(4096, 0.70, 8), (9216, 0.30, 10), (2304, 0.45, 6)],
                                     [(9216, 0.30, 8), (4096, 0.70, 4)], [(16384, 0.30, 8), (256, 0.70, 4)]])
@pytest.mark.parametrize("reject", [False, True])
def test_default_batch_equals_solo_runs(P, systems, reject):
    ell = 0.3 if reject else 4.0
    ps = [P.make_params(n, eta, ell, cells, seed=31 + i, system=i, flags=P.EC_FLAG_REJECT if reject else 0)
          for i, (n, eta, cells) in enumerate(systems)]
    b = P.Batch(ps)
    b.sweep(2)
    b.stream.synchronize()
    for p, s in zip(ps, b.systems):
        g = P.System(p)
        g.sweep(2)
        for a, c in zip(s.get_positions(), g.get_positions()):
            np.testing.assert_array_equal(a, c)
        np.testing.assert_array_equal(s.get_digests(2), g.get_digests(2))
        g.close()
    b.close()
