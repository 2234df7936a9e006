"""GPU set-up and readback kernels at the sizes where their indexing can go
wrong, at both parities of the stored layout: the smallest box, odd boxes,
boxes with bricks of several shapes."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

BOXES = [(2, 3, 2), (17, 19, 23), (64, 4, 32), (130, 6, 5)]


@pytest.fixture(scope="module")
def rf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_08820_amd as rf
    return rf


@pytest.mark.parametrize("rounds", [7, 10])
@pytest.mark.parametrize("dims", BOXES)
def test_thermal_start_at_both_parities(rf, ora, dims, rounds):
    """Stored in FP32 the start is the FP64 oracle's to one rounding of the
    deviation d (2^-24 |d|, |d| <= 8 w here) plus the oracle's own FP64 noise."""
    rho, u = wl.random_velocity(dims, seed=3)
    kw = dict(kT=1e-4, seed=(5 << 32) + 9, stream_id=2, philox_rounds=rounds)
    want = ora.init_thermal(ora.make_params(kT=1e-4, seed=kw["seed"], stream_id=2, rounds=rounds), dims, rho, u)
    w = ora.tables()["w"][:, None]
    for t in (0, 1):
        lat = rf.Lattice(dims, **kw)
        lat.t = t
        lat.init_thermal(rho, u)
        got = lat.populations().cpu().numpy()
        assert np.all(np.abs(got - want) <= 2.0 ** -24 * np.abs(want - w) * 1.001 + 1e-14)
        lat.close()
