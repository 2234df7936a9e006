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


def state(ora, dims, seed):
    rho, u = wl.random_velocity(dims, seed)
    f = ora.init_equilibrium(dims, rho, u)
    return f + 1e-3 * ora.tables()["w"][:, None] * wl.normal_array(f.shape, seed + 1)


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("dims", BOXES)
def test_readbacks_and_parity_change(rf, ora, dims, storage):
    """The readbacks of one state agree at both parities: populations bit for
    bit (the change of layout moves stored words), moments with FP64 sums of
    those populations.  A moment is formed in FP32 from deviations that sum to
    less than 1 over at most 8 additions a value: 8 x 2^-24, and rho rounds once
    more at 1."""
    lat = rf.Lattice(dims, storage=storage, kT=1e-4, seed=3)
    lat.set_populations(state(ora, dims, 7))
    even = lat.populations().cpu().numpy()
    e, b = ora.tables()["e"], 9.5 * 2.0 ** -24
    want = (e @ even)[:10]
    assert np.max(np.abs(lat.moments().cpu().numpy() - want)) <= b
    lat.t = 3
    np.testing.assert_array_equal(lat.populations().cpu().numpy(), even)
    assert np.max(np.abs(lat.moments().cpu().numpy() - want)) <= b
    lat.t = 8
    np.testing.assert_array_equal(lat.populations().cpu().numpy(), even)
    lat.close()


def test_moments_of_a_box_beyond_the_cache(rf, ora):
    """Populations of more than 256 MiB are read past the caches at even step
    counts: the same fields as through the odd layout, bit for bit."""
    dims = (130, 160, 128)
    lat = rf.Lattice(dims, kT=1e-4, seed=3)
    lat.init_thermal()
    even = lat.moments().cpu().numpy()
    lat.t = 1
    np.testing.assert_array_equal(lat.moments().cpu().numpy(), even)
    lat.close()
