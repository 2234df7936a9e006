"""The block shapes of the step give the bits of the tiled kernel: blocks of
consecutive nodes for rows that do not fill waves (row ends inside a wave, rows
shorter than a wave, one block and several), one-wave segments of the 16-bit
steps with noise and of odd steps longer than a block, and both cache policies."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_08820_amd as rf
    return rf


def run(rf, dims, rows, steps, every=0, **kw):
    lat = rf.Lattice(dims, **kw)
    lat.set_row_blocks(rows)
    if kw["kT"] > 0:
        lat.init_thermal()
    else:
        lat.init_equilibrium(u=0.01 * np.random.default_rng(1).standard_normal((3, lat.n)))
    lat.stats_config(every)
    lat.step(steps)
    lat.sync()
    f, s = lat.populations(), lat.stats()
    lat.close()
    return f, s


BOXES = [(2, 3, 2), (17, 19, 23), (63, 2, 2), (65, 4, 16), (96, 6, 32), (130, 9, 5), (300, 3, 4),
         (64, 3, 2), (192, 5, 4), (320, 2, 16), (1088, 2, 2)]


@pytest.mark.parametrize("storage,kT,extra", [
    ("f32", 1e-4, {}), ("f16", 1e-4, dict(tau_ghost=0.8)), ("bf16", 1e-4, dict(model="bgk")),
    ("bf16", 0.0, dict(storage_scale=0.01))])
@pytest.mark.parametrize("dims", BOXES)
def test_block_shapes_store_the_same_bits(rf, dims, storage, kT, extra):
    kw = dict(storage=storage, kT=kT, tau=0.7, seed=5, **extra)
    a, sa = run(rf, dims, True, 7, every=3, **kw)
    b, sb = run(rf, dims, False, 7, every=3, **kw)
    assert bool((a == b).all())
    assert sa["samples"] == sb["samples"] == 3
    if dims[0] % 64 == 0:
        return  # whole rows add each wave in FP32
    # both add the same FP32 values in FP64, in another order: within n 2^-53 of
    # the sum of magnitudes, which is at most sqrt(n sum of squares)
    n = sa["nodes"] * sa["samples"]
    squares = dict(sum_drho="sum_drho2", mass_dev="sum_drho2", sum_j="sum_j2", momentum="sum_j2", sum_pi="sum_pi2")
    for k, v in sa.items():
        size = np.sqrt(n * sa[squares[k]]) if k in squares else np.abs(v)
        assert np.all(np.abs(v - sb[k]) <= n * 2.0 ** -53 * size), k


@pytest.mark.parametrize("storage,dims", [("f32", (256, 128, 112)), ("f16", (256, 256, 112)), ("f32", (100, 256, 128))])
def test_boxes_beyond_the_cache(rf, storage, dims):
    kw = dict(storage=storage, kT=1e-4, tau=0.7, seed=5)
    a, _ = run(rf, dims, True, 3, **kw)
    b, _ = run(rf, dims, False, 3, **kw)
    assert bool((a == b).all())


@pytest.mark.parametrize("storage,dims", [("f32", (16, 16, 16)), ("f32", (2, 3, 2)), ("f16", (64, 9, 16)),
                                          ("f32", (64, 64, 40)), ("f32", (17, 19, 23))])
def test_statistics_of_one_call_and_of_many(rf, storage, dims):
    """The partials of a call's sampled steps are added together at its end, in
    more than one batch where they exceed their slots: the sums are bit for bit
    those of one call per step."""
    lats = [rf.Lattice(dims, storage=storage, kT=1e-4, tau=0.7, seed=2) for _ in range(2)]
    for lat in lats:
        lat.init_thermal()
        lat.stats_config(1)
    lats[0].step(70)
    for _ in range(70):
        lats[1].step(1)
    a, b = (lat.stats() for lat in lats)
    assert a["samples"] == 70
    for k in a:
        np.testing.assert_array_equal(a[k], b[k], err_msg=k)
    for lat in lats:
        lat.close()
