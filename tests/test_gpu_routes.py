"""The kernels that a box's step takes beyond the memory-side cache and on rows of
special lengths store the bits of the tiled kernel."""
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


# flat blocks streamed (whole and half lines, partial bricks), rows left to tiles: narrow
# ones and ones that fill their tiles
FLAT = [("f32", (96, 161, 170)), ("f32", (16, 420, 401)), ("f32", (1040, 51, 52)), ("f32", (48, 255, 230)),
        ("f32", (1008, 52, 53)), ("f16", (63, 290, 290)), ("bf16", (300, 132, 130))]


@pytest.mark.parametrize("kT", [1e-4, 0.0])
@pytest.mark.parametrize("storage,dims", FLAT)
def test_rows_that_do_not_fill_waves_beyond_the_cache(rf, storage, dims, kT):
    kw = dict(storage=storage, kT=kT, tau=0.7, seed=5)
    if storage != "f32" and kT == 0.0:
        kw["storage_scale"] = 0.01
    a, sa = run(rf, dims, True, 4, every=3, **kw)
    b, sb = run(rf, dims, False, 4, every=3, **kw)
    assert bool((a == b).all())
    assert sa["samples"] == sb["samples"] == 2
    # both add the same FP32 values in FP64, in another order
    n = sa["nodes"] * sa["samples"]
    for k in ("sum_drho2", "sum_j2", "sum_u2", "sum_pi2"):
        assert np.all(np.abs(sa[k] - sb[k]) <= n * 2.0 ** -53 * np.abs(sa[k])), k


# rows longer than a block: odd steps in tiles and in waves, streamed and not
LONG = [("f32", (1152, 3, 5)), ("f32", (1088, 3, 4)), ("f32", (1280, 50, 52)), ("f32", (1216, 50, 52)),
        ("f16", (1280, 72, 70)), ("f16", (1088, 72, 80)), ("bf16", (2048, 5, 3))]


@pytest.mark.parametrize("kT", [1e-4, 0.0])
@pytest.mark.parametrize("storage,dims", LONG)
def test_rows_longer_than_a_block(rf, storage, dims, kT):
    kw = dict(storage=storage, kT=kT, tau=0.7, seed=6)
    if storage != "f32" and kT == 0.0:
        kw["storage_scale"] = 0.01
    a, _ = run(rf, dims, True, 5, **kw)
    b, _ = run(rf, dims, False, 5, **kw)
    assert bool((a == b).all())


@pytest.mark.parametrize("storage,dims", [("f16", (256, 250, 80)), ("bf16", (192, 190, 142))])
def test_16_bit_steps_with_noise_at_the_size_of_the_cache(rf, storage, dims):
    kw = dict(storage=storage, kT=1e-4, tau=0.7, seed=7)
    a, _ = run(rf, dims, True, 5, **kw)
    b, _ = run(rf, dims, False, 5, **kw)
    assert bool((a == b).all())


@pytest.mark.parametrize("storage,kT,dims", [("f16", 0.0, (64, 36, 100)), ("bf16", 0.0, (128, 32, 31)),
                                             ("f16", 0.0, (1280, 16, 15)), ("f32", 1e-4, (64, 63, 30)),
                                             ("f32", 1e-4, (192, 32, 32)), ("f32", 0.0, (64, 64, 30))])
def test_small_boxes_that_stream(rf, storage, kT, dims):
    kw = dict(storage=storage, kT=kT, tau=0.7, seed=8)
    if kT == 0.0 and storage != "f32":
        kw["storage_scale"] = 0.01
    a, sa = run(rf, dims, True, 5, every=2, **kw)
    b, sb = run(rf, dims, False, 5, every=2, **kw)
    assert bool((a == b).all())
    assert sa["samples"] == sb["samples"] == 3
