"""The kernels that a box's step takes beyond the memory-side cache and on rows of
special lengths store the bits of the tiled kernel."""
import numpy as np
import pytest

import workloads as wl

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


# every count of blocks that a CU is held to beyond the cache
HELD = [("f32", nx, kT) for nx in (64, 128, 192, 256, 320, 384, 448, 512, 640, 768, 896, 1024) for kT in (1e-4, 0.0)]
HELD += [(s, nx, 0.0) for s, nx in (("f16", 64), ("bf16", 128), ("f16", 192), ("bf16", 256), ("f16", 1024))]


@pytest.mark.parametrize("storage,nx,kT", HELD)
def test_rows_with_fewer_waves_beyond_the_cache(rf, storage, nx, kT):
    kw = dict(storage=storage, kT=kT, tau=0.7, seed=8, model="bgk")
    if storage != "f32":
        kw["storage_scale"] = 0.01
    dims = (nx, 47, (3200000 if storage == "f32" else 6400000) // (47 * nx))
    a, sa = run(rf, dims, True, 4, every=3, **kw)
    b, sb = run(rf, dims, False, 4, every=3, **kw)
    assert bool((a == b).all())
    n = sa["nodes"] * sa["samples"]
    for k in ("sum_drho2", "sum_j2", "sum_u2", "sum_pi2"):
        assert np.all(np.abs(sa[k] - sb[k]) <= n * 2.0 ** -53 * np.abs(sa[k])), k


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


# recursive ghosts are a kernel of their own in every block shape: flat, rows, waves (16
# bits with noise; odd steps of long rows), and the tiles of all of them
@pytest.mark.parametrize("storage,kT", [("f32", 1e-4), ("f32", 0.0), ("f16", 1e-4), ("bf16", 1e-4)])
@pytest.mark.parametrize("dims", [(17, 19, 23), (65, 4, 16), (130, 9, 5), (64, 3, 2), (192, 5, 4), (1088, 2, 2)])
def test_recursive_ghosts_in_every_block_shape(rf, dims, storage, kT):
    kw = dict(storage=storage, kT=kT, tau=0.7, tau_bulk=1.2, model="rec", tau_ghost=list(np.linspace(0.6, 1.8, 17)), seed=9)
    a, sa = run(rf, dims, True, 7, every=3, **kw)
    b, sb = run(rf, dims, False, 7, every=3, **kw)
    assert bool((a == b).all())
    assert sa["samples"] == sb["samples"] == 3


# the tiled kernel, which rows that do not fill waves reach beyond 4 GiB and with row
# blocks off
TILED = {
    "ragged_130x9x5": ((130, 9, 5), dict(kT=1e-4, tau=0.55, seed=11)),
    "ragged_300x3x4": ((300, 3, 4), dict(kT=1e-4, tau=0.6, seed=12)),
    "odd_17x19x23_mrt": ((17, 19, 23), dict(kT=1e-5, tau=0.8, tau_bulk=1.0, tau_ghost=list(np.linspace(0.7, 1.6, 17)),
                                            seed=7, stream_id=3)),
    "wide_1088x2x2": ((1088, 2, 2), dict(kT=1e-4, tau=0.65, seed=17)),
    "rec_17x19x23": ((17, 19, 23), dict(kT=1e-4, tau=0.7, tau_bulk=1.2, model="rec",
                                        tau_ghost=list(np.linspace(0.55, 1.9, 17)), seed=20)),
    "rec_kT0_33x7x6": ((33, 7, 6), dict(kT=0.0, tau=0.9, model="rec", tau_ghost=1.5)),
    "rec_128x5x3": ((128, 5, 3), dict(kT=1e-4, tau=0.6, model="rec", tau_ghost=0.8, seed=21)),
}


@pytest.mark.parametrize("case", list(TILED))
def test_tiled_trajectories_match_the_oracle(rf, ora, case):
    """max |f_gpu - f_oracle| / (w_i rho0) <= 1e-5 at every step, as for every other
    kernel (the bar of the method's specification)."""
    dims, kw = TILED[case]
    rho, u = wl.random_velocity(dims, 31)
    w = ora.tables()["w"][:, None]
    ref = ora.init_equilibrium(dims, rho, u)
    ref = ref + 1e-3 * w * wl.normal_array(ref.shape, 32)
    lat = rf.Lattice(dims, **kw)
    lat.set_row_blocks(False)
    lat.set_populations(ref)
    p = ora.make_params(kT=kw["kT"], tau_shear=kw["tau"], tau_bulk=kw.get("tau_bulk"), tau_ghost=kw.get("tau_ghost", 1.0),
                        seed=kw.get("seed", 1), stream_id=kw.get("stream_id", 0), rounds=7, model=kw.get("model", "reg"))
    for t in range(40):
        lat.step(1)
        ref = ora.step(p, dims, ref, t)
        assert np.max(np.abs(lat.populations().cpu().numpy() - ref) / w) <= 1e-5, t + 1
    lat.close()
