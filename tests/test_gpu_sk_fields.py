"""Structure factor of fields of unlike size: each field's spectrum is as exact
as its own values allow, whatever the other nine hold.  Boxes with an even and an
odd number of x-rows, several rows to a block and one pair, every kind of
transform length."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

BOXES = [(16, 16, 16), (2, 3, 3), (60, 45, 37), (256, 3, 5), (512, 3, 4), (1024, 3, 3), (97, 6, 13), (130, 9, 5)]


@pytest.fixture(scope="module")
def rf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_08820_amd as rf
    return rf


def shells(dims):
    nx, ny, nz = dims
    k = [np.fft.fftfreq(n, 1.0 / n) for n in (nz, ny, nx)]
    s = np.rint(np.sqrt(k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2] ** 2)).astype(int).ravel()
    return s


def populations(ora, m):
    """f_i = w_i (1 + sum_k m_k e_ki / b_k) with the ten moments m (10, N)."""
    t = ora.tables()
    return t["w"][:, None] * (1.0 + (t["e"][:10].T / t["b"][:10]) @ m)


def density_deviation(f, w):
    """rho - rho0 as the kernels form it: FP32 sums of three along x, y and z."""
    d = (f - w[:, None]).astype(np.float32).reshape(3, 3, 3, -1)  # c_z, c_y, c_x
    for axis in (2, 1, 0):
        lo, mid, hi = np.moveaxis(d, axis, 0)
        d = (lo + hi) + mid
    return d.astype(np.float64)


def check_field(got, field, dims, shell):
    """A transform of N FP32 values errs by at most delta of its norm, delta = 4
    roundings of 2^-24 for each of log2 N levels; a shell's share of that error
    adds to it by the triangle inequality."""
    n = field.size
    p = (np.abs(np.fft.fftn(field.reshape(dims[::-1]))) ** 2 / n).ravel()
    want = np.bincount(shell[1:], p[1:], minlength=len(got))
    delta = 4.0 * max(np.log2(n), 1.0) * 2.0 ** -24
    assert np.all(np.abs(got - want) <= 2.0 * delta * np.sqrt(want * p.sum()) + delta ** 2 * p.sum())


@pytest.mark.parametrize("weak", [(0, 1, 4, 6, 8), (3, 2, 5, 7, 9), (0, 5), (1, 2, 3)])
@pytest.mark.parametrize("dims", BOXES)
def test_weak_fields_beside_strong_ones(rf, ora, dims, weak):
    m = 1e-3 * np.random.default_rng(4).standard_normal((10, int(np.prod(dims))))
    m[list(weak)] *= 1e-6
    lat = rf.Lattice(dims, kT=1e-4)
    lat.set_populations(populations(ora, m))
    fields = lat.moments().cpu().numpy().astype(np.float64)
    fields[0] = density_deviation(lat.populations().cpu().numpy(), ora.tables()["w"])
    lat.sk_sample()
    shell = shells(dims)
    for f in range(10):
        check_field(lat.sk(f)[0], fields[f], dims, shell)
    lat.close()


def test_a_field_that_overflows_leaves_the_others(rf, ora):
    """Populations of opposite sign with c_x = +-1 and no c_y, c_z make j_x
    overflow in FP32 and no other of the ten fields: only its sums are not finite."""
    dims = (16, 4, 5)
    n = int(np.prod(dims))
    f = populations(ora, 1e-3 * np.random.default_rng(5).standard_normal((10, n)))
    f[14, 7], f[12, 7] = 3e38, -3e38  # i = (c_x + 1) + 3 (c_y + 1) + 9 (c_z + 1)
    lat = rf.Lattice(dims, kT=1e-4)
    lat.set_populations(f)
    fields = lat.moments().cpu().numpy()
    finite = np.isfinite(fields).all(axis=1)
    assert not finite[1] and finite[[0, 2, 3]].all()
    lat.sk_sample()
    for k in range(10):
        sums = lat.sk(k)[0]
        assert np.isfinite(sums).all() == finite[k], k
    lat.close()


@pytest.mark.parametrize("dims", [(16, 12, 10), (1030, 3, 2)])
def test_a_captured_sample_counts_when_its_graph_runs(rf, dims):
    """Sums after reset, after the capture of a sample (nothing has run) and after
    each of three replays, eager work between them."""
    import torch
    stream = torch.cuda.Stream()
    lat = rf.Lattice(dims, kT=1e-4, seed=2, stream=stream)
    lat.init_thermal()
    lat.sk_sample()
    one = [lat.sk(f)[0] for f in range(10)]
    assert all(s.max() > 0 for s in one)
    lat.reset_sk()
    lat.sync()
    graph = torch.cuda.CUDAGraph()
    if dims[0] > 1024:  # hipFFT's way: eager samples only
        lat.sk_sample()
        for f in range(10):
            np.testing.assert_allclose(lat.sk(f)[0], one[f], rtol=1e-12)
        lat.close()
        return
    with torch.cuda.graph(graph, stream=stream):
        lat.sk_sample()
    for f in range(10):
        assert not lat.sk(f)[0].any()
    for k in range(1, 4):
        with torch.cuda.stream(stream):
            graph.replay()
        lat.moments()
        lat.sync()
        for f in range(10):
            # the same products, added in an order of their own
            np.testing.assert_allclose(lat.sk(f)[0], k * one[f], rtol=1e-12)
    lat.close()


@pytest.mark.parametrize("dims", [(128, 64, 128), (90, 96, 100), (64, 130, 61), (100, 70, 59)])
def test_blocks_that_walk_several_tiles(rf, ora, dims):
    """More tiles of columns than the 51 blocks a field of the last pass: tiles met in
    its loop, a partial one last, blocks with a tile fewer; z sides of powers of two,
    of small radices and prime."""
    nx, ny, nz = dims
    columns = 1
    while columns < 64 and nz * 2 * columns <= 4096:
        columns *= 2
    assert -(-ny * (nx // 2 + 1) // columns) > 51
    lat = rf.Lattice(dims, kT=1e-4, tau=0.8, seed=9)
    lat.init_thermal()
    lat.step(1)
    fields = lat.moments().cpu().numpy().astype(np.float64)
    fields[0] = density_deviation(lat.populations().cpu().numpy(), ora.tables()["w"])
    lat.sk_sample()
    shell = shells(dims)
    for f in range(10):
        sums, counts, _ = lat.sk(f)
        np.testing.assert_array_equal(counts, np.bincount(shell[1:], minlength=len(sums)))
        check_field(sums, fields[f], dims, shell)
    lat.close()
