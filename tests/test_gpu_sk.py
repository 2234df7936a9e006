"""Structure factor over the lengths its transforms distinguish: powers of two,
the radices 3, 5 and 7, other primes (as a factor and as the whole length), odd
and even sides, the smallest box, tiles of every width, and the sides that go to
hipFFT; both parities of the stored layout."""
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


BOXES = [(2, 3, 2), (4, 2, 5), (16, 16, 16), (64, 8, 32), (17, 19, 23), (30, 42, 7), (55, 36, 20), (97, 6, 13),
         (6, 61, 128), (256, 9, 4), (5, 512, 3), (3, 4, 1024), (1024, 2, 3), (1030, 3, 2), (134, 96, 90)]


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("dims", BOXES)
def test_shell_sums_match_fp64_transforms(rf, dims, storage):
    """Against numpy's FP64 transform of the moments read from the GPU.  Both the
    fields (read as FP32; rho with its mean, 2^-24 of 1 against fluctuations of
    1e-2) and the transform round at 2^-24 per operation: 2e-5 of a shell's sum
    as in the step tests, and of the field's mean shell where a shell is empty."""
    nx, ny, nz = dims
    lat = rf.Lattice(dims, storage=storage, kT=1e-4, tau=0.8, seed=9)
    lat.init_thermal()
    k = [np.fft.fftfreq(n, 1.0 / n) for n in (nz, ny, nx)]
    shell = np.rint(np.sqrt(k[0][:, None, None] ** 2 + k[1][None, :, None] ** 2 + k[2] ** 2)).astype(int).ravel()
    shell[0] = -1
    for steps in (0, 1):  # parities 0 and 1
        lat.step(steps)
        lat.reset_sk()
        lat.sk_sample()
        lat.sk_sample()
        m = lat.moments().cpu().numpy().astype(np.float64).reshape(10, nz, ny, nx)
        m[0] -= 1.0
        for f in range(10):
            p = (np.abs(np.fft.fftn(m[f])) ** 2 / lat.n).ravel()
            sums, counts, samples = lat.sk(f)
            want = np.bincount(shell[1:], p[1:], minlength=len(sums))
            assert samples == 2
            np.testing.assert_array_equal(counts, np.bincount(shell[1:], minlength=len(sums)))
            np.testing.assert_allclose(sums, 2 * want, rtol=2e-5, atol=2e-5 * want.mean())
    lat.close()
