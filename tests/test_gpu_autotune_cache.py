"""Which cached launch shapes a batch takes over: its own kernels' alone."""
import pytest

pytestmark = pytest.mark.gpu

DIMS = [(16, 12, 10), (20, 8, 6)]


@pytest.fixture(scope="module")
def rf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2507_08820_amd as rf
    return rf


def boxes_hash():
    h = 1469598103934665603
    for d in (x for dims in DIMS for x in dims):
        h = ((h ^ d) * 1099511628211) % 2 ** 64
    return h


def batch(rf, **kw):
    return rf.Batch([dict(dims=d, kT=1e-4) for d in DIMS], **kw)


def test_a_choice_of_other_kernels_is_not_taken_over(rf, tmp_path):
    cache = tmp_path / "tune.txt"
    # a line without the revision of the kernels
    cache.write_text(f"gfx950:s0:r7:n{len(DIMS)}:{boxes_hash():016x} 128 64 0.001\n")
    b = batch(rf)
    assert b.autotune(trial_steps=2, cache_path=cache)[1] != 64  # 64 is none of the candidates
    lines = cache.read_text().splitlines()
    assert len(lines) == 2  # timed, and appended
    # ghosts with rates of their own run another kernel
    g = batch(rf, tau_ghost=0.8)
    g.autotune(trial_steps=2, cache_path=cache)
    lines = cache.read_text().splitlines()
    assert len(lines) == 3 and len({line.split()[0] for line in lines}) == 3
    # and a choice of its own kernel is taken over as it stands
    key = lines[1].split()[0]
    cache.write_text(f"{key} 128 64 0.001\n")
    assert batch(rf).autotune(trial_steps=2, cache_path=cache)[:2] == (128, 64)
    assert len(cache.read_text().splitlines()) == 1
