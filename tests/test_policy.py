"""CPU checks of the rules that pick a kernel by size (csrc/policy.hpp, plain host
code): measured boxes on both sides of each line."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_08820_amd", "csrc")


@pytest.fixture(scope="module")
def evaluate(tmp_path_factory):
    """Values of C++ expressions over policy.hpp, as integers."""
    tmp = tmp_path_factory.mktemp("policy")

    def run(expressions):
        src = tmp / "probe.cpp"
        lines = "\n".join(f'  std::printf("%lld\\n", static_cast<long long>({e}));' for e in expressions)
        src.write_text(f"#include <cstdio>\n#include \"policy.hpp\"\nusing namespace rflbm;\nint main() {{\n{lines}\n}}\n")
        exe = tmp / "probe"
        subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
        return [int(v) for v in subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()]

    return run


def test_structure_factor_route(evaluate):
    """Boxes whose transforms in LDS were faster than hipFFT's, and slower ones."""
    own = [(2, 2, 2), (256, 256, 256), (512, 512, 512), (1000, 100, 50), (100, 100, 100), (17, 19, 23), (61, 61, 61),
           (101, 101, 101), (72, 72, 199), (64, 251, 64), (251, 64, 64), (509, 45, 45), (8, 8, 509), (2, 1021, 2),
           (122, 122, 64), (61, 256, 256), (143, 143, 143), (187, 187, 187), (209, 209, 209), (238, 238, 238),
           (255, 255, 255), (363, 363, 363), (256, 286, 256), (222, 222, 222), (212, 212, 212), (348, 348, 348),
           (406, 406, 406), (183, 183, 183), (305, 305, 305)]
    hipfft = [(1030, 3, 2), (2, 2, 2048), (1021, 2, 2), (509, 8, 8), (1021, 32, 32), (32, 1021, 32), (32, 32, 1021),
              (45, 45, 331), (45, 45, 509), (2, 1021, 509), (509, 2, 1021), (26, 199, 199), (38, 701, 38),
              (134, 96, 90), (137, 149, 151), (242, 242, 242), (260, 260, 260), (286, 286, 286), (374, 374, 374),
              (520, 520, 130), (272, 544, 136), (286, 256, 256), (256, 256, 286), (236, 236, 236), (244, 244, 244),
              (344, 344, 344), (366, 366, 366), (488, 488, 488)]
    got = evaluate([f"sk_fits({x}, {y}, {z})" for x, y, z in own + hipfft])
    assert [d for d, g in zip(own + hipfft, got) if g != (d in own)] == []


def test_largest_prime(evaluate):
    def prime(n):
        return max(d for d in range(2, n + 1) if n % d == 0 and all(d % k for k in range(2, d)))
    assert evaluate([f"largest_prime({n})" for n in range(2, 200)]) == [prime(n) for n in range(2, 200)]


def test_reads_past_the_caches(evaluate):
    """Even step counts, beyond 256 MiB, rows of whole 128-byte lines."""
    def q(dims, size, odd=0):
        return f"read_streams({dims[0] * size}, {27 * dims[0] * dims[1] * dims[2] * size}ull, {odd})"
    yes = [((192, 192, 192), 4), ((256, 256, 256), 2), ((96, 256, 256), 4), ((288, 256, 256), 4)]
    no = [((128, 128, 128), 4), ((255, 256, 200), 2), ((255, 256, 200), 4), ((288, 256, 256), 2), ((200, 200, 200), 4),
          ((1000, 64, 100), 4), ((16, 512, 512), 4), ((8, 1024, 600), 4), ((192, 192, 192), 4, 1)]
    assert evaluate([q(*c) for c in yes + no]) == [1] * len(yes) + [0] * len(no)


MIB = 1 << 20


def test_batches(evaluate):
    """(populations, row lengths in bytes, FP32, sampled step, largest replica):
    default or non-temporal even steps, ranges or turns, as measured."""
    cases = [  # MiB, gcd of the rows, f32, stats, nodes of the largest, blocks a tile -> nt, ranges
        ((7, 80, 1, 0, 20 ** 3, 0), (0, 1)), ((216, 256, 1, 0, 64 ** 3, 0), (0, 1)), ((216, 256, 0, 0, 128 ** 3, 0), (0, 1)),
        ((273, 384, 1, 0, 96 ** 3, 0), (1, 0)), ((273, 384, 1, 1, 96 ** 3, 0), (1, 0)), ((304, 128, 1, 0, 32 ** 3, 0), (1, 0)),
        ((296, 192, 1, 0, 48 ** 3, 0), (0, 1)), ((683, 192, 1, 0, 48 ** 3, 0), (1, 0)), ((309, 400, 1, 0, 10 ** 6, 0), (0, 1)),
        ((1236, 400, 1, 0, 10 ** 6, 0), (0, 0)), ((937, 520, 1, 1, 455000, 0), (0, 0)), ((864, 512, 1, 0, 128 ** 3, 0), (1, 0)),
        ((864, 512, 1, 0, 128 ** 3, 1), (1, 0)), ((2223, 64, 1, 0, 96 ** 3, 0), (1, 0)), ((2223, 64, 1, 0, 96 ** 3, 1), (1, 1)),
        ((1304, 64, 1, 0, 96 ** 3, 1), (1, 0)), ((432, 256, 0, 0, 128 ** 3, 0), (1, 0)), ((432, 256, 0, 1, 128 ** 3, 1), (1, 0)),
        ((540, 128, 0, 0, 64 ** 3, 0), (1, 0)), ((1111, 32, 0, 0, 96 ** 3, 0), (0, 0)), ((1111, 32, 0, 1, 96 ** 3, 0), (1, 0)),
        ((1458, 192, 0, 0, 96 ** 3, 1), (0, 0)), ((618, 200, 0, 0, 10 ** 6, 0), (0, 0)), ((618, 200, 0, 1, 10 ** 6, 0), (0, 0)),
        ((824, 400, 0, 1, 200 ** 3, 0), (1, 0)), ((300, 360, 0, 1, 180 ** 3, 0), (1, 1)), ((307, 576, 1, 1, 144 ** 3, 0), (1, 1)),
        ((307, 576, 1, 0, 144 ** 3, 0), (0, 1)), ((296, 192, 1, 1, 48 ** 3, 0), (0, 1)), ((141, 260, 0, 0, 455000, 0), (0, 1)),
    ]
    got = evaluate([e for (mb, rows, f32, stats, n, tile), _ in cases for e in (
        f"batch_even_nt({mb * MIB}ull, {rows}, {f32}, {stats}, {n})",
        f"batch_in_ranges({mb * MIB}ull, {rows}, {f32}, {tile})")])
    assert [c for c, a, b in zip(cases, got[::2], got[1::2]) if (a, b) != c[1]] == []


TILES, FLAT, ROWS, WAVES = range(4)
BYTES = {"f32": 4, "f16": 2}


def box(dims, storage, noise, row_blocks=1, in_turn=0):
    """StepBox of a box by itself (or of `in_turn` MiB stepped in turn)."""
    size = 27 * dims[0] * dims[1] * dims[2] * BYTES[storage]
    return (f"StepBox{{{dims[0]}u, {BYTES[storage]}u, {str(bool(noise)).lower()}, {str(bool(row_blocks)).lower()}, "
            f"{str(size < 1 << 32).lower()}, {str(in_turn > 0).lower()}, {in_turn * MIB if in_turn else size}ull}}")


def routes(evaluate, cases):
    """Cases (dims, storage, noise, odd, stats) whose route is not the one given."""
    got = evaluate([f"step_route({box(d, s, n)}, {odd}, {st})" for (d, s, n, odd, st), _ in cases])
    return [(c, g) for c, g in zip(cases, got) if g != c[1]]


def test_rows_that_do_not_fill_waves(evaluate):
    cases = []
    for odd in (0, 1):
        for stats in (0, 1):
            flat = [((130, 50, 70), "f32"), ((17, 19, 23), "f32"), ((63, 128, 128), "f32"), ((48, 200, 220), "f32"),
                    ((96, 256, 256), "f32"), ((32, 512, 512), "f32"), ((30, 500, 500), "f32"), ((464, 120, 120), "f32"),
                    ((352, 256, 128), "f32"), ((1000, 80, 80), "f32"), ((255, 256, 200), "f32"), ((1270, 64, 64), "f32"),
                    ((40, 400, 400), "f16"), ((63, 300, 240), "f16"), ((1008, 110, 110), "f16"), ((2000, 80, 80), "f16")]
            tiles = [((63, 300, 140), "f32"), ((33, 320, 320), "f32"), ((48, 300, 300), "f32"), ((480, 120, 120), "f32"),
                     ((736, 100, 96), "f32"), ((2016, 48, 48), "f32"), ((1264, 64, 64), "f32"), ((56, 300, 340), "f16"),
                     ((63, 300, 280), "f16"), ((350, 350, 350), "f32")]
            cases += [((d, s, noise, odd, stats), FLAT) for d, s in flat for noise in (0, 1)]
            cases += [((d, s, noise, odd, stats), TILES) for d, s in tiles for noise in (0, 1)]
    assert routes(evaluate, cases) == []
    assert evaluate([f"step_route({box((130, 50, 70), 'f32', 1, row_blocks=0)}, 0, 0)"]) == [TILES]


def test_streamed_flat_blocks(evaluate):
    yes = [((96, 256, 256), "f32"), ((160, 160, 100), "f32"), ((416, 200, 200), "f32"), ((16, 700, 700), "f32"),
           ((464, 120, 120), "f32"), ((1040, 80, 80), "f32")]
    no = [((96, 200, 110), "f32"), ((300, 200, 100), "f32"), ((255, 256, 200), "f32"), ((40, 400, 400), "f32"),
          ((96, 256, 256), "f16"), ((300, 280, 260), "f16")]
    assert evaluate([f"step_streams({box(d, s, 1)})" for d, s in yes + no]) == [1] * len(yes) + [0] * len(no)


def test_rows_of_whole_waves(evaluate):
    cases = []
    for d in [(64, 64, 64), (256, 256, 256), (1024, 64, 64), (320, 96, 96)]:
        for s, noise in (("f32", 1), ("f32", 0), ("f16", 0)):
            cases += [((d, s, noise, 0, 0), WAVES), ((d, s, noise, 1, 0), ROWS), ((d, s, noise, 0, 1), ROWS),
                      ((d, s, noise, 1, 1), ROWS)]
    for odd in (0, 1):
        cases += [(((192, 192, 192), "f16", 1, odd, 0), WAVES), (((320, 96, 96), "f16", 1, odd, 0), WAVES),
                  (((256, 128, 128), "f16", 1, odd, 0), WAVES), (((256, 256, 256), "f16", 1, odd, 0), TILES),
                  (((192, 192, 192), "f16", 1, odd, 1), TILES)]
    assert routes(evaluate, cases) == []


def test_rows_longer_than_a_block(evaluate):
    """Odd steps in tiles or waves, even ones in waves, streamed beyond 256 MiB."""
    tiles = [((1280, 64, 64), "f32"), ((1152, 96, 96), "f32"), ((1920, 64, 22), "f32"), ((2048, 16, 16), "f32"),
             ((2048, 64, 64), "f16"), ((1280, 64, 64), "f16"), ((1792, 48, 64), "f16")]
    waves = [((1088, 64, 64), "f32"), ((1216, 64, 64), "f32"), ((4160, 16, 64), "f32"), ((1088, 64, 64), "f16"),
             ((2048, 32, 64), "f16"), ((1920, 64, 96), "f16")]
    cases = [((d, s, 0, 1, 0), TILES) for d, s in tiles] + [((d, s, 0, 1, 0), WAVES) for d, s in waves]
    cases += [((d, s, 0, 0, 0), WAVES) for d, s in tiles + waves] + [((d, s, 0, 0, 1), TILES) for d, s in tiles + waves]
    assert routes(evaluate, cases) == []
    yes = [((1280, 64, 32), "f32", 1), ((1280, 64, 64), "f16", 0), ((256, 128, 96), "f32", 1), ((2048, 64, 64), "f32", 0)]
    no = [((1088, 64, 32), "f32", 1), ((1280, 64, 56), "f16", 0), ((256, 128, 88), "f32", 1), ((1024, 64, 46), "f32", 1),
          ((256, 256, 92), "f16", 0)]
    assert evaluate([f"step_streams({box(*c)})" for c in yes + no]) == [1] * len(yes) + [0] * len(no)


def test_16_bit_steps_with_noise_stream_from_the_size_of_the_cache(evaluate):
    yes = [((256, 256, 80), "f16", 1), ((192, 192, 140), "f16", 1), ((256, 256, 256), "f16", 1)]
    no = [((256, 256, 72), "f16", 1), ((192, 192, 128), "f16", 1), ((256, 256, 80), "f16", 0), ((256, 128, 80), "f32", 1)]
    assert evaluate([f"step_streams({box(*c)})" for c in yes + no]) == [1] * len(yes) + [0] * len(no)
    cases = [(((256, 256, 80), "f16", 1, odd, 0), TILES) for odd in (0, 1)]
    cases += [(((256, 256, 72), "f16", 1, odd, 0), WAVES) for odd in (0, 1)]
    assert routes(evaluate, cases) == []


def test_blocks_a_cu_is_held_to(evaluate):
    """Memory-bound steps that stream from memory; not in the cache, with noise in 16
    bits, or in long rows of an odd number of waves."""
    f32 = [((64, 512, 512), 20, 16), ((128, 301, 299), 20, 8), ((192, 256, 300), 20, 5), ((256, 256, 256), 20, 4),
           ((384, 207, 247), 20, 2), ((448, 111, 87), 20, 2), ((512, 256, 128), 20, 2), ((640, 200, 160), 20, 2),
           ((1024, 61, 53), 20, 2), ((1280, 64, 64), 20, 2), ((4096, 32, 24), 20, 2)]
    free = [(704, 100, 120), (960, 60, 61), (1088, 64, 64), (128, 128, 128), (64, 64, 64), (64, 64, 32), (130, 150, 150),
            (192, 100, 150)]
    f16 = [((64, 512, 512), 16, 20), ((128, 299, 397), 16, 10), ((192, 256, 300), 16, 6), ((256, 256, 256), 16, 0),
           ((384, 207, 247), 16, 0), ((1280, 100, 100), 16, 0), ((2048, 64, 96), 16, 0)]
    cases = [((d, "f32", noise), w, r) for d, w, r in f32 for noise in (0, 1)]
    cases += [((d, "f32", noise), 0, 0) for d in free for noise in (0, 1)] + [((d, "f16", 0), 0, 0) for d in free[3:]]
    cases += [(((320, 256, 200), "f32", 0), 20, 3), (((576, 150, 150), "f32", 0), 20, 2),
              (((320, 256, 200), "f32", 1), 0, 0), (((576, 150, 150), "f32", 1), 0, 0)]
    cases += [((d, "f16", 0), w, r) for d, w, r in f16] + [((d, "f16", 1), 0, 0) for d, _, _ in f16]
    got = evaluate([f"step_blocks({box(*c)}).{k}" for c, _, _ in cases for k in ("waves", "rows")])
    assert [c for c, w, r in zip(cases, got[::2], got[1::2]) if (w, r) != c[1:]] == []
    assert evaluate([f"step_blocks({box((64, 64, 64), 'f32', 1, in_turn=270)}).waves"]) == [20]


def test_small_boxes(evaluate):
    """Memory-bound steps of 6 to 18.5 MiB, in FP32 with noise 4 to 24."""
    yes = [((64, 64, 64), "f16", 0), ((64, 64, 32), "f16", 0), ((1280, 16, 16), "f16", 0), ((4096, 8, 8), "f16", 0),
           ((64, 64, 28), "f32", 0), ((64, 64, 32), "f32", 1), ((128, 32, 16), "f32", 1), ((192, 64, 16), "f32", 1),
           ((64, 64, 48), "f32", 1), ((320, 21, 25), "f32", 0), ((512, 21, 31), "f16", 0), ((128, 28, 60), "f32", 1)]
    no = [((64, 64, 16), "f16", 0), ((64, 64, 88), "f16", 0), ((64, 64, 64), "f16", 1), ((64, 64, 32), "f16", 1),
          ((2048, 16, 16), "f16", 0), ((63, 64, 64), "f16", 0), ((64, 64, 64), "f32", 0), ((64, 64, 44), "f32", 0),
          ((64, 64, 64), "f32", 1), ((64, 64, 6), "f32", 1), ((64, 64, 12), "f32", 0), ((63, 64, 32), "f32", 1)]
    assert evaluate([f"step_streams({box(*c)})" for c in yes + no]) == [1] * len(yes) + [0] * len(no)
    assert routes(evaluate, [(((1280, 16, 16), "f16", 0, 1, 0), TILES), (((2048, 16, 16), "f16", 0, 1, 0), WAVES)]) == []


def test_boxes_stepped_in_turn(evaluate):
    """The size that counts is that of all of them, streamed from 256 MiB."""
    got = evaluate([f"step_streams({box((64, 64, 64), 'f32', 1, in_turn=mb)})" for mb in (54, 216, 270, 432)])
    assert got == [0, 0, 1, 1]


def test_one_thread_a_node(evaluate):
    """Every box below 2^32 nodes in a launch that HIP takes (fewer than 2^32 threads
    along an axis)."""
    for n in (1, 255, 256, 257, 512 ** 3, 2 ** 31, 2 ** 31 + 1, 2 ** 32 - 257, 2 ** 32 - 256, 2 ** 32 - 255, 2 ** 32 - 1):
        x, y = evaluate([f"node_grid({n}ull).x", f"node_grid({n}ull).y"])
        assert x * 256 < 2 ** 32 and y < 2 ** 16 and x * y * 256 >= n and x * (y - 1) * 256 < n
