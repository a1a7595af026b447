"""The rules that shape the head kernels' launches (csrc/head_rules.hpp), asked through a small program for the CPU.  No GPU."""
import os
import subprocess

import pytest

from paper_2605_14305_amd import binding as fb
import test_gpu_f32_head as f32_head
import test_gpu_runs as gpu_runs
import test_gpu_shares as shares

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask(lines): the rules' answers, one integer per line."""
    exe = str(tmp_path_factory.mktemp("rules") / "head_rules")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", os.path.join(HERE, "c_abi", "head_rules.cpp"), "-o", exe], check=True)

    def run(lines):
        r = subprocess.run([exe], input="\n".join(" ".join(map(str, l)) for l in lines), text=True, capture_output=True, check=True)
        return [int(x) for x in r.stdout.split()]
    return run


def test_w_of_which_the_infinity_cache_keeps_some_is_read_by_ordinary_loads(ask):
    short = [(17354, 4864, 2), (10577, 5056, 2), (40000, 2560, 2), (32000, 1536, 2), (50257, 2048, 2), (32000, 1024, 4),
             (32768, 4096, 2), (65536, 1024, 4), (36864, 4096, 2), (73728, 1024, 4)]
    longer = [(36865, 4096, 2), (73729, 1024, 4), (126464, 4096, 2), (151936, 3584, 2), (2**31 - 1, 2**31 - 64, 2)]
    assert ask([("streams_w", *s, 1, 0) for s in short + longer]) == [0] * len(short) + [1] * len(longer)


def test_rows_that_share_lines_are_read_by_ordinary_loads(ask):
    d = [1, 257, 1046, 1531, 1644, 2548, 2577, 4100, 32, 1024, 1056, 2560]
    assert ask([("streams_w", (600 << 20) // (4 * x), x, 4, 1, 0) for x in d]) == [int(x % 32 == 0) for x in d]


def test_a_w_that_row_tiles_share_is_read_by_ordinary_loads(ask):
    assert ask([("streams_w", 126464, 4096, 2, tiles, loss) for loss in (0, 1) for tiles in (1, 2, 3, 8)]) == [1, 0, 0, 0, 1, 1, 0, 0]


LAUNCHES = [(33, 128, 64, 128), (33, 256, 64, 256), (257, 4096, 96, 256)]  # rows from, to, least, most


def _rounds(n_tiles, row_tiles):
    """Rounds of the busiest XCD: token tile t and all its row tiles run on XCD t % 8, one workgroup on each of 32 CUs."""
    per_xcd = [0] * 8
    for t in range(n_tiles):
        per_xcd[t % 8] += row_tiles
    return -(-max(per_xcd) // 32)


def _height(M, m, unit=32):
    return -(-(-(-M // m)) // unit) * unit


@pytest.mark.parametrize("d", [512, 1024, 1088, 4096])
def test_more_row_tiles_only_where_the_busiest_xcd_gains(ask, d):
    for first, last, least, most in LAUNCHES:
        tiles = [*range(1, 70, 3), 97, 128, 187, 250, 256, 301, 391]
        sizes = [(M, n) for M in range(first, last + 1, 1 if last <= 256 else 37) for n in tiles]
        picked = ask([("row_tiles", M, n, d, least, most) for M, n in sizes])
        for (M, n), m in zip(sizes, picked):
            fewest = -(-M // most)
            assert m >= fewest and _height(M, m) <= most and (m - 1) * _height(M, m) < M  # no row tile without rows
            if m > fewest:
                assert _height(M, m) >= least
                assert _rounds(n, m) * (_height(M, m) + 64) < _rounds(n, fewest) * (_height(M, fewest) + 64)


def test_row_tiles_of_calls_that_were_measured(ask):
    # rows, token tiles, d, least, most; what more row tiles (10 -> 14 and so on) made slower
    slower = [(2310, 18, 4608, 96, 256), (432, 50, 6016, 96, 256), (7676, 2, 576, 96, 256), (484, 187, 3712, 96, 256),
              (144, 117, 3968, 64, 256), (384, 173, 3584, 96, 256), (256, 310, 5312, 64, 256)]
    assert ask([("row_tiles", *r) for r in slower]) == [10, 4, 30, 2, 1, 2, 1]
    faster = [(1596, 32, 1984, 96, 256), (1422, 70, 1088, 96, 256), (2214, 69, 3392, 96, 256), (2870, 95, 1472, 96, 256),
              (256, 33, 1024, 64, 256), (528, 63, 3072, 96, 256), (256, 63, 1024, 64, 256), (128, 125, 4096, 64, 128)]
    assert ask([("row_tiles", *r) for r in faster]) == [8, 7, 10, 13, 4, 4, 4, 2]
    assert ask([("row_tiles", 300, 197, 2048, 96, 256), ("row_tiles", 2048, 494, 4096, 96, 256)]) == [2, 8]


def test_cross_entropy_in_eight_wavefronts_where_they_are_ahead(ask):
    calls = {(300, 2, 2048): 1, (300, 2, 4096): 1, (384, 2, 4096): 1, (440, 2, 3072): 1, (512, 2, 3072): 1, (700, 3, 1024): 1, (2048, 8, 512): 1,
             (385, 2, 3136): 0, (512, 2, 3584): 0, (450, 2, 4352): 0, (300, 2, 4160): 0, (700, 3, 1088): 0, (2048, 8, 4096): 0, (300, 3, 2048): 0}
    assert ask([("loss_takes_eight_wavefronts", *c) for c in calls]) == list(calls.values())


def test_fp32_row_tiles_only_where_the_busiest_cu_gains(ask):
    def work(M, n, m):
        workgroups = -(-n * m // 256) if n < 64 else _rounds(n, m)
        return workgroups * (_height(M, m, 16) + 16) + 24 * (workgroups == 1 and _height(M, m, 16) >= 48)
    sizes = [(M, n) for M in [*range(1, 200), 347, 512, 1000, 4000, 65535] for n in [*range(1, 130, 3), 187, 250, 256, 301, 500, 2000, 1 << 25]]
    for (M, n), m in zip(sizes, ask([("f32_row_tiles", *s) for s in sizes])):
        fewest = -(-M // 64)
        assert fewest <= m <= -(-M // 16)
        assert m == fewest or work(M, n, m) < work(M, n, fewest)
    # rows and token tiles of calls that were slower in 3, 8, 4 and 3 row tiles, and of one that was slower in one than in two
    assert ask([("f32_row_tiles", *s) for s in [(113, 117), (347, 33), (162, 65), (100, 92), (60, 146)]]) == [4, 11, 6, 4, 2]
    assert ask([("f32_row_tiles", *s) for s in [(32, 79), (64, 125), (48, 284), (16, 500), (32, 500)]]) == [2, 2, 1, 1, 1]


def test_what_the_gpu_tests_at_the_line_for_non_temporal_loads_run(ask):
    (V0, d0), (V1, d1) = shares.LINE_OF_A_ROUND
    assert ask([("streams_w", V0, d0, 2, 1, 0), ("streams_w", V1, d1, 2, 1, 0)]) == [0, 1]
    for variant, rows in shares.ROUNDS_AT_THE_LINE:
        unit, per = {fb.FEF_GEMM_STREAM: (64, 4), fb.FEF_GEMM_ROWSTREAM: (16, 8)}.get(variant, (256, 1))
        most = 256 if variant == fb.FEF_GEMM_TILED256 else 128
        for V in (V0, V1):
            tiles = -(-V // unit) if per == 1 else min(256, -(-(-(-V // unit)) // per))
            assert ask([("row_tiles", M, tiles, d0, 64, most) for M in rows]) == [1] * len(rows)
        assert {_height(M, 1) for M in rows} == set(range(32, most + 1, 32))
    for V, (below, above), rows in shares.LINES_OF_A_LOSS:
        whole = -(-V // 256) % 256 > 200  # else shares of the vocabulary, one row tile
        tiles = [ask([("row_tiles", R, -(-V // 256), d, 64 if R <= 256 else 96, 256) for R in rows]) if whole else [1] * len(rows)
                 for d in (below, above)]
        assert tiles == [[-(-R // 256) for R in rows]] * 2
        for t in set(tiles[0]):
            assert ask([("streams_w", V, d, 2, t, 1) for d in (below, above)]) == [0, 1]
        if whole:
            every = {(1, h) for h in range(32, 257, 32)} | {(2, h) for h in range(160, 257, 32)}
            assert {(t, _height(R, t)) for R, t in zip(rows, tiles[0])} == every


def test_what_the_gpu_tests_of_the_fp32_head_run(ask):
    def line(test, name):
        return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == name)
    sizes = line(f32_head.test_f32_to_either_side_of_the_line_for_non_temporal_loads, "d,V")
    assert ask([("streams_w", V, d, 4, 1, 0) for d, V in sizes]) == [0, 1, 1, 0, 0]
    assert all(ask([("f32_row_tiles", M, -(-V // 64)) for M in (16, 32, 48, 64)]) == [1] * 4 for _, V in sizes)
    def heights(rows):
        return {_height(M, m, 16) for M, m in zip(rows, ask([("f32_row_tiles", M, 512) for M in rows]))}
    assert heights((34, 48, 50, 64, 98, 130)) == {48, 64} and heights((16, 18, 32, 34)) == {16, 32, 48}  # the tests of steps


def test_which_of_the_two_kernels_up_to_32_rows(ask):
    sizes = {(32768, 4096): 0, (32769, 4096): 1, (32769, 1024): 1, (65536, 1024): 1, (65537, 1024): 0, (147456, 1024): 0, (147457, 1024): 1,
             (1, 512): 0, (2**31 - 1, 512): 1, (100003, 512): 1, (100003, 2048): 1}
    assert ask([("slices_serve", *s) for s in sizes]) == list(sizes.values())


def test_where_h_in_lds_falls_behind(ask):
    """Calls that the kernel with H in LDS made slower, and the nearest ones that it does not."""
    behind = [(65537, 512), (81920, 512), (65153, 1024), (65536, 1024), (65537, 2048), (73728, 2048)]
    others = [(65536, 512), (81921, 512), (131072, 512), (65152, 1024), (65536, 2048), (73729, 2048), (70000, 2560), (70000, 4096)]
    assert ask([("slices_lag", *s) for s in behind + others]) == [1] * len(behind) + [0] * len(others)
    assert ask([("slices_serve", *s) for s in others]) == [1] * len(others)


def test_which_runs_are_walked_in_one(ask):
    short = {(16, 128, 1024): 1, (16, 129, 1024): 0, (64, 128, 1024): 0, (16, 96, 512): 1, (16, 112, 512): 0}
    assert ask([("short_runs_serve", *s) for s in short]) == list(short.values())
    lag = {(2, 160, 1024): 1, (64, 256, 1024): 1, (64, 159, 1024): 0, (65, 256, 1024): 0, (64, 256, 1536): 0}  # rows, runs, d
    assert ask([("short_runs_lag", *s) for s in lag]) == list(lag.values())
    # rows of a tile, longest run, d; the last row: calls that were slower in one walk
    double = {(64, 256, 512): 0, (64, 257, 512): 1, (128, 512, 1024): 1, (40, 384, 1024): 1, (40, 448, 1024): 0, (64, 320, 4096): 1, (64, 384, 4096): 0,
              (110, 448, 2560): 1, (110, 449, 2560): 0,
              (128, 320, 3584): 0, (40, 512, 4096): 0, (110, 512, 2048): 0}
    assert ask([("double_runs_serve", *s) for s in double]) == list(double.values())


def test_pieces_of_short_vocabularies(ask):
    def shape(M, V, d, unit):
        runs = -(-V // 256) if unit == 256 else min(256, -(-(-(-V // unit)) // (4 if unit == 64 else 8)))
        return ask([("piece_shape", M, V, d, runs, unit)])
    for M, V, d, unit in [(64, 16385, 4096, 64), (257, 8000, 4096, 256), (8, 4000, 2112, 64), (16, 6000, 1024, 64), (65, 8193, 1024, 64), (64, 12289, 1024, 64),
                          (129, 6000, 1216, 256), (192, 12289, 4096, 256), (193, 12289, 2048, 256), (192, 10241, 2048, 256), (256, 9000, 1536, 256), (64, 4000, 448, 64)]:
        assert shape(M, V, d, unit) == [0, 0, 0, 0], (M, V, d)
    for unit in (16, 64, 256):
        for M in (9, 33, 64, 65, 128, 129, 256) if unit == 256 else (9, 33, 64, 65, 128):
            for V in (1, 15, 64, 65, 777, 5000, 8437, 12288) + ((16384,) if M != 129 else ()):
                pieces, tokens, rows, tiles = shape(M, V, 4096, unit)
                assert tokens in (64, 128) and rows in (64, 128) and tiles == -(-M // rows)      # the instantiations
                assert pieces * tokens == (128 if unit == 16 else 256)                           # longest run: no token is left out
    for call in [(128, 16384, 1280, 64), (64, 12288, 512, 64), (128, 8192, 512, 64), (256, 8192, 1280, 256), (256, 16384, 2560, 256), (192, 12288, 2560, 256),
                 (9, 5120, 512, 64)]:
        assert shape(*call)[0], call
    # calls that pieces made slower, and their nearest neighbours that they do not
    for M, V, d, pays in [(193, 8193, 1792, 0), (224, 12288, 2496, 0), (192, 8193, 1792, 1), (225, 12288, 2496, 1), (224, 8192, 1792, 1), (224, 8193, 2560, 1),
                          (193, 4097, 960, 0), (256, 5120, 512, 0), (256, 4096, 512, 1), (192, 5120, 512, 1), (256, 5120, 1024, 1)]:
        assert bool(shape(M, V, d, 256)[0]) == bool(pays), (M, V, d)


UNITS = {fb.FEF_GEMM_STREAM: 64, fb.FEF_GEMM_ROWSTREAM: 16, fb.FEF_GEMM_TILED256: 256}


def _runs(V, unit):
    return -(-V // 256) if unit == 256 else min(256, -(-(-(-V // unit)) // (4 if unit == 64 else 8)))


def _kernel(ask, variant, M, d, V):
    """Which kernel or form of the tile kernel a round over M rows takes."""
    if variant == fb.FEF_GEMM_SKINNY:
        return "lds" if ask([("slices_serve", V, d)]) == [1] and ask([("slices_lag", V, d)]) == [0] else "registers"
    unit = UNITS[variant]
    n = _runs(V, unit)
    pieces, tokens, rows, _ = ask([("piece_shape", M, V, d, n, unit)])
    if pieces:
        return ("pieces", unit, tokens, rows)
    if unit == 256:
        return ("tiles", unit)
    longest, m = -(-(-(-V // unit)) // n) * unit, ask([("row_tiles", M, n, d, 64, 128)])[0]
    if ask([("short_runs_serve", unit, longest, d)]) == [1] and ask([("short_runs_lag", M, n, d)]) == [0]:
        return ("short", unit)
    return ("double" if ask([("double_runs_serve", -(-M // m), longest, d)]) == [1] else "tiles", unit)


def test_what_the_gpu_tests_of_runs_and_pieces_run(ask):
    shapes = {_kernel(ask, variant, M, d, V) for variant, d, V, rows in gpu_runs.PIECES for M in rows}
    assert shapes == {("pieces", unit, 64, rows) for unit in (16, 64, 256) for rows in (64, 128)} | {("pieces", 256, 128, 64), ("pieces", 256, 128, 128)}
    # no other shape exists: that is all that head_runs.hip instantiates
    grid = [(M, V, d, _runs(V, unit), unit) for unit in (16, 64, 256) for M in range(1, 257 if unit == 256 else 129, 5) for V in range(1, 16385, 241)
            for d in (512, 1280, 2560, 4096)]
    answers = ask([("piece_shape", *q) for q in grid])
    assert {("pieces", q[4], answers[4 * i + 1], answers[4 * i + 2]) for i, q in enumerate(grid) if answers[4 * i]} <= shapes
    assert {_kernel(ask, v, M, 4096, V) for v, rows in shares.TILES_AT_THE_LINE for M in rows for V in (36864, 36865)} == {("tiles", 64), ("tiles", 16)}
    forms = {name: _kernel(ask, *call) for name, call in shares.BANNED.items()}
    assert forms == {"tiles, runs of 64": ("tiles", 64), "tiles, runs of 16": ("tiles", 16), "short runs": ("short", 16),
                     "double runs of 64": ("double", 64), "double runs of 16": ("double", 16), "pieces of 128": ("pieces", 256, 128, 128),
                     "H in registers": "registers", "H in registers, 32 rows": "registers", "H in LDS": "lds", "H in LDS, 32 rows": "lds",
                     "H in LDS, from any slice": "lds", "H in LDS, two tiles": "lds"}


def test_losses_with_all_rows_in_one_row_tile(ask):
    calls = {(256, 50257): 0, (257, 50257): 1, (304, 57344): 1, (304, 57345): 0, (305, 49152): 1, (305, 49153): 0, (320, 45057): 1, (320, 45056): 0, (321, 46000): 0}
    assert ask([("loss_wide_serves", *c) for c in calls]) == list(calls.values())
