"""The rules that shape the head kernels' launches (csrc/head_rules.hpp), asked through a small program for the CPU.  No GPU."""
import os
import subprocess

import pytest

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


def test_w_that_fits_the_infinity_cache_is_read_by_ordinary_loads(ask):
    short = [(17354, 4864, 2), (10577, 5056, 2), (40000, 2560, 2), (32000, 1536, 2), (50257, 2048, 2), (32000, 1024, 4),
             (32768, 4096, 2), (65536, 1024, 4)]
    longer = [(32769, 4096, 2), (65537, 1024, 4), (126464, 4096, 2), (151936, 3584, 2), (2**31 - 1, 2**31 - 64, 2)]
    assert ask([("streams_w", *s, 1, 0) for s in short + longer]) == [0] * len(short) + [1] * len(longer)


def test_rows_that_share_lines_are_read_by_ordinary_loads(ask):
    d = [1, 257, 1046, 1531, 1644, 2548, 2577, 4100, 32, 1024, 1056, 2560]
    assert ask([("streams_w", (600 << 20) // (4 * x), x, 4, 1, 0) for x in d]) == [int(x % 32 == 0) for x in d]


def test_a_w_that_row_tiles_share_is_read_by_ordinary_loads(ask):
    assert ask([("streams_w", 126464, 4096, 2, tiles, loss) for loss in (0, 1) for tiles in (1, 2, 3, 8)]) == [1, 0, 0, 0, 1, 1, 0, 0]
