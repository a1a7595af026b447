"""The build's check of the assembly around the in-place multiplies: what it has to find, and that a library which fails it
does not take the place of the one before.  No compiler, no GPU."""
import pytest

from paper_2605_14305_amd import build as b


def _kernel(*body):
    return ["_ZN3fef20head_tiled256_kernelILi1EE:", *["\t" + x for x in body], "\ts_endpgm", ".Lfunc_end0:"]


def _mul(n, acc=None):
    r = f"v[{4 * n}:{4 * n + 3}]"
    return f"v_mfma_f32_16x16x32_bf16 {r}, v[100:103], v[104:107], {acc or r}"


GOOD = [_mul(0), _mul(1), _mul(2), _mul(3), "ds_read_b128 v[108:111], v90", _mul(0)]


def test_accepts():
    b.check_accumulators(_kernel(*GOOD), verbose=False)
    b.check_accumulators(_kernel("v_mov_b32_e32 v0, 0", *GOOD, "v_mul_f32_e32 v0, v0, v91"), verbose=False)
    b.check_accumulators(_kernel(*GOOD, "v_cndmask_b32_e32 v100, 0, v100, vcc", "s_nop 7", _mul(1)), verbose=False)
    b.check_accumulators(_kernel("s_cbranch_scc1 .LBB0_1", "s_endpgm", *GOOD), verbose=False)


@pytest.mark.parametrize("body, what", [
    ([_mul(0), _mul(1, "v[0:3]")], "not in place"),
    ([_mul(0), _mul(1), _mul(2), _mul(0)], "less than four"),
    ([*GOOD, "v_mov_b64_e32 v[2:3], v[92:93]", _mul(1)], "touches an accumulator"),
    ([*GOOD, "v_mov_b32_e32 v104, v92", _mul(1)], "just wrote"),
    ([*GOOD, "v_mov_b32_e32 v104, v92", "s_nop 0", _mul(1)], "just wrote"),
    (["s_endpgm", *GOOD, "v_mov_b32_e32 v1, v92", _mul(1)], "touches an accumulator"),  # behind an early end
    (["v_mov_b32_e32 v1, v92"], "no multiply"),
])
def test_finds(body, what):
    with pytest.raises(RuntimeError, match=what):
        b.check_accumulators(_kernel(*body), verbose=False)


def test_a_failed_check_leaves_the_library(tmp_path, monkeypatch):
    lib = tmp_path / "lib.so"
    lib.write_text("before")

    def run(cmd, **kw):
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("built")
    monkeypatch.setattr(b, "LIB", str(lib))
    monkeypatch.setattr(b.subprocess, "run", run)
    seen = []

    def check(verbose, extra_flags=()):
        seen.append(tuple(extra_flags))
        raise RuntimeError("found")
    monkeypatch.setattr(b, "check_accumulators_isa", check)
    with pytest.raises(RuntimeError, match="found"):
        b.build(verbose=False, extra_flags=["-DX=1"])
    assert lib.read_text() == "before" and [p.name for p in tmp_path.iterdir()] == ["lib.so"] and seen == [("-DX=1",)]
    monkeypatch.setattr(b, "check_accumulators_isa", lambda verbose, extra_flags=(): None)
    b.build(verbose=False)
    assert lib.read_text() == "built"
