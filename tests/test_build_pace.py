"""The build's spacing of paced kernels: only s_nop lines are added, only in
functions that carry the mark and only in long basic blocks, after every
PACE-th vector instruction in a row and nowhere else; the count starts over at
a label, a branch and an instruction of another unit."""
import random

import pytest

from paper_2107_07104_amd.csrc import build as B


def _function(rng, name, marked, lines):
    out = [f"{name}:", "; %bb.0:"] + (["\t;APP", f"\t{B.MARK}"] if marked else [])
    for k in range(lines):
        r = rng.random()
        if r < 0.75:
            out.append(rng.choice(["\tv_fma_f32 v1, v2, v3, v4", "\tv_exp_f32_e32 v1, v2"]))
        elif r < 0.9:
            out.append(rng.choice(["\ts_add_u32 s0, s0, 1", "\tds_read_b32 v0, v1",
                                   "\tglobal_load_dword v0, v[2:3], off", "\tv_nop"]))
        elif r < 0.93:
            out.append(f".LBB{k}:")
        elif r < 0.96:
            out.append("\ts_cbranch_vccnz .LBB0")
        else:
            out.append("\t; comment v_add")
    return out + ["\ts_endpgm", f".Lfunc_end_{name}:"]


@pytest.mark.parametrize("lines", [0, 20, 60, 400, 3000])
@pytest.mark.parametrize("marked", [(False, False), (True, False), (True, True)])
def test_only_marked_functions_get_s_nop(lines, marked):
    rng = random.Random(lines)
    fns = [_function(rng, f"f{k}", m, lines) for k, m in enumerate(marked)]
    tail = ["\t.section meta", "v_not_code: 1"]
    src = "\n".join(sum(fns, []) + tail)
    out, n = B.pace(src)
    assert n == sum(marked)
    got = out.split("\n")
    assert [l for l in got if l != "\ts_nop 0"] == src.split("\n")
    at = 0
    for fn, m in zip(fns, marked):
        # this function's share of the output
        part = []
        for want in fn:
            while got[at] == "\ts_nop 0":
                part.append(got[at])
                at += 1
            part.append(want)
            at += 1
        if not m:
            assert part == fn
            continue
        run = 0
        for a, b in zip(part, part[1:] + [""]):
            if a.startswith("\tv_") and "v_nop" not in a:
                run += 1
                assert (b == "\ts_nop 0") <= (run == B.PACE)
                if b == "\ts_nop 0":
                    run = 0
            elif not a.startswith("\t;") and a != "\tv_nop":
                run = 0


def test_a_long_block_is_spaced_at_every_pace():
    body = ["\tv_add_f32 v0, v0, v1"] * 120
    src = "\n".join(["k:", f"\t{B.MARK}", *body, "\ts_endpgm", ".Lfunc_end0:"])
    out, _ = B.pace(src)
    assert out.count("s_nop") == 120 // B.PACE
    short = "\n".join(["k:", f"\t{B.MARK}", *body[:B.PACE_BLOCK - 1], "\ts_endpgm", ".Lfunc_end0:"])
    assert B.pace(short)[0] == short
