"""The tile loads are inline assembly, into which the compiler does not track one documented hazard:
a scalar register that a vector instruction writes may not be read by a vector memory instruction
within five wait states.  The compiled kernels are searched for such pairs."""
import os
import re
import subprocess

import pytest

from paper_2607_12121_amd import build


def _scalars(arg):
    m = re.match(r"s\[(\d+):(\d+)\]$", arg)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", arg)
    return {int(m[1])} if m else set()


def _hazards(lines):
    """(vector memory instructions, offending pairs); a label counts as no wait state."""
    seen, bad, recent = 0, [], []
    for line in lines:
        text = line.split(";")[0].strip()
        if not text or text[0] in ".#" or text.endswith(":"):
            continue
        op, *args = [a for a in re.split(r"[ ,\t]+(?![^\[]*\])", text) if a]
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            seen += 1
            used, states = set().union(*map(_scalars, args)) if args else set(), 0
            for wait, wrote, what in reversed(recent):
                if states >= 5:
                    break
                if wrote & used:
                    bad.append((what, text))
                    break
                states += wait
        wrote = set()
        if args and op.startswith(("v_readfirstlane", "v_readlane", "v_cmp")):
            wrote = _scalars(args[0])
        elif len(args) > 1 and op.startswith("v_") and ("_co_" in op or "div_scale" in op):
            wrote = _scalars(args[1])
        nop = re.match(r"s_nop (\w+)", text)
        recent = (recent + [(int(nop[1], 0) + 1 if nop else 1, wrote, text)])[-8:]
    return seen, bad


def test_hazard_search_finds_a_planted_pair():
    near = ["v_readfirstlane_b32 s9, v1", "s_mov_b32 m0, s4", "buffer_load_dwordx4 v1, s[8:11], 0 offen lds"]
    assert len(_hazards(near)[1]) == 1
    assert _hazards(near[:1] + ["s_nop 4"] + near[1:]) == (1, [])
    assert _hazards(["v_readfirstlane_b32 s12, v1"] + near[1:]) == (1, [])


@pytest.mark.parametrize("source", ["k_attn.hip", "k_gemm.hip"])
def test_no_vector_memory_read_of_a_fresh_scalar(source, tmp_path):
    out = tmp_path / "k.s"
    subprocess.run([build.hipcc(), *[f for f in build.HIPCC_FLAGS if f != "-Wall"], "--cuda-device-only", "-S",
                    os.path.join(build.CSRC, source), "-o", str(out)], check=True, capture_output=True)
    seen, bad = _hazards(out.read_text().splitlines())
    assert seen > 500
    assert not bad, bad[:3]
