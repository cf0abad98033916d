"""Wait states of the hand-written instruction blocks (gfx950): the compiler
puts none inside a block, nor between a block and the code before it.  A vector
instruction that reads a scalar register or VCC written by a vector instruction
needs two in between, a memory instruction that reads such a scalar register
five, a lane shift (DPP) two after the write of its source, and a lane read one."""
import re
import subprocess

import pytest

from paper_1512_01641_amd import build as B


def _regs(op):
    op = op.strip()
    if op == "vcc":
        return {"vcc"}
    m = re.fullmatch(r"-?\|?([sv])(\d+)\|?", op)
    if m:
        return {m[1] + m[2]}
    m = re.fullmatch(r"([sv])\[(\d+):(\d+)\]", op)
    return {m[1] + str(k) for k in range(int(m[2]), int(m[3]) + 1)} if m else set()


def _parse(line):
    """(mnemonic, written, read, wait states) of one instruction."""
    op, _, rest = line.partition(" ")
    if op == "s_nop":
        return op, set(), set(), int(rest, 0) + 1
    args = re.split(r",\s*(?![^\[]*\])", re.split(r"\s+(?:wave_shr|wave_shl|row_|quad_perm|offset|offen|bound_ctrl)", rest)[0])
    n_out = 0 if op.startswith(("ds_write", "buffer_", "global_", "s_cmp", "s_cbranch", "s_waitcnt")) else 1
    if "_co_" in op or op.startswith("v_div_scale"):
        n_out = 2
    w = set().union(*[_regs(a) for a in args[:n_out]]) if n_out else set()
    r = set().union(*[_regs(a) for a in args[n_out:]]) if args[n_out:] else set()
    if op == "v_writelane_b32":
        r |= w
    return op, w, r, 1


def hazards(text):
    """Hazards in the blocks between #ASMSTART and #ASMEND of a listing."""
    out, recent, inside = [], [], False   # recent: (vector, written, in a block, wait states after it)
    for raw in text.splitlines():
        if "#ASMSTART" in raw or "#ASMEND" in raw:
            inside = "#ASMSTART" in raw
            continue
        line = re.sub(r"\s+", " ", raw.split(";")[0].split("//")[0]).strip()
        if not line or line.startswith(".") or line.endswith(":"):
            if line.endswith(":") and not inside:
                recent = []
            continue
        op, w, r, states = _parse(line)
        vector = op.startswith("v_")
        for was_vector, written, was_inside, since in recent:
            if not (was_vector and (inside or was_inside)):
                continue
            hit = written & r
            if op.startswith(("buffer_", "global_")) and since < 5 and any(x[0] == "s" for x in hit):
                out.append("%s: %d wait states after the write of %s, 5 needed" % (line, since, sorted(hit)))
            if not vector:
                continue
            lane = op.startswith(("v_readlane", "v_readfirstlane"))
            need = 0
            if any(x == "vcc" or x[0] == "s" for x in hit):
                need = 2
            if any(x[0] == "v" and x != "vcc" for x in hit):
                need = max(need, 1 if lane else 2 if "_dpp" in op and _dpp_source(line) & hit else 0)
            if since < need:
                out.append("%s: %d wait states after the write of %s, %d needed" % (line, since, sorted(hit), need))
        recent = [(a, b, c, d + states) for a, b, c, d in recent if d + states < 5]
        recent.append((vector, w, inside, 0))
    return out


def _dpp_source(line):
    return _regs(line.split(",")[1])


def test_rules_find_each_hazard():
    def block(*lines):
        return "#ASMSTART\n" + "\n".join(lines) + "\n#ASMEND\n"
    assert hazards(block("v_cmp_eq_f32_e32 vcc, v1, v2", "v_max3_f32 v1, v2, v3, v4",
                         "v_addc_co_u32_e32 v5, vcc, v5, v5, vcc"))
    assert not hazards(block("v_cmp_eq_f32_e32 vcc, v1, v2", "s_nop 1", "v_addc_co_u32_e32 v5, vcc, v5, v5, vcc"))
    assert hazards(block("v_max3_f32 v1, v2, v3, v4", "s_nop 0", "v_add_f32_dpp v2, v1, v3 wave_shr:1 row_mask:0xf"))
    assert not hazards(block("v_max3_f32 v3, v2, v3, v4", "v_add_f32_dpp v2, v1, v3 wave_shr:1 row_mask:0xf"))
    assert hazards("v_readfirstlane_b32 s4, v1\n" + block("s_nop 3", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"))
    assert not hazards("v_readfirstlane_b32 s4, v1\n" + block("s_nop 4", "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"))
    assert hazards("v_or_b32_e32 v7, v1, v2\n" + block("v_readlane_b32 s88, v7, s3"))
    assert not hazards("v_or_b32_e32 v7, v1, v2\ns_or_b32 s1, s2, 63\n" + block("v_readlane_b32 s88, v7, s3"))


@pytest.mark.parametrize("src", ["k_align.hip", "k_expand.hip"])
def test_blocks_keep_their_wait_states(src, tmp_path):
    out = tmp_path / "listing.s"
    subprocess.run([B.HIPCC, *B.FLAGS, "-w", "-S", "--cuda-device-only", B.CSRC + "/" + src, "-o", str(out)], check=True,
                   capture_output=True)
    text = out.read_text()
    assert text.count("#ASMSTART") > 0
    found = hazards(text)
    assert not found, "\n".join(found[:8])
