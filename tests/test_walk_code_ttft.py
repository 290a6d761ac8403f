"""The minimum-TTFT walk's block of 16 depth steps, checked as the other rule's
is: on the gfx950 code object that the library's flags produce, every computed
entry must be the first instruction of its step, and the back-edge must return
to step 0."""
import os
import re

import paper_2602_06502_amd._build as B
from test_walk_code import _disassemble


def test_ttft_walk_entries_land_on_step_starts(tmp_path):
    ins = _disassemble(tmp_path)
    at = {a: i for i, (a, _) in enumerate(ins)}
    lit = r"(0x[0-9a-f]+|\d+)"
    blocks = 0
    for i, (_, text) in enumerate(ins):
        if text != "s_getpc_b64 s[92:93]":
            continue
        blocks += 1
        pc = ins[i + 1][0]
        assert re.fullmatch(r"v_readfirstlane_b32 s95, v\d+", ins[i - 1][1])
        assert ins[i + 1][1] == "s_and_b32 s94, s95, 15"  # e < 16
        mul = re.fullmatch(r"s_mul_i32 s94, s94, " + lit, ins[i + 2][1])
        add = re.fullmatch(r"s_add_u32 s94, s94, " + lit, ins[i + 3][1])
        assert [x[1] for x in ins[i + 4:i + 8]] == [
            "s_add_u32 s92, s92, s94", "s_addc_u32 s93, s93, 0", "s_bfe_u32 s95, s95, 0x20004",
            "s_setpc_b64 s[92:93]"]
        step, off = int(mul.group(1), 0), int(add.group(1), 0)
        assert pc + off == ins[i + 8][0]
        rel = {0: set(), 1: set()}
        for e in range(16):
            j = at[pc + e * step + off]
            m = re.fullmatch(r"v_cmp_eq_u32_e64 s\[\d+:\d+\], (\d+), (v\d+)", ins[j + 2][1])
            assert ins[j][1].startswith("ds_read_b32") and m and int(m.group(1)) == e
            rel[e & 1].add(m.group(2))
            # three decisions, each bounded by a saturating sum
            body = [x[1] for x in ins[j:at[pc + (e + 1) * step + off]]]
            assert sum(x.startswith("v_add_i32") and x.endswith("clamp") for x in body) == 3
        assert len(rel[0]) == 1 and len(rel[1]) == 1 and rel[0] != rel[1]
        j = at[pc + 16 * step + off]
        assert {re.fullmatch(r"v_add_u32_e32 (v\d+), -16, \1", ins[k][1]).group(1)
                for k in (j, j + 1)} == rel[0] | rel[1]
        assert ins[j + 2][1] == "s_sub_u32 s95, s95, 1"
        addr, br = ins[j + 3]
        simm = int(br.split()[-1], 0)
        simm = simm - 65536 if simm >= 32768 else simm
        assert br.startswith("s_cbranch_scc0") and addr + 4 + 4 * simm == pc + off
    src = open(os.path.join(B.CSRC, "dm_select.hip")).read()
    assert blocks == int(re.search(r"constexpr int kPrefetch = (\d+);", src).group(1))
