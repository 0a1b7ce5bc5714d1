"""Wait states of lane reads, scalar results and lane-row swaps on the built
gfx950 code, on the machinery of isa_hazards (no GPU needed).  The panel
factorization and the sums of the few-column solves issue these instructions
from inline asm, which gets no wait states from the compiler:

  lane_src   VALU writes a VGPR -> v_readlane / v_readfirstlane reads it:       1
  sgpr_use   VALU writes an SGPR -> a VALU instruction reads it:                 2
  perm_src   VALU writes a VGPR -> v_permlane16_swap / 32_swap reads it:         2
  mfma_perm  MFMA writes a VGPR -> a swap reads it: at least as many as the
             compiler leaves before the plain VALU readers of the same opcode
             anywhere in the build.

The checker is pinned on small listings with a planted hazard."""
from __future__ import annotations

import collections
import os

import pytest

from tests import isa_hazards as hz

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_28179_amd", "libglass.so")
LANE_READ = ("v_readlane_b32", "v_readfirstlane_b32")
SWAP = ("v_permlane16_swap", "v_permlane32_swap")


def _sgpr_reads(ins) -> set:
    o = hz.operands(ins.ops)
    dst = 2 if ins.mn.startswith(hz._CARRY_OUT) else 1
    return set().union(*(hz.regs(x, "s") for x in o[dst:])) if ins.mn.startswith("v_") else set()


def check(funcs, mfma_need=None):
    """[(rule, function, writer, reader, wait states)] and the readers seen per rule."""
    mfma_min = {} if mfma_need is not None else hz.check(funcs)["mfma_valu_min"]
    viol, seen = [], collections.Counter()
    for f in funcs:
        fn = hz.Function(f)
        lane = [i.mn.startswith(LANE_READ) for i in fn.ins]
        swap = [i.mn.startswith(SWAP) for i in fn.ins]
        sread = [_sgpr_reads(i) for i in fn.ins]
        src = [hz.regs(hz.operands(i.ops)[1]) if l else set() for i, l in zip(fn.ins, lane)]
        seen["lane_src"] += sum(lane)
        seen["perm_src"] += sum(swap)
        at = {id(inf): k for k, inf in enumerate(fn.info)}

        def near(k, need, pred):
            return fn.readers_within(k, need, lambda r: pred(at[id(r)]))

        for k, inf in enumerate(fn.info):
            hits = []
            if inf.vw:
                w = inf.vw
                hits += [("lane_src", j, d) for j, d in near(k, 1, lambda j: bool(src[j] & w))]
                need = 2
                if inf.mfma:
                    need = mfma_need if mfma_need is not None else mfma_min.get(fn.ins[k].mn, 0)
                rule = "mfma_perm" if inf.mfma else "perm_src"
                hits += [(rule, j, d) for j, d in near(k, need, lambda j: swap[j] and bool((fn.info[j].vr | fn.info[j].vw) & w))]
            s = {x for x in inf.sw if x != "vcc"}
            if inf.valu and s:
                seen["sgpr_use"] += 1
                hits += [("sgpr_use", j, d) for j, d in near(k, 2, lambda j: bool(sread[j] & s))]
            viol += [(rule, fn.name, fn.ins[k], fn.ins[j], d) for rule, j, d in hits]
    return viol, seen


def _listing(body: str) -> list[dict]:
    lines, addr = ["0000000000001000 <k>:"], 0x1000
    for ins in body.strip().splitlines():
        lines.append(f"\t{ins.strip()}  // {addr:012X}: 00000000")
        addr += 4
    return hz.parse("\n".join(lines))


@pytest.mark.parametrize("body,rules", [
    ("v_fmac_f32_e32 v1, v2, v3\nv_readlane_b32 s4, v1, 5\ns_endpgm", ["lane_src"]),
    ("v_fmac_f32_e32 v1, v2, v3\nv_mov_b32_e32 v7, v8\nv_readlane_b32 s4, v1, 5\ns_endpgm", []),
    ("v_readlane_b32 s4, v1, 5\ns_nop 0\nv_rsq_f32_e32 v2, s4\ns_endpgm", ["sgpr_use"]),
    ("v_readlane_b32 s4, v1, 5\ns_nop 1\nv_rsq_f32_e32 v2, s4\ns_endpgm", []),
    ("v_cmp_gt_f32_e64 s[6:7], v1, v2\nv_cndmask_b32_e64 v3, v4, v5, s[6:7]\ns_endpgm", ["sgpr_use"]),
    ("v_mov_b32_e32 v1, v2\ns_nop 0\nv_permlane16_swap_b32_e32 v1, v3\ns_endpgm", ["perm_src"]),
    ("v_mov_b32_e32 v3, v2\ns_nop 0\nv_permlane32_swap_b32_e32 v1, v3\ns_endpgm", ["perm_src"]),
    ("v_mov_b32_e32 v1, v2\ns_nop 1\nv_permlane16_swap_b32_e32 v1, v3\ns_endpgm", []),
    ("v_mfma_f32_4x4x1_16b_f32 v[0:3], v4, v5, v[0:3]\ns_nop 3\nv_permlane32_swap_b32_e32 v0, v2\ns_endpgm",
     ["mfma_perm"]),
])
def test_checker_flags_planted_hazards(body, rules):
    assert sorted({v[0] for v in check(_listing(body), mfma_need=6)[0]}) == rules


def test_built_code_has_none():
    if not os.path.exists(os.path.join(hz.LLVM, "llvm-objdump")):
        pytest.skip("ROCm LLVM tools not installed")
    assert os.path.exists(LIB), "libglass.so is not built"
    funcs, _ = hz.scan_library(LIB)
    viol, seen = check(funcs)
    assert min(seen[r] for r in ("lane_src", "sgpr_use", "perm_src")) > 100, seen
    shown = [f"{rule} in {name}: {w.mn} {w.ops} -> {r.mn} {r.ops} after {d} wait states" for rule, name, w, r, d in viol[:10]]
    assert viol == [], "\n".join(shown)
