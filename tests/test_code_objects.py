"""What the compiler made of the kernels: spills, and the registers of LDS reads in flight."""
import os
import re

import pytest

from paper_2608_24070_amd import slim
from tests import code_objects


def test_kernels_keep_their_registers():
    # a spilled register is reloaded behind a wait for every load in flight, which a pipelined loop cannot afford
    kernels = code_objects.kernel_metadata(slim.LIB_PATH)
    assert sum("6k_tileI" in n for n in kernels) == 4 and sum("5k_midI" in n for n in kernels) == 4
    spilled = {n: k[".vgpr_spill_count"] for n, k in kernels.items() if k[".vgpr_spill_count"] or k[".sgpr_spill_count"]}
    assert not spilled, spilled


def _registers(text):
    out = set()
    for bank, lo, hi, bank1, one in re.findall(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
        out |= {(bank, i) for i in range(int(lo), int(hi) + 1)} if bank else {(bank1, int(one))}
    return frozenset(out)


def touched_in_flight(body):
    """Instructions that name a vector register whose LDS read may not have returned, over all paths of a function: LDS
    operations return in order, and s_waitcnt lgkmcnt(n) leaves at most the last n of them outstanding. A read is
    tracked by how many operations were issued after it; where paths meet, the fewest count."""
    at = {a: i for i, (a, _) in enumerate(body)}
    ins = []
    for addr, text in body:
        op, _, rest = text.partition(" ")
        wait = re.search(r"lgkmcnt\((\d+)\)", text) if op == "s_waitcnt" else None
        reads = op.startswith("ds_") and ("read" in op or "permute" in op or "swizzle" in op or "_rtn" in op)
        target = None
        if op.startswith(("s_cbranch", "s_branch")):
            offset = int(rest.split()[0])
            target = at[addr + 4 + 4 * (offset - 65536 if offset >= 32768 else offset)]
        ins.append((op, int(wait.group(1)) if wait else None, _registers(rest) if op != "s_waitcnt" else frozenset(),
                    _registers(rest.split(",")[0]) if reads else frozenset(),
                    op.startswith(("ds_", "s_load", "s_buffer_load")), target))
    joins = {t for *_, t in ins if t is not None}
    state, bad, work = {}, set(), [(0, {})]
    while work:
        i, live = work.pop()
        while True:
            if i in joins or i == 0:
                known = state.setdefault(i, None)
                if known is not None:
                    merged = dict(known)
                    for r, n in live.items():
                        merged[r] = min(n, merged.get(r, n))
                    if merged == known:
                        break
                    live = merged
                state[i] = dict(live)
            op, wait, regs, dest, counts, target = ins[i]
            if wait is not None:
                live = {r: n for r, n in live.items() if n < wait}
            if live and any(r in live for r in regs):
                bad.add(body[i])
            if counts:
                live = {r: n + 1 for r, n in live.items()}
                for r in dest:
                    live[r] = 0
            if op == "s_endpgm":
                break
            if target is not None:
                if op == "s_branch":
                    i = target
                    continue
                work.append((target, dict(live)))
            i += 1
    return bad


def test_touched_in_flight_sees_a_missing_wait():
    ok = [(0, "ds_read_b128 v[0:3], v9"), (8, "ds_read_b64 v[4:5], v9"), (16, "s_waitcnt lgkmcnt(1)"),
          (20, "v_add_f32_e32 v6, v0, v3"), (24, "s_cbranch_scc0 1"), (28, "s_waitcnt lgkmcnt(0)"),
          (32, "v_mov_b32_e32 v7, v6"), (36, "s_endpgm")]
    assert not touched_in_flight(ok)
    early = list(ok)
    early[3] = (20, "v_add_f32_e32 v6, v0, v4")
    assert touched_in_flight(early) == {early[3]}
    # only on the path that jumps over the wait
    jumped = list(ok)
    jumped[6] = (32, "v_mov_b32_e32 v7, v5")
    assert touched_in_flight(jumped) == {jumped[6]}


# The kernels whose LDS reads are written out and waited for by count
@pytest.mark.skipif(not os.path.exists(code_objects.OBJDUMP), reason="no llvm-objdump")
def test_written_out_reads_land_before_their_registers_are_used(tmp_path):
    bodies = code_objects.disassembly(slim.LIB_PATH, str(tmp_path))
    names = [n for n in bodies if re.search(r"\d(k_tileI|k_midI|k_adapter_tn|k_hybrid_gemm|k_grad_w|k_grad_w_smallI)", n)
             and not n.endswith(".kd")]
    assert len(names) == 4 + 4 + 1 + 2 + 2 + 2, names
    for n in names:
        assert sum(t.startswith("ds_read") for _, t in bodies[n]) > 16, n
        assert not touched_in_flight(bodies[n]), n
