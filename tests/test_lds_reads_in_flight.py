"""The FFN and logits kernels read LDS fragments into registers that the compiler takes as written at
once, and wait for them by count.  That is sound only if the code the compiler makes touches no such
register before its wait.  Shown here for every path through the built kernels: the assembly is walked
with the list of LDS reads in flight (they return in issue order; a wait for "at most n pending"
leaves at most the youngest n)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2510_19366_amd import build as hip_build

pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")


def registers(text):
    out = {(k, i) for k, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text) for i in range(int(lo), int(hi) + 1)}
    return frozenset(out | {(k, int(i)) for k, i in re.findall(r"\b([va])(\d+)\b", text)})


def kernels(asm):
    """name -> (instructions, label -> positions)"""
    out, name = {}, None
    for line in asm.split("\n"):
        line = line.split(";")[0].strip()
        m = re.match(r"^([.\w$]+):$", line)
        if m and m[1].startswith("_Z"):
            name, out[m[1]] = m[1], ([], {})
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and m:
            out[name][1].setdefault(m[1], []).append(len(out[name][0]))
        elif name and line and not line.startswith("."):
            out[name][0].append(line)
    return {k: v for k, v in out.items() if any(i.startswith("s_endpgm") for i in v[0])}


def touched_in_flight(ins, labels):
    """Instructions that touch a register an LDS read in flight will write, and the number of LDS reads."""
    bad, reads, seen, work = set(), 0, [set() for _ in ins], [(0, ())]
    while work:
        pc, flight = work.pop()
        while pc < len(ins) and flight not in seen[pc]:
            seen[pc].add(flight)
            text = ins[pc]
            op, rest = (text.split(None, 1) + [""])[:2]
            pending = frozenset().union(*flight)
            if op.startswith("ds_"):
                dst, _, src = rest.partition(",")
                writes = op.startswith(("ds_read", "ds_bpermute", "ds_permute")) or "_rtn" in op
                reads += writes
                if registers(src if writes else rest) & pending:
                    bad.add((pc, text))
                flight += (registers(dst) if writes else frozenset(),)
            elif op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", rest)
                assert m or "cnt" in rest, f"unknown form: {text}"
                if m:  # scalar loads count too, which only makes the wait longer
                    flight = flight[len(flight) - min(len(flight), int(m[1])):]
            elif registers(rest) & pending:
                bad.add((pc, text))
            flight = flight[-32:]
            if op.startswith("s_cbranch") or op == "s_branch":
                t = rest.strip()
                at = labels[t[:-1]] if re.match(r"^\d+[fb]$", t) else labels[t]
                to = min(p for p in at if p > pc) if t.endswith("f") and t[0].isdigit() else at[0]
                if op == "s_branch":
                    pc = to
                    continue
                work.append((to, flight))
            if op == "s_endpgm":
                break
            pc += 1
    return bad, reads


def test_the_walk_sees_an_early_use_and_a_late_wait():
    head = ["ds_read_b128 v[0:3], v9", "ds_read_b128 v[4:7], v9 offset:16"]
    assert not touched_in_flight(head + ["s_waitcnt lgkmcnt(1)", "v_mov_b32 v8, v3", "s_endpgm"], {})[0]
    assert touched_in_flight(head + ["s_waitcnt lgkmcnt(1)", "v_mov_b32 v8, v4", "s_endpgm"], {})[0]
    loop = head + ["s_cbranch_scc1 .L", "s_waitcnt lgkmcnt(0)", "v_add_u32 v9, v4, v4", "s_endpgm"]
    assert not touched_in_flight(loop, {".L": [3]})[0]
    assert touched_in_flight(loop, {".L": [4]})[0]


@pytest.mark.parametrize("source", ["ffn_bf16.hip", "ffn_fused_bf16.hip", "ffn.hip", "route.hip"])
def test_no_register_is_touched_before_its_read_has_returned(source, tmp_path):
    out = tmp_path / "device.s"
    subprocess.run(["hipcc", *hip_build.FLAGS, "--offload-device-only", "-S", os.path.join(hip_build.CSRC, source),
                    "-o", str(out)], check=True, capture_output=True)
    total = 0
    for name, (ins, labels) in kernels(out.read_text()).items():
        bad, reads = touched_in_flight(ins, labels)
        assert not bad, (name, sorted(bad)[:5])
        total += reads
    assert total > 0
