"""What the compiler makes of the matrix kernels: no vector register spilled, and no LDS read in flight touched.

The projection kernels use up to 256 registers a wave, and a spill in their loops costs several times their time.
Some of them read LDS by instructions whose result the compiler takes as written at once (the wait is its own
instruction, tied to the registers): nothing may read or overwrite such a register before a wait that covers it.
"""
import os
import re
import subprocess

import pytest

from paper_2609_34370_amd import build

SOURCES = ["lm_head.hip", "linear.hip", "attention.hip"]


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """Device assembly and resource remarks of each source, with the build's flags."""
    d = tmp_path_factory.mktemp("asm")
    jobs = {}
    for src in SOURCES:
        out = str(d / (src + ".s"))
        cmd = [build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage",
               os.path.join(build.CSRC, src), "-o", out]
        jobs[src] = (out, subprocess.Popen(cmd, stderr=subprocess.PIPE, text=True))
    result = {}
    for src, (out, p) in jobs.items():
        remarks = p.communicate()[1]
        assert p.returncode == 0, remarks
        result[src] = (open(out).read(), remarks)
    return result


@pytest.mark.parametrize("src", SOURCES)
def test_no_vector_register_is_spilled(compiled, src):
    remarks = compiled[src][1]
    names = re.findall(r"Function Name: (\S+)", remarks)
    spills = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", remarks)]
    assert names and len(names) == len(spills)
    assert {n: s for n, s in zip(names, spills) if s} == {}


def kernels(asm):
    """(name, basic blocks) of each function: a block is (label, instructions)."""
    for m in re.finditer(r"^(_Z\w+):[^\n]*$(.*?)^\.Lfunc_end", asm, re.M | re.S):
        blocks, cur = [], ("", [])
        for line in m[2].split("\n"):
            line = line.split(";")[0].strip()
            label = re.match(r"(\.L\w+):$", line)
            if label:
                blocks.append(cur)
                cur = (label[1], [])
            elif line and not line.startswith("."):
                cur[1].append(line)
                if line.startswith(("s_cbranch", "s_branch", "s_endpgm")):
                    blocks.append(cur)
                    cur = ("", [])
        blocks.append(cur)
        yield m[1], blocks


def registers(text):
    out = set()
    for kind, lo, hi in re.findall(r"\b([va])\[(\d+):(\d+)\]", text):
        out |= {(kind, i) for i in range(int(lo), int(hi) + 1)}
    return out | {(kind, int(i)) for kind, i in re.findall(r"\b([va])(\d+)\b", text)}


def touched_in_flight(blocks):
    """Instructions that name a register an LDS read still in flight will write, and the count of LDS reads.
    LDS operations of a wave return in order; scalar loads share their counter."""
    at = {label: i for i, (label, _) in enumerate(blocks) if label}
    bad, reads, seen, work = set(), 0, set(), [(0, ())]
    while work:
        i, flight = work.pop()
        if (i, flight) in seen:
            continue
        seen.add((i, flight))
        assert len(seen) < 100000
        flight, falls = list(flight), True
        for ins in blocks[i][1]:
            op, rest = ins.split(None, 1) if " " in ins or "\t" in ins else (ins, "")
            if op == "s_waitcnt":
                m = re.search(r"lgkmcnt\((\d+)\)", rest)
                if m:
                    flight = flight[len(flight) - int(m[1]):] if int(m[1]) < len(flight) else flight
                    flight = [] if m[1] == "0" else flight
                continue
            if registers(rest) & {r for dst in flight for r in dst}:
                bad.add(ins)
            if op.startswith("ds_"):
                returns = op.startswith("ds_read") or "permute" in op or "swizzle" in op
                reads += returns
                flight.append(tuple(sorted(registers(rest.split(",")[0]))) if returns else ())
            elif op.startswith(("s_load", "s_buffer_load")):
                flight.append(())
            if op.startswith(("s_cbranch", "s_branch")):
                work.append((at[rest.strip()], tuple(flight[-32:])))
                falls = op.startswith("s_cbranch")
            elif op == "s_endpgm":
                falls = False
        if falls and i + 1 < len(blocks):
            work.append((i + 1, tuple(flight[-32:])))
    return bad, reads


@pytest.mark.parametrize("src", ["lm_head.hip", "linear.hip"])
def test_no_lds_read_in_flight_is_touched(compiled, src):
    checked = 0
    for name, blocks in kernels(compiled[src][0]):
        bad, reads = touched_in_flight(blocks)
        assert not bad, (name, sorted(bad)[:5])
        checked += reads > 0
    assert checked >= 6


def test_the_check_sees_a_read_before_its_wait():
    blocks = [("", ["ds_read_b128 v[4:7], v0", "v_add_u32_e32 v1, v2, v3", "s_waitcnt lgkmcnt(0)",
                    "v_add_u32_e32 v1, v4, v3", "s_endpgm"])]
    assert touched_in_flight(blocks) == (set(), 1)
    early = [("", ["ds_read_b128 v[4:7], v0", "ds_read_b128 v[8:11], v0", "s_waitcnt lgkmcnt(1)", "v_mov_b32_e32 v1, v5",
                   "v_mov_b32_e32 v9, v1", "s_waitcnt lgkmcnt(0)", "s_endpgm"])]
    assert touched_in_flight(early) == ({"v_mov_b32_e32 v9, v1"}, 2)
    loop = [("", ["s_nop 0"]), (".LBB0_1", ["v_mov_b32_e32 v1, v4", "ds_read_b128 v[4:7], v0", "s_cbranch_scc1 .LBB0_1"]),
            ("", ["s_endpgm"])]
    assert touched_in_flight(loop)[0] == {"v_mov_b32_e32 v1, v4", "ds_read_b128 v[4:7], v0"}
