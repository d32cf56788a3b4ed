"""The hand-scheduled instruction run of the encoder's two-byte recurrence, checked as it was assembled for gfx950 (CPU only): the
hardware does not check the distances between a matrix instruction and what reads its sums, and the compiler does not look into
the run, so nothing else would notice a step that is too short."""
import os
import re
import subprocess

import pytest

from paper_2211_13939_amd import build

# gfx950: a sum of a 4-pass matrix instruction may be read by a vector instruction 8 wait states after it (what the compiler leaves
# behind its own: s_nop 7); an operand written by a vector instruction may be read by a matrix instruction 2 later
SUM_TO_VECTOR, VECTOR_TO_MATRIX = 8, 2


def _regs(text):
    """'v[200:203]' -> {('v', 200), ...}; 'v7' -> {('v', 7)}; anything else -> {}"""
    m = re.fullmatch(r"([va])\[(\d+):(\d+)\]", text)
    if m:
        return {(m[1], r) for r in range(int(m[2]), int(m[3]) + 1)}
    m = re.fullmatch(r"([va])(\d+)", text)
    return {(m[1], int(m[2]))} if m else set()


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "encoder.s")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC] + flags + ["--cuda-device-only", "-S", "-x", "hip", os.path.join(build.CSRC, "encoder.hip"), "-o", out],
                   check=True, stderr=subprocess.DEVNULL)
    return open(out).read()


@pytest.fixture(scope="module")
def runs(assembly):
    body = assembly[re.search(r"^_ZN3tts\S*k_enc_lstm_sp\S*:", assembly, re.M).start():]
    body = body[:body.index("s_endpgm")]
    blocks = [b for b in re.findall(r"#ASMSTART\n(.*?);;#ASMEND", body, re.S) if "smfmac" in b]
    assert len(blocks) == 2                     # the two buffers of h
    return [[[a for a in re.split(r"[\s,]+", line.strip()) if a] for line in b.splitlines() if line.strip()] for b in blocks]


def test_nothing_of_the_run_is_spilled(assembly):
    entry = re.search(r"\.name:\s+_ZN3tts\S*k_enc_lstm_sp.*?\.wavefront_size", assembly, re.S)[0]
    assert int(re.search(r"vgpr_spill_count: (\d+)", entry)[1]) == 0 and int(re.search(r"private_segment_fixed_size: (\d+)", entry)[1]) == 0


def test_every_read_is_waited_for(runs):
    """LDS reads return in order: no matrix instruction takes a register whose read may still be on its way, and none is on its
    way at the end of the run, where the compiler takes the outputs as written."""
    for run in runs:
        on_the_way = [{("?", 0)}] * 15          # what the compiler may have queued in front
        for op, *a in run:
            if op == "s_waitcnt":
                n = int(re.fullmatch(r"lgkmcnt\((\d+)\)", a[0])[1])
                on_the_way = on_the_way[len(on_the_way) - n:] if n else []
            elif op == "ds_read_b128":
                on_the_way.append(_regs(a[0]))
            else:
                taken = set().union(*(_regs(x) for x in a))
                assert not any(taken & r for r in on_the_way), (op, a)
        assert on_the_way == []


def test_distances_to_and_from_matrix_instructions(runs):
    for run in runs:
        state, summed, written = 0, {}, {}
        for op, *a in run + run:                # (the next step follows: the sums of the one before are what it clears)
            if op in ("s_waitcnt", "ds_read_b128"):
                state += op == "ds_read_b128"
            elif op == "s_nop":
                state += int(a[0]) + 1
            elif op.startswith("v_smfmac"):
                for r in set().union(*(_regs(x) for x in a)):
                    assert state - written.get(r, -99) > VECTOR_TO_MATRIX, (a, r)
                summed.update({r: state for r in _regs(a[0])})
                state += 1
            else:
                for r in set().union(*(_regs(x) for x in a)):
                    assert state - summed.get(r, -99) > SUM_TO_VECTOR, (op, a, r)
                written.update({r: state for r in _regs(a[0])})
                state += 1


def test_every_weight_takes_part_once(runs):
    """64 instructions a step, all with weights of their own: 52 fragments in registers, 12 in LDS (piece i of group U at offset
    (3 U + i) * 2048), each requested one group ahead."""
    for run in runs:
        lds, in_regs, n, first = {}, set(), 0, {200: 0, 208: 1, 216: 2}
        used = []
        for op, *a in run:
            if op.startswith("v_smfmac"):
                w = a[2]
                m = re.fullmatch(r"v\[(200|208|216):\d+\]", w)
                if m:
                    used.append((n // 16, lds.pop(int(m[1]), first[int(m[1])])))
                else:
                    assert w not in in_regs
                    in_regs.add(w)
                n += 1
            elif op == "ds_read_b128":
                reg, m = min(r for _, r in _regs(a[0])), re.fullmatch(r"offset:\((\d)\*3\+(\d)\)\*2048", a[2])
                if m and reg in first:
                    lds[reg] = 3 * int(m[1]) + int(m[2])
        assert n == 64 and len(in_regs) == 52
        assert used == [(p // 3, p) for p in range(12)]
        assert lds == first                     # the next step's first group
