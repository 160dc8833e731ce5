"""The GEMM kernels update their accumulators with matrix instructions written in assembly, whose latency the compiler does not
know: it may place a move of an accumulator right behind the instruction that writes it.  This looks through the assembly of
the library's own kernels for such moves, and for vector instructions that write an operand right in front of one."""
import functools
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

from paper_2604_05091_amd import build

READ_STATES = 11   # wait states that a read of the result of a 16 x 16 x 32 product (8 passes) has to keep
OPERAND_STATES = 1


def registers(token):
    m = re.match(r"([av])\[(\d+):(\d+)\]", token)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    m = re.match(r"([av])(\d+)\b", token)
    return {(m.group(1), int(m.group(2)))} if m else set()


def findings(assembly):
    """(function, instruction) for every access of an accumulator, or write of an operand, that comes too close; the distance is
    counted along the text, an instruction a wait state (a product that follows: four)."""
    out, function, results, writes = [], None, [], []   # results, writes: (wait states since, registers)
    for line in assembly.split("\n"):
        if m := re.match(r"(_Z\w+):", line):
            function, results, writes = m.group(1), [], []
            continue
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op.startswith("v_mfma"):
            if any(w & (registers(args[1]) | registers(args[2])) and d < OPERAND_STATES for d, w in writes):
                out.append((function, text))
            results = [(d + 4, w) for d, w in results if d < READ_STATES] + [(0, registers(args[0]))]
            writes = []
            continue
        touched = set().union(*(registers(a.split(" ")[0]) for a in args)) if rest else set()
        if any(w & touched and d < READ_STATES for d, w in results):
            out.append((function, text))
        states = int(args[0]) + 1 if op == "s_nop" else 1
        results = [(d + states, w) for d, w in results if d + states < READ_STATES]
        writes = [(d + states, w) for d, w in writes if d + states < OPERAND_STATES]
        if op.startswith("v_"):
            writes.append((0, registers(args[0].split(" ")[0])))
    return out


def test_findings_on_small_texts():
    product = "_Z1k:\n v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n"
    assert findings(product + " s_nop 0\n v_accvgpr_read_b32 v9, a3\n") == [("_Z1k", "v_accvgpr_read_b32 v9, a3")]
    assert findings(product + " v_accvgpr_mov_b32 a9, a0\n") != []
    assert findings(product + " s_nop 15\n v_accvgpr_read_b32 v9, a3\n") == []
    assert findings(product + " v_accvgpr_read_b32 v9, a4\n") == []
    assert findings("_Z1k:\n v_mov_b32 v5, v9\n v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n") != []


@functools.cache
def assemblies():
    def assembly(source):
        r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", "-o", "-", os.path.join(build.CSRC, source)],
                           capture_output=True, text=True, check=True)
        return r.stdout

    sources = ("gemm.hip", "gemm_ring.hip")
    with ThreadPoolExecutor() as ex:
        return list(zip(sources, ex.map(assembly, sources)))


def test_no_accumulator_is_touched_too_early():
    for source, text in assemblies():
        assert "v_mfma_f32_16x16x32_bf16" in text
        assert findings(text) == [], source


def set_too_late(assembly):
    """(function, instruction) for every product whose accumulator a vector instruction wrote less than two wait states before."""
    out, function, writes = [], None, []
    for line in assembly.split("\n"):
        if m := re.match(r"(_Z\w+):", line):
            function, writes = m.group(1), []
            continue
        text = line.split(";")[0].strip()
        if not text or text.startswith(".") or text.endswith(":"):
            continue
        op, _, rest = text.partition(" ")
        args = [a.strip() for a in rest.split(",")]
        if op.startswith("v_mfma") and any(w & registers(args[3]) and d < 2 for d, w in writes):
            out.append((function, text))
        states = int(args[0]) + 1 if op == "s_nop" else 1
        writes = [(d + states, w) for d, w in writes if d + states < 2]
        if op.startswith("v_") and not op.startswith("v_mfma"):
            writes.append((0, registers(args[0].split(" ")[0])))
    return out


def test_no_accumulator_is_set_too_late():
    late = "_Z1k:\n v_accvgpr_write_b32 a0, 0\n v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\n"
    assert set_too_late(late) != [] and set_too_late(late.replace("0\n", "0\n s_nop 1\n")) == []
    for source, text in assemblies():
        assert set_too_late(text) == [], source
