"""Wait states that the compiler does not count by itself, checked in the assembly it makes of the kernels (no GPU).

The input gradient's expansion zeroes the accumulators of a sparse matrix instruction from inline assembly, which the compiler does not
know for a vector instruction.  The hardware wants two wait states between a vector instruction's result and a matrix instruction that
reads it, along every path."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAIT_STATES = 2


def vector_registers(operand):
    m = re.fullmatch(r"v\[(\d+):(\d+)\]|v(\d+)", operand)
    if not m:
        return set()
    return {int(m[3])} if m[3] else set(range(int(m[1]), int(m[2]) + 1))


def parse(text):
    """[(label or None, mnemonic, operands, line number)] of the instructions, and the position of every label."""
    code, labels = [], {}
    for number, line in enumerate(text.splitlines(), 1):
        line = line.split(";")[0].strip()
        if re.fullmatch(r"[.\w$]+:", line):
            labels[line[:-1]] = len(code)
        elif re.match(r"[a-z]\w+(\s|$)", line):
            name, _, rest = line.partition(" ") if " " in line else line.partition("\t")
            code.append((name, re.findall(r"v\[\d+:\d+\]|[.\w$]+", rest), number))
    return code, labels


def too_close(text):
    """Lines of sparse matrix instructions that come fewer than WAIT_STATES behind a vector instruction that writes what they read."""
    code, labels = parse(text)
    jumps = {}                                       # position of a label -> positions of the branches that go there
    for k, (name, operands, _) in enumerate(code):
        if name in ("s_branch",) or name.startswith("s_cbranch"):
            jumps.setdefault(labels[operands[0]], []).append(k)

    def near(k, waited, reads):                      # does an instruction up to and with k, `waited` states away, write one of `reads`?
        while waited < WAIT_STATES and k >= 0:
            name, operands, _ = code[k]
            if name in ("s_branch", "s_endpgm") and not jumped[0]:
                return False                         # not a way to get to what follows
            jumped[0] = False
            if name.startswith("v_") and not name.startswith(("v_mfma", "v_smfmac")) and operands and vector_registers(operands[0]) & reads:
                return True
            waited += int(operands[0]) + 1 if name == "s_nop" else 1
            if waited < WAIT_STATES:
                for j in jumps.get(k, []):
                    jumped[0] = True
                    if near(j, waited, reads):
                        return True
                jumped[0] = False
            k -= 1
        return False

    found, seen, jumped = [], 0, [False]
    for k, (name, operands, number) in enumerate(code):
        if name.startswith("v_smfmac"):
            seen += 1
            reads = set().union(*(vector_registers(o) for o in operands))
            for start in [k - 1] + jumps.get(k, []):
                jumped[0] = start != k - 1
                if near(start, 0, reads):
                    found.append(number)
                    break
    return found, seen


def test_the_check_itself():
    write, use = "v_mov_b64 v[4:5], 0\n", "v_smfmac_f32_16x16x64_bf16 v[2:5], v[8:11], v[12:19], v20\n"
    assert too_close(write + use) == ([2], 1)
    assert too_close(write + "s_nop 0\n" + use) == ([3], 1)
    assert too_close(write + "s_nop 1\n" + use) == ([], 1)
    assert too_close("v_mov_b64 v[6:7], 0\n" + use) == ([], 1)
    # over the back edge of a loop, and not past a branch that leads elsewhere
    assert too_close("s_nop 1\n.L:\n" + use + write + "s_cbranch_scc1 .L\n") == ([3], 1)
    assert too_close("s_nop 1\n.L:\ns_nop 1\n" + use + write + "s_cbranch_scc1 .L\n") == ([], 1)
    assert too_close(".M:\n" + write + "s_branch .M\n" + use) == ([], 1)


@pytest.mark.timeout(600)
def test_expansion_waits_for_its_zeroes(tmp_path):
    spec = importlib.util.spec_from_file_location("_sste_build", os.path.join(ROOT, "paper_2409_09099_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    out = str(tmp_path / "dgrad.s")
    cmd = [hipcc] + [f for f in build.FLAGS if f != "-shared"] + ["--offload-device-only", "-S", os.path.join(build.CSRC, "gemm_dgrad.hip"), "-o", out]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout[-4000:]
    with open(out) as f:
        found, seen = too_close(f.read())
    assert seen >= 100 and not found, "%d of %d expansions, the first at line %s" % (len(found), seen, found[:1])
