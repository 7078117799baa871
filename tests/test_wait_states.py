"""Wait states around inline assembly, which the compiler does not look into: the generated code of the matrix-core kernels, walked
along every path.  A matrix instruction may read a vector register two instructions behind the vector instruction that
wrote it, and its own results (32 x 32 x 16, eight passes) are there twelve wait states behind its issue; a matrix instruction
issues eight wait states behind the one before it at the earliest.  Pairs that the compiler sees both ends of are its own business."""
import os
import re
import subprocess

import pytest

from paper_2509_09682_amd import build as B

VALU_TO_MFMA, MFMA_TO_USE, MFMA_ISSUE = 2, 12, 8
FAR = 64
REG = re.compile(r"\b([va])(?:(\d+)\b|\[(\d+):(\d+)\])")


def _regs(text):
    return {(m[1], i) for m in REG.finditer(text) for i in (range(int(m[2]), int(m[2]) + 1) if m[2] else range(int(m[3]), int(m[4]) + 1))}


def parse(lines):
    """Kernels as lists of blocks: name -> [(label, [(op, written, read, text, inline)], targets, falls through)]."""
    kernels, blocks, inline = {}, None, False
    for raw in lines:
        line = raw.strip()
        if m := re.match(r"(_Z\w+):", line):
            kernels[m[1]] = blocks = [["", [], [], True]]
        elif line.startswith(".Lfunc_end"):
            blocks = None
        elif blocks is None:
            continue
        elif line.startswith((";;#ASMSTART", ";;#ASMEND")):
            inline = line.startswith(";;#ASMSTART")
        elif m := re.match(r"(\.LBB\w+):", line):
            blocks.append([m[1], [], [], True])
        elif line and line[0] not in ";.":
            text = line.split(";")[0].strip()
            op, _, rest = text.partition(" ")
            first, _, others = rest.partition(",")
            writes = op.startswith(("v_", "ds_read", "global_load_dword", "scratch_load", "buffer_load")) and not op.startswith("v_cmp")
            written = _regs(first) if writes else set()
            blocks[-1][1].append((op, written, _regs(others) if writes else _regs(rest), text, inline))
            if op.startswith(("s_branch", "s_cbranch")):
                blocks[-1][2].append(rest.strip())
                blocks[-1][3] = op != "s_branch"
                blocks.append(["", [], [], True])
            elif op == "s_endpgm":
                blocks[-1][3] = False
                blocks.append(["", [], [], True])
    return kernels


def walk(block, state, found):
    """state: (register, kind, inline) -> wait states since that write, and 'issue' -> since the last matrix instruction."""
    state = dict(state)

    def pass_time(n):
        for k in list(state):
            state[k] += n
            if state[k] >= FAR and k != "issue":
                del state[k]

    for op, written, read, text, inline in block[1]:
        if op == "s_nop":
            pass_time(int(text.split()[1]) + 1)
            continue
        mfma = op.startswith("v_mfma")
        if mfma and state["issue"] < MFMA_ISSUE:
            pass_time(MFMA_ISSUE - state["issue"])
        accumulators = set()
        if mfma:  # the same registers taken on by the next matrix instruction: forwarded
            d, _, _, c = text.partition(" ")[2].split(", ")[:4]
            accumulators = _regs(d) if c == d else set()
        for r in (written | read) - accumulators:
            for kind, need in (("valu", VALU_TO_MFMA if mfma and r in read else 0), ("mfma", MFMA_TO_USE)):
                for by in (False, True):
                    age = state.get((r, kind, by))
                    if age is not None and age < need and (by or inline):
                        found.add((text, kind, age))
        for r in written:
            for kind in ("valu", "mfma"):
                for by in (False, True):
                    state.pop((r, kind, by), None)
        pass_time(1)
        if mfma:
            state["issue"] = 1
        if op.startswith("v_"):
            for r in written:
                state[(r, "mfma" if mfma else "valu", inline)] = 1 if mfma else 0
    return state


def faults(blocks):
    where = {b[0]: i for i, b in enumerate(blocks) if b[0]}
    entry = {0: {"issue": FAR}}
    found, todo = set(), [0]
    while todo:
        i = todo.pop()
        out = walk(blocks[i], entry[i], found)
        out["issue"] = min(out["issue"], FAR)
        nexts = [where[t] for t in blocks[i][2] if t in where] + ([i + 1] if blocks[i][3] and i + 1 < len(blocks) else [])
        for j in nexts:
            old = entry.get(j)
            if old is None:
                new = dict(out)
            else:
                new = {k: min(v for v in (old.get(k), out.get(k)) if v is not None) for k in old.keys() | out.keys()}
                new["issue"] = max(old["issue"], out["issue"])
            if new != old:
                entry[j] = new
                todo.append(j)
    return found


def test_the_walk_finds_what_it_looks_for():
    def of(*body):
        return faults(parse(["_Zk:", *body, "s_endpgm", ".Lfunc_end0:"])["_Zk"])

    product = [";;#ASMSTART", "v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]", ";;#ASMEND"]
    assert of("v_mov_b32_e32 v4, v9", "s_waitcnt lgkmcnt(0)", *product)
    assert not of("v_mov_b32_e32 v4, v9", "s_nop 1", *product)
    assert of(*product, "s_nop 9", "v_accvgpr_read_b32 v20, a3")
    assert not of(*product, "s_nop 11", "v_accvgpr_read_b32 v20, a3") and not of(*product, *product, "s_nop 15", "v_accvgpr_read_b32 v20, a3")
    # round a loop, and by the shorter of two ways in
    assert of(".LBB0_1:", *product, "s_nop 3", "v_mov_b32_e32 v5, v9", "s_cbranch_scc1 .LBB0_1")
    assert of("v_mov_b32_e32 v4, v9", "s_cbranch_scc1 .LBB0_2", "s_nop 7", ".LBB0_2:", *product)


def test_wait_states_of_the_tile_kernels(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no HIP compiler here")
    flags = [f for f in B.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    jobs = []
    for d in (64, 128, 256):
        out = tmp_path / f"d{d}.s"
        cmd = [hipcc, *flags, "-I", os.path.join(B.ROOT, "include"), "-I", B.CSRC, "--cuda-device-only", "-S",
               os.path.join(B.CSRC, f"cce_tile_d{d}.hip"), "-o", str(out)]
        jobs.append((out, subprocess.Popen(cmd, stdout=subprocess.DEVNULL, stderr=subprocess.DEVNULL)))
    seen = 0
    for out, job in jobs:
        assert job.wait() == 0
        for name, blocks in parse(out.read_text().splitlines()).items():
            seen += any(i[4] and i[0].startswith("v_mfma") for b in blocks for i in b[1])
            assert not faults(blocks), name
            # m0, which inline assembly cannot name as changed (the compiler reserves it): a kernel's own or the compiler's
            uses = {i[4] for b in blocks for i in b[1] if re.search(r"\bm0\b|_lds_", i[3])}
            assert len(uses) <= 1, name
    assert seen >= 4  # the kernels of hidden size 256 with matrix instructions in inline assembly
