"""Wait states around the matrix instructions of the persistent prefill kernels, which are written as assembly statements that
the compiler's hazard recogniser does not look into (csrc/bm_gemm_bf16.hip, BM_MFMA1).  Read off the assembly that the
build's compiler emits for the build's flags (own code, device side only), along every path of the control flow."""
import os
import re
import subprocess

from paper_2511_10054_amd import build

CAP = 64              # wait states that are told apart
RESULT_WAIT = 32      # the two s_nop 15 behind a tile's last MFMA; an MFMA of 8 passes needs 11
ZERO_WAIT = 8         # the s_nop 7 behind the zeroing of the accumulators; at most 2 are needed


def _accumulators(code):
    regs = {int(n) for n in re.findall(r"\ba(\d+)\b", code)}
    for lo, hi in re.findall(r"\ba\[(\d+):(\d+)\]", code):
        regs.update(range(int(lo), int(hi) + 1))
    return regs


def _blocks(body):
    """Basic blocks in program order: name -> instructions, and name -> names of the blocks that may follow."""
    blocks, name = {"entry": []}, "entry"
    for line in body.split("\n"):
        label = re.match(r"^(\.LBB\w+):", line)
        if label:
            name = label.group(1)
            blocks[name] = []
            continue
        code = line.split(";")[0].strip()
        if not code or code.startswith(".") or code.endswith(":"):
            continue
        blocks[name].append(code)
        if re.match(r"s_c?branch", code):
            name += "+"
            blocks[name] = []
    names = list(blocks)
    follow = {}
    for i, n in enumerate(names):
        last = blocks[n][-1] if blocks[n] else ""
        branch = re.match(r"s_c?branch\w*\s+(\S+)", last)
        follow[n] = [branch.group(1)] if branch else []
        if not re.match(r"s_branch|s_endpgm", last) and i + 1 < len(names):
            follow[n].append(names[i + 1])
    return blocks, follow


def shortest_distances(body):
    """(wait states from an MFMA to the first other instruction that names its result, wait states from a vector write of an
    accumulator to the first MFMA that names it): the shortest over all paths, each with the later instruction."""
    blocks, follow = _blocks(body)
    steps = {}
    for n, codes in blocks.items():
        steps[n] = []
        for c in codes:
            wait = 1 + int(c.split()[1], 0) if c.startswith("s_nop") else 1
            target = _accumulators(c.split(",")[0]) if c.startswith("v_") else set()
            steps[n].append((c, wait, _accumulators(c), target, c.startswith("v_mfma")))
    best = {"result": (CAP, ""), "zeroing": (CAP, "")}

    def run(entry, n, note):
        mfma, other, now = [-a for a in entry[0]], [-a for a in entry[1]], 0      # times of the last writes
        for code, wait, named, target, matrix in steps[n]:
            if named and note:
                kind, times = ("zeroing", other) if matrix else ("result", mfma)
                age = now - max(times[r] for r in named)
                best[kind] = min(best[kind], (age, code))
            for r in target:
                (mfma if matrix else other)[r] = now + 1
            now += wait
        return tuple([min(CAP, now - t) for t in times] for times in (mfma, other))

    state = {"entry": ([CAP] * 256, [CAP] * 256)}                                  # wait states since the last writes
    work = ["entry"]
    while work:
        n = work.pop()
        out = run(state[n], n, False)
        for m in follow[n]:
            merged = out if m not in state else tuple([min(a, b) for a, b in zip(*pair)] for pair in zip(state[m], out))
            if state.get(m) != merged:
                state[m] = merged
                work.append(m)
    for n in state:
        run(state[n], n, True)
    return best["result"], best["zeroing"]


def test_distances_of_a_made_up_kernel():
    loop = "v_accvgpr_write_b32 a0, 0\ns_nop 1\n.LBB0_1:\nv_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]\ns_cbranch_scc1 .LBB0_1\n"
    assert shortest_distances(loop + "s_nop 3\nv_accvgpr_read_b32 v0, a3\ns_endpgm") == ((5, "v_accvgpr_read_b32 v0, a3"),
                                                                                       (2, "v_mfma_f32_16x16x32_bf16 a[0:3], v[0:3], v[4:7], a[0:3]"))
    assert shortest_distances(loop + "v_accvgpr_mov_b32 a9, a0\ns_nop 15\nv_accvgpr_read_b32 v0, a3\ns_endpgm")[0][0] == 1
    other = loop + "s_cbranch_scc0 .LBB0_2\ns_nop 15\n.LBB0_2:\ns_nop 7\nglobal_store_dwordx4 v[0:1], a[0:3], off\ns_endpgm"
    assert shortest_distances(other)[0] == (10, "global_store_dwordx4 v[0:1], a[0:3], off")


def test_accumulators_are_left_alone_until_their_results_are_there(tmp_path):
    out = tmp_path / "gemm.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, *flags, "-S", "--cuda-device-only", "-o", str(out), os.path.join(build.CSRC, "bm_gemm_bf16.hip")],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN2bm\w*k64w\w*):[^\n]*\n(.*?)\.end_amdhsa_kernel", out.read_text(), flags=re.S | re.M)
    assert len(kernels) >= 3, [k for k, _ in kernels]
    for name, body in kernels:
        result, zeroing = shortest_distances(body)
        print(name, result, zeroing)
        assert result[0] >= RESULT_WAIT, (name, result)
        assert zeroing[0] >= ZERO_WAIT, (name, zeroing)
