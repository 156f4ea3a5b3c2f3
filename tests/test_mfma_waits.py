"""Wait states between a matrix product and the first use of its result, in
the assembly of the MLP kernels compiled here.  v_mfma_f32_16x16x32_bf16
takes 4 passes of 4 cycles, and a use of its result other than by the next
product must be 4 passes + 4 states behind (passes + 3 in the published table
for gfx942); on every path of the control flow the first such use is counted in
issued instructions, an s_nop n as n + 1."""
import os
import re
import subprocess

import pytest

from paper_2010_13513_amd import build

STATES = 8


def _registers(text):
    out = {m[1] + m[2] for m in re.finditer(r"\b([av])(\d+)\b", text)}
    for m in re.finditer(r"\b([av])\[(\d+):(\d+)\]", text):
        out |= {f"{m[1]}{r}" for r in range(int(m[2]), int(m[3]) + 1)}
    return out


def _kernels(asm):
    """Instructions and label positions of every kernel."""
    out, name = {}, None
    for line in asm.splitlines():
        text = line.split(";")[0].strip()
        if m := re.match(r"^(_Z\w+):", line):
            name, ins, labels = m[1], [], {}
            out[name] = (ins, labels)
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and (m := re.match(r"^(\.LBB\w+):", line)):
            labels[m[1]] = len(ins)
        elif name and text and not text.startswith(".") and not text.endswith(":"):
            ins.append(text)
    return out


def shortest_wait(ins, labels, at, limit):
    """States from the product ins[at] to the first other use of its result on
    any path, `limit` if there is none that close."""
    regs = _registers(ins[at].split()[1])
    todo, best, best_at = [(at + 1, 0)], limit, {}
    while todo:
        p, states = todo.pop()
        if p >= len(ins) or states >= best or best_at.get(p, limit) <= states:
            continue
        best_at[p] = states
        op = ins[p].split()[0]
        if op.startswith("v_mfma"):
            # the next product takes the result as its sum (its own operands
            # are loads) and starts the count again, at its own entry
            assert not _registers(",".join(ins[p].split(",")[1:3])) & regs, ins[p]
            continue
        if _registers(ins[p]) & regs:
            best = states
            continue
        states += int(ins[p].split()[1], 0) + 1 if op == "s_nop" else 1
        if op == "s_endpgm":
            continue
        if op.startswith(("s_branch", "s_cbranch")):
            todo.append((labels[ins[p].split()[1]], states))
        if op != "s_branch":
            todo.append((p + 1, states))
    return best


def test_products_of_the_mlp_kernels(tmp_path):
    if not os.path.exists(build.GEN_OUT):
        build.generate(False)
    src, out = os.path.join(build.HERE, "csrc", "mlp.hip"), str(tmp_path / "mlp.s")
    cmd = [build.hipcc(), "--offload-arch=gfx950"] + build.FLAGS + ["--cuda-device-only", "-S", "-o", out, src]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    with open(out) as f:
        kernels = _kernels(f.read())
    found = {}
    for name, (ins, labels) in kernels.items():
        waits = [shortest_wait(ins, labels, p, 64) for p, t in enumerate(ins) if t.startswith("v_mfma")]
        if waits:
            found[name] = min(waits)
            assert any(w < 64 for w in waits), name                    # a use was found
    print(found)
    assert {n for n in ("k_forward", "k_backward") if any(n in k for k in found)} == {"k_forward", "k_backward"}
    assert min(found.values()) >= STATES


@pytest.mark.parametrize("tail,states", [
    (["s_nop 3", "v_accvgpr_read_b32 v0, a2"], 4),
    (["s_cbranch_scc0 .LBB0_1", "s_nop 7", "v_mov_b32_e32 v9, 0", "v_accvgpr_read_b32 v0, a0"], 1),   # branch taken
    (["s_nop 1", "v_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]", "v_accvgpr_read_b32 v0, a0"], 64)])
def test_the_count_itself(tail, states):
    ins = ["v_mfma_f32_16x16x32_bf16 a[0:3], v[2:5], v[6:9], a[0:3]"] + tail
    assert shortest_wait(ins, {".LBB0_1": len(ins) - 1}, 0, 64) == states
