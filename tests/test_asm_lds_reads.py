"""Static check of LDS reads issued as inline assembly (CPU only).

`attn_block_kernel` issues its LDS operand reads as inline assembly and waits for
them with explicit `s_waitcnt lgkmcnt` statements that name the results; the
compiler believes a result is there as soon as the read is issued.  In the gfx950
assembly of every instantiation no instruction may touch a register that a read
still has in flight (LDS reads complete in order, so `lgkmcnt(n)` leaves the last
n), and the kernels use no scratch memory (a spilled result would be stored before
it has arrived).
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_31224_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _regs(operands):
    out = set()
    for f, a, b in re.findall(r"\b([va])\[(\d+):(\d+)\]", operands):
        out |= {(f, i) for i in range(int(a), int(b) + 1)}
    for f, a in re.findall(r"(?<![\w\[])([va])(\d+)\b", operands):
        out.add((f, int(a)))
    return out


def _touches_in_flight(body):
    """Instructions that touch the result of an LDS read still in flight, in layout order."""
    pending, bad = [], []
    for line in body:
        m = re.match(r"([a-z]\w+)\s*(.*)", line)
        if not m:
            continue
        op, rest = m.groups()
        if op == "s_waitcnt":
            w = re.search(r"lgkmcnt\((\d+)\)", rest)
            if w:
                n = int(w.group(1))
                pending = pending[max(0, len(pending) - n):] if n else []
            continue
        used = _regs(rest)
        bad += [(line, read) for read, dest in pending if used & dest]
        if op.startswith("ds_read"):
            pending.append((line, _regs(rest.split(",")[0])))
        elif op.startswith(("ds_", "s_load", "s_buffer")):
            pending.append((line, set()))
    return bad


def _kernels(source, name, tmp):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    out = tmp / (source + ".s")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    f"-I{os.path.join(ROOT, 'include')}", "--cuda-device-only", "-S",
                    os.path.join(CSRC, source), "-o", str(out)], check=True, capture_output=True)
    found, body, current = {}, [], None
    for raw in open(out):
        line = raw.split(";")[0].strip()
        if current is None and name in line and line.endswith(":") and not line.startswith("."):
            current, body = line[:-1], []
        elif current is not None:
            body.append(line)
            m = re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", line)
            if m:
                found[current] = (body, int(m.group(1)))
                current = None
    return found


def test_the_scan_sees_a_read_in_flight():
    read, wait = "ds_read_b128 v[4:7], v1 offset:0", "s_waitcnt lgkmcnt(0)"
    assert not _touches_in_flight([read, wait, "v_mov_b32_e32 v9, v5"])
    assert _touches_in_flight([read, "v_mov_b32_e32 v9, v5", wait])
    assert _touches_in_flight([read, "ds_read_b128 v[8:11], v1 offset:16", "s_waitcnt lgkmcnt(1)",
                               "v_add_u32_e32 v8, 1, v8"])


@pytest.mark.parametrize("source,name,count", [("attn_block.hip", "attn_block_kernel", 6)])
def test_lds_reads_waited(source, name, count, tmp_path):
    kernels = _kernels(source, name, tmp_path)
    assert len(kernels) == count, sorted(kernels)
    for kernel, (body, scratch) in kernels.items():
        assert any(line.startswith("ds_read") for line in body), kernel
        assert not _touches_in_flight(body), kernel
        assert scratch == 0, kernel
