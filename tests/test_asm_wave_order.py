"""Static check of the order of a wave's own LDS accesses (CPU only).

In `attn_f32_kernel` a wave writes the rows of a K block to LDS and other lanes of the
same wave read them, without a workgroup barrier.  The hardware keeps a wave's LDS
accesses in order, but the compiler keeps one lane's only as far as it cannot tell their
addresses apart, so an ordering point has to stand between them.  In the gfx950 assembly of
every instantiation there is one, the rows are written before it, and no LDS write comes
between it and the reads.
"""
import os
import shutil
import subprocess

import pytest

from tests.test_asm_lds_reads import CSRC, HIPCC, ROOT


def _bodies(path, name):
    """The lines of every kernel whose symbol holds `name`."""
    found, current = {}, None
    for raw in open(path):
        line = raw.strip()
        if current is None and name in line and line.split(";")[0].strip().endswith(":") and not line.startswith("."):
            current = line.split(":")[0]
            found[current] = []
        elif current is not None:
            if line.startswith(".amdhsa_"):
                current = None
            else:
                found[current].append(line)
    return found


def _around_the_points(body):
    """The LDS accesses just before and just after each ordering point."""
    lds = lambda line: line.split()[0] if line.startswith("ds_") else None
    for i, line in enumerate(body):
        if "wave barrier" in line:
            yield (next((x for x in map(lds, reversed(body[:i])) if x), None),
                   next((x for x in map(lds, body[i:]) if x), None))


def test_the_scan_sees_the_accesses():
    body = ["ds_write_b128 v0, v[4:7]", "; wave barrier", "v_nop", "ds_read_b128 v[8:11], v1"]
    assert list(_around_the_points(body)) == [("ds_write_b128", "ds_read_b128")]
    assert list(_around_the_points(body[:1] + body[2:])) == []


def test_k_blocks_pass_between_lanes_in_order(tmp_path):
    if not os.path.exists(HIPCC) and not shutil.which("hipcc"):
        pytest.skip("hipcc not available")
    out = tmp_path / "attn_f32.s"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    f"-I{os.path.join(ROOT, 'include')}", "--cuda-device-only", "-S",
                    os.path.join(CSRC, "attn_f32.hip"), "-o", str(out)], check=True, capture_output=True)
    kernels = _bodies(out, "attn_f32_kernel")
    assert len(kernels) == 12, sorted(kernels)
    for kernel, body in kernels.items():
        points = list(_around_the_points(body))
        assert points, kernel
        for before, after in points:
            assert before.startswith("ds_write") and after.startswith("ds_read"), (kernel, before, after)
