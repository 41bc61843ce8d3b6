"""Kernel launches convert their arguments as a function call does (csrc/rcp_internal.hpp, enqueue): compiled on the host."""
import os
import subprocess

import pytest

from paper_2502_15779_amd import _build

SOURCE = r"""
#include "rcp_internal.hpp"
__global__ void kernel(const float* in, float* out, size_t n, float scale) { out[threadIdx.x] = n ? in[0] * scale : 0.0f; }
void launch(const void* raw, void* raw_out, const float* in, float* out, int n, double scale)
{
    rcp::enqueue(&kernel, 1, 64, 0, nullptr, %s);
}
"""


def _compiles(tmp_path, arguments):
    src = tmp_path / "launch.hip"
    src.write_text(SOURCE % arguments)
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + _build.COMPILE_FLAGS
    cmd += ["-I", os.path.join(_build.ROOT, "include"), "-I", _build.CSRC, "--cuda-host-only", "-fsyntax-only", str(src)]
    return subprocess.run(cmd, capture_output=True, text=True)


@pytest.mark.parametrize("arguments,accepted", [
    ("in, out, n, scale", True), ("nullptr, out, 1u, 1", True), ("out, out, n, 1.0f", True),
    ("raw, out, n, 1.0f", False), ("in, raw_out, n, 1.0f", False), ("in, in, n, 1.0f", False), ("in, out, out, 1.0f", False)])
def test_arguments_convert_as_in_a_call(tmp_path, arguments, accepted):
    res = _compiles(tmp_path, arguments)
    assert (res.returncode == 0) == accepted, res.stderr
    assert accepted or "does not convert" in res.stderr
