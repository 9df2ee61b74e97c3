"""b1 may start at any element (W1 and W2 at 16 bytes): the four-bias read of the bulk hash, compiled for
the host with the alignment sanitizer (a wider read from such an address stops the program), gives the elements'
values."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2508_19740_amd", "csrc")

PROGRAM = r"""
#include "hash_bulk.h"
using namespace spotlight::hashdev;
alignas(16) static float f[12];
alignas(16) static bf16_raw h[12];
int main()
{
    for (int i = 0; i < 12; ++i) { f[i] = i + 0.5f; h[i].v = static_cast<uint16_t>(0x3f80 + i); }
    float v[4];
    for (int at = 0; at < 8; ++at) {
        spotlight::bulk::load_bias4(f + at, v);
        for (int e = 0; e < 4; ++e) if (v[e] != at + e + 0.5f) return 1;
        spotlight::bulk::load_bias4(h + at, v);
        for (int e = 0; e < 4; ++e) if (v[e] != 1.0f + (at + e) * 0x1p-7f) return 2;
    }
    return 0;
}
"""


def test_biases_are_read_at_any_element(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / "bias.hip", tmp_path / "bias"
    src.write_text(PROGRAM)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-Wno-unused-command-line-argument",
                    "-Xarch_host", "-fsanitize=alignment", "-Xarch_host", "-fsanitize-trap=alignment",
                    "-I", CSRC, "-I", os.path.join(CSRC, "..", "..", "include"), str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
