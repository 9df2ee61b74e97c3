"""Host rules of the bulk hash, compiled for the CPU: how the tiles of a head are shared out over workgroups."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_19740_amd", "csrc")

RUNS = r"""
#include <stdio.h>
#include <string.h>
#include "hash_bulk.h"
using namespace spotlight;
static int bad(const char* what, long tiles, int heads, int run) { printf("%s: %ld tiles, %d heads, run %d\n", what, tiles, heads, run); return 1; }
int main()
{
    const long some[] = {1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 19, 31, 33, 63, 65, 100, 313, 2047, 2048, 4097, 131072};
    const int heads[] = {1, 4, 8, 31, 32, 256, 512, 4096};
    for (long tiles : some)
        for (int h : heads) {
            for (int run = 1; run <= 64; ++run) {
                const int even = bulk::even_runs(tiles, run);
                const long groups = (tiles + run - 1) / run;
                if (even < 1 || even > run || (tiles + even - 1) / even > groups || (even - 1) * groups >= tiles) return bad("even", tiles, h, even);
            }
            for (int least : {512, 1024, 2048, 4096}) {
                const int run = bulk::short_runs(tiles, h, least);
                const long groups = (tiles + run - 1) / run;
                if (run < 1 || run > 16) return bad("range", tiles, h, run);
                if (run > 1 && (groups * h < least || (groups * run - tiles) * 8 > tiles)) return bad("short", tiles, h, run);
            }
            for (int per_cu : {1, 2}) {
                const int run = bulk::whole_generations(tiles, h, 256, per_cu);
                const long groups = (tiles + run - 1) / run;
                if (run < 1 || run > 16 || (run - 1) * groups >= tiles) return bad("generations", tiles, h, run);
            }
        }
    return 0;
}
"""

def _program(tmp_path, text, name):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    src, exe = tmp_path / f"{name}.hip", tmp_path / name
    src.write_text(text)
    subprocess.run([hipcc, "--offload-host-only", "-O1", "-std=c++17", "-Wno-unused-command-line-argument", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)], check=True)
    return str(exe)


def test_runs_are_even(tmp_path):
    run = subprocess.run([_program(tmp_path, RUNS, "runs")], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
