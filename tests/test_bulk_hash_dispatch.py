"""Host rules of the bulk hash, compiled for the CPU: how the tiles of a head are shared out over workgroups, and
which calls stay with the vector-ALU kernels because those are faster there."""
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

SHARES = r"""
#include <stdio.h>
#include <vector>
#include "hash_bulk.h"
using namespace spotlight;
int main()
{
    const long some[] = {1, 2, 3, 5, 8, 9, 16, 17, 31, 63, 100, 127, 128, 129, 313, 625, 2047, 4097};
    for (long tiles : some)
        for (int heads : {1, 3, 4, 28, 32, 255, 256, 300, 512, 600})
            for (int per_cu : {1, 2}) {
                const bulk::Shares s = bulk::shares_of(tiles, heads, 256, per_cu);
                std::vector<char> seen(tiles * heads, 0);
                int before = 1 << 30, longest = 0, shortest = 1 << 30;
                for (unsigned id = 0; id < static_cast<unsigned>(s.parts) * heads; ++id) {
                    const bulk::Share w = bulk::share_of(id, s.parts, heads, s.run, s.longer);
                    if (w.head < 0 || w.head >= heads || w.tiles > before || w.tile >= tiles) { printf("share %u of %ld x %d\n", id, tiles, heads); return 1; }
                    before = w.tiles;
                    longest = w.tiles > longest ? w.tiles : longest;
                    shortest = w.tiles < shortest ? w.tiles : shortest;
                    for (long t = w.tile; t < w.tile + w.tiles && t < tiles; ++t)
                        if (seen[w.head * tiles + t]++) { printf("tile twice: %ld x %d, %ld\n", tiles, heads, t); return 1; }
                }
                for (char c : seen) if (c != 1) { printf("tile left out: %ld x %d\n", tiles, heads); return 1; }
                if (longest > 17 || longest - shortest > 1 || (s.longer && s.parts * heads > 256 * per_cu)) { printf("runs: %ld x %d: %d %d %d\n", tiles, heads, s.parts, s.run, s.longer); return 1; }
            }
    // open rows: one generation where the segments allow it
    for (long segments : {1, 2, 16, 56, 64, 300, 512, 4096}) {
        const int parts = bulk::open_parts(segments, 512);
        if (parts < 1 || parts > 512 || (segments <= 64 && (segments * parts > 512 || segments * (parts + 1) <= 512))) { printf("open %ld: %d\n", segments, parts); return 1; }
    }
    return 0;
}
"""

ROUTES = r"""
#include <stdio.h>
#include <string.h>
#include "hash_bulk.h"
using namespace spotlight;
int main(int argc, char** argv)
{
    int heads, rows, bits, hidden, x_size, w_size;
    while (scanf("%d %d %d %d %d %d", &heads, &rows, &bits, &hidden, &x_size, &w_size) == 6) {
        spotlight_ctx ctx;
        memset(&ctx, 0, sizeof(ctx));
        ctx.n_cus = 256;
        ctx.max_lds = 160 * 1024;
        hashdev::HashArgs a;
        memset(&a, 0, sizeof(a));
        float scratch;
        a.wnorm = &scratch;
        a.n_rows = rows; a.hidden = hidden; a.L = bits; a.W = bits / 32;
        printf("%d\n", bulk_hash_applies(&ctx, a, heads, x_size, w_size) ? 1 : 0);
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


def test_every_tile_belongs_to_one_workgroup(tmp_path):
    run = subprocess.run([_program(tmp_path, SHARES, "shares")], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_routes(tmp_path):
    """(heads, rows, bits, hidden, weight bytes) -> whether the matrix-core kernels take the call."""
    routes = {
        (8, 8, 128, 256, 2): 0, (8, 9, 128, 256, 2): 1, (512, 16, 128, 256, 2): 0, (512, 17, 128, 256, 2): 1,
        (8, 31, 512, 0, 2): 0, (8, 32, 512, 0, 2): 1,
        (8, 31, 64, 256, 2): 0, (8, 31, 96, 256, 2): 1, (8, 32, 64, 256, 2): 1, (512, 18, 64, 256, 2): 1, (8, 20, 64, 128, 2): 1,
        # long codes behind a narrow layer of binary32 weights, few vectors
        (8, 17, 512, 64, 4): 0, (8, 17, 1024, 128, 4): 0, (8, 17, 384, 64, 4): 1, (8, 17, 512, 136, 4): 1, (8, 32, 512, 64, 4): 1,
        (8, 17, 512, 64, 2): 1, (512, 17, 512, 64, 4): 1,
        # one word behind a wide layer of bfloat16 weights
        (512, 24, 32, 512, 2): 0, (512, 25, 32, 512, 2): 1, (512, 24, 32, 256, 2): 1, (512, 24, 32, 512, 4): 1, (512, 24, 64, 512, 2): 1,
        (512, 24, 32, 1152, 2): 1,
        # a word or more for every hidden unit, on large grids
        (512, 90, 512, 16, 4): 0, (512, 90, 1024, 16, 2): 0, (512, 90, 384, 16, 4): 1, (512, 90, 512, 16, 2): 1, (512, 32, 1024, 16, 4): 1,
        (8, 300, 1024, 16, 4): 1, (8, 4000, 1024, 16, 4): 0, (512, 90, 1024, 64, 4): 1,
        # what LDS holds
        (8, 64, 128, 1152, 4): 1, (8, 64, 128, 1224, 4): 0,
    }
    text = "\n".join(f"{h} {r} {b} {n} 2 {w}" for h, r, b, n, w in routes)
    run = subprocess.run([_program(tmp_path, ROUTES, "routes")], input=text, capture_output=True, text=True, check=True)
    got = dict(zip(routes, map(int, run.stdout.split())))
    assert got == routes
