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

CHAINS = r"""
#include <stdio.h>
#include "hash_open.h"
using namespace spotlight;
int main()
{
    for (int n = 0; n <= screen::kChains; ++n) {
        const int lanes = 64 * screen::chain_waves(n);
        if (n > lanes || lanes > 64 * screen::kOpenWaves) { printf("%d chains, %d lanes\n", n, lanes); return 1; }
    }
    return 0;
}
"""

QUOTA = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "hash_bulk.h"
using namespace spotlight;
int main()
{
    for (int slots : {256, 512, 768})
        for (int n : {1, 2, 3, 8, 56, 64, 100, 128, slots / 2})
            for (int kind = 0; kind < 6; ++kind) {
                std::vector<int> tiles(n);
                for (int s = 0; s < n; ++s) tiles[s] = kind == 0 ? 2048 : kind == 1 ? rand() % 2049 : kind == 2 ? (s == n / 2 ? 2048 : 1) : kind == 3 ? (s == 0) : kind == 4 ? 190 + rand() % 9 : (s % 3 ? 0 : 577);
                int total = 0;
                for (int t : tiles) total += t;
                if (total == 0) continue;
                auto parts_with = [&](int q) { int p = 0; for (int t : tiles) p += (t + q - 1) / q; return p; };
                const int q = bulk::open_quota(total, n, slots, parts_with);
                if (q < 1 || parts_with(q) > slots || (q > 1 && parts_with(q - 1) <= slots)) { printf("%d segments, %d slots, kind %d: %d\n", n, slots, kind, q); return 1; }
                unsigned used = 0;
                for (int t : tiles) {
                    const unsigned w = bulk::open_workgroups(t, q, parts_with(q), slots);
                    used += w;
                    if ((t == 0) != (w == 0) || static_cast<unsigned>(t) > w * q || w > static_cast<unsigned>(t)) { printf("%d segments, %d slots, kind %d: %d tiles, %u\n", n, slots, kind, t, w); return 1; }
                }
                if (used > static_cast<unsigned>(slots)) { printf("%d segments, %d slots, kind %d: %u workgroups\n", n, slots, kind, used); return 1; }
            }
    return 0;
}
"""

WALK = r"""
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "hash_bulk.h"
using namespace spotlight;
using Bits = std::vector<uint32_t>;
struct Seen { std::vector<int> rows; int advances = 0, fullest = 0; };
// OpenWalk of one share, its lanes in turn; the bitmap is `counted` in the beginning and `met` afterwards.  False: out of range, or no end.
static bool walk(const Bits& counted, const Bits& met, int n_rows, int part, int parts, Seen& seen)
{
    constexpr int kEntries = sizeof(bulk::OpenRows::row) / sizeof(uint16_t);
    std::vector<uint16_t> list(kEntries + 64, 0xfffe);
    const int n_words = (n_rows + 31) / 32;
    int total = 0;
    for (int w = 0; w < n_words; ++w) total += __builtin_popcount(bulk::open_word(counted.data(), w, n_rows));
    const bulk::OpenShare share = bulk::open_share(total, part, parts);
    if (share.from >= share.to) return true;
    int next = 0, skip = share.from;
    while (skip >= __builtin_popcount(bulk::open_word(counted.data(), next, n_rows))) skip -= __builtin_popcount(bulk::open_word(counted.data(), next++, n_rows));
    int count = 0, tiles = 0, left = share.to - share.from;
    while (left > 0) {
        if (++seen.advances > n_words / 64 + 2) return false;
        const int rest = count - tiles * bulk::kTile;
        if (rest < 0 || rest >= bulk::kTile) return false;
        for (int r = 0; r < rest; ++r) list[r] = list[tiles * bulk::kTile + r];
        int upto = 0;
        for (int lane = 0; lane < 64; ++lane) {
            const uint32_t bits = bulk::open_word(met.data(), next + lane, n_rows);
            bulk::list_rows(list.data(), bits, next + lane, rest, upto - skip, left);
            upto += __builtin_popcount(bits);
        }
        const bulk::OpenSpan s = bulk::after_span(rest, upto - skip, left, next + 64, n_rows);
        next += 64, skip = 0;
        count = s.count, left = s.left, tiles = s.tiles;
        if (count < 0 || count > kEntries || tiles * bulk::kTile > (count + 31) / 32 * 32 || (tiles == 0 && left == 0 && count > 0)) return false;
        for (size_t e = kEntries; e < list.size(); ++e) if (list[e] != 0xfffe) return false;
        seen.fullest = count > seen.fullest ? count : seen.fullest;
        const int whole = left > 0 ? tiles * bulk::kTile : count;
        for (int e = 0; e < whole; ++e) {
            if (list[e] >= n_rows) return false;
            seen.rows.push_back(list[e]);
        }
    }
    return true;
}
static Bits random_bits(int words, int of_256) { Bits b(words, 0); for (auto& w : b) for (int i = 0; i < 32; ++i) w |= (rand() % 256 < of_256 ? 1u : 0u) << i; return b; }
int main()
{
    int most = 0, fullest = 0;
    for (int n_rows : {1, 31, 32, 33, 2047, 2048, 2049, 4700, 30001, 65536}) {
        const int words = (n_rows + 31) / 32;
        for (int parts : {1, 2, 7, 128, 512})
            for (int of_256 : {0, 1, 24, 128, 255, 256}) {
                const Bits open = random_bits(words, of_256);
                std::vector<int> want, got;
                for (int r = 0; r < n_rows; ++r) if (open[r / 32] >> (r % 32) & 1) want.push_back(r);
                for (int part = 0; part < parts; ++part) {
                    Seen seen;
                    if (!walk(open, open, n_rows, part, parts, seen)) { printf("range: %d rows, part %d of %d, %d\n", n_rows, part, parts, of_256); return 1; }
                    got.insert(got.end(), seen.rows.begin(), seen.rows.end());
                    most = seen.advances > most ? seen.advances : most;
                    fullest = seen.fullest > fullest ? seen.fullest : fullest;
                    // a bitmap that changes after it has been counted: it ends, in range
                    for (int met : {0, 3, 128, 256}) {
                        Seen other;
                        if (!walk(open, random_bits(words, met), n_rows, part, parts, other)) { printf("changed: %d rows, part %d of %d, %d then %d\n", n_rows, part, parts, of_256, met); return 1; }
                    }
                    if (parts > 7 && part > 9 && part < parts - 9) part += 50, got.clear(), want.clear();   // (a few of many shares)
                }
                if (got != want && parts <= 7) { printf("rows: %d, %d parts, %d\n", n_rows, parts, of_256); return 1; }
            }
    }
    Bits open(2048, ~0u);     // one row short of a span: 31 rows wait in front of the next 2048
    open[3] = 0xfffffffeu;
    Seen seen;
    if (!walk(open, open, 65536, 0, 1, seen) || seen.rows.size() != 65535) { printf("all open but one\n"); return 1; }
    fullest = seen.fullest > fullest ? seen.fullest : fullest;
    if (most < 32 || fullest != 2079) { printf("advances %d, list %d\n", most, fullest); return 1; }
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

TWO_PASSES = r"""
#include <stdio.h>
#include <string.h>
#include "hash_open.h"
using namespace spotlight;
int main()
{
    int heads, rows, bits, hidden;
    while (scanf("%d %d %d %d", &heads, &rows, &bits, &hidden) == 4) {
        spotlight_ctx ctx;
        memset(&ctx, 0, sizeof(ctx));
        ctx.n_cus = 256;
        ctx.max_lds = 160 * 1024;
        hashdev::HashArgs a;
        memset(&a, 0, sizeof(a));
        float scratch;
        uint32_t open;
        a.wnorm = &scratch;
        a.open = &open;
        a.n_rows = rows; a.hidden = hidden; a.L = bits; a.W = bits / 32;
        const bool two = screen::applies(&ctx, a, heads);
        uint32_t counts;
        a.open_counts = two && bulk::counts_open_rows(a, heads, ctx.n_cus) ? &counts : nullptr;
        for (int slots : {256, 512, 768}) {     // shared out by count, or the same number of workgroups for every segment
            const bulk::OpenGrid g = bulk::open_grid(a, heads, slots);
            const long segments = (rows + 65535) / 65536;
            if (a.open_counts && 2 * segments * heads <= slots ? g.run != -heads || (int)g.grid.x != slots : g.run < 1 || g.grid.x != segments * g.run || (int)g.grid.y != heads) { printf("grid\n"); return 1; }
        }
        printf("%d %d %d\n", two, two && screen::resident(hidden, a.W), two && screen::open_serves(hidden, a.W));
        a.open = nullptr;
        if (screen::applies(&ctx, a, heads)) printf("without room for a bitmap\n");
        a.open = &open, a.wnorm = nullptr;
        if (screen::applies(&ctx, a, heads)) printf("with the matrix cores switched off\n");
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


def test_open_rows_are_shared_out_over_the_heads(tmp_path):
    """As few tiles for a workgroup as the chip's workgroups allow, whichever heads the open rows are in, and none for no tile."""
    run = subprocess.run([_program(tmp_path, QUOTA, "quota")], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_no_lane_runs_two_chains_of_a_list(tmp_path):
    run = subprocess.run([_program(tmp_path, CHAINS, "chains")], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout


def test_open_rows_are_walked_once_and_to_an_end(tmp_path):
    """The second pass's walk over the rows left open: every row in one share and once, also over full lists with a partial tile in
    front of them; and an end in range where another call on the same context has changed the bitmap meanwhile."""
    run = subprocess.run([_program(tmp_path, WALK, "walk")], capture_output=True, text=True, timeout=100)
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


def test_routes_of_two_passes(tmp_path):
    """(heads, rows, bits, hidden) of bfloat16 vectors and weights -> whether two passes take the call, whether the first holds all weights in
    LDS, whether hash_open_kernel is the second: the shapes of the GPU tests, whose kernels these decide, and both sides of every line."""
    routes = {
        # every kernel of either pass
        (8, 16400, 32, 16): "1 1 0", (8, 16400, 64, 32): "1 1 0", (8, 16400, 96, 48): "1 1 0", (8, 16400, 128, 128): "1 1 0", (8, 16400, 160, 112): "1 1 0",
        (8, 16400, 256, 128): "1 1 0", (8, 16400, 64, 144): "1 1 0", (8, 16400, 128, 256): "1 1 0", (8, 16400, 192, 256): "1 0 0", (8, 16400, 160, 288): "1 0 1",
        (8, 16400, 256, 400): "1 0 1", (8, 16400, 128, 512): "1 0 0", (8, 16400, 256, 512): "1 0 1", (8, 16400, 224, 528): "1 0 0", (8, 16400, 256, 1008): "1 0 0",
        (8, 16400, 32, 1024): "1 0 0", (8, 16400, 96, 80): "1 1 0", (8, 16384, 160, 272): "1 0 1", (8, 16384, 160, 256): "1 0 0", (8, 16384, 128, 288): "1 1 0", (8, 16384, 128, 304): "1 0 0",
        # grids of other shapes
        (1, 131073, 64, 64): "1 1 0", (3, 43700, 64, 64): "1 1 0", (512, 256, 64, 64): "1 1 0", (512, 257, 64, 64): "1 1 0", (300, 511, 64, 64): "1 1 0",
        (300, 513, 64, 64): "1 1 0", (28, 4703, 64, 64): "1 1 0", (2, 65600, 64, 64): "1 1 0", (2, 65600, 256, 512): "1 0 1", (2, 33000, 256, 512): "1 0 1",
        (9, 66000, 256, 64): "1 1 0", (66, 2100, 64, 64): "1 1 0", (200, 700, 256, 512): "1 0 1", (1, 70000, 64, 64): "1 1 0", (1024, 4133, 32, 1024): "1 0 0",
        (1024, 4133, 256, 512): "1 0 1", (512, 256, 32, 1024): "1 0 0",
        # eight tiles for every compute unit, a round of a workgroup
        (1, 65505, 64, 64): "1 1 0", (1, 65504, 64, 64): "0 0 0", (512, 255, 64, 64): "0 0 0", (255, 256, 64, 64): "0 0 0", (256, 256, 64, 64): "1 1 0",
        # long codes, weights not in LDS: rounds of the first pass that are half empty
        (300, 257, 256, 256): "0 0 0", (257, 288, 256, 256): "0 0 0", (256, 300, 256, 256): "0 0 0", (300, 384, 256, 256): "0 0 0", (200, 352, 256, 256): "1 0 0",
        (257, 511, 256, 256): "1 0 0", (300, 257, 256, 512): "0 0 0", (300, 384, 256, 512): "1 0 1", (228, 257, 256, 512): "1 0 1", (300, 257, 160, 1024): "0 0 0",
        (300, 257, 128, 256): "1 1 0", (300, 257, 128, 512): "1 0 0", (300, 257, 256, 128): "1 1 0",
        # networks
        (8, 16400, 288, 256): "0 0 0", (8, 16400, 128, 264): "0 0 0", (8, 16400, 128, 1040): "0 0 0", (8, 16400, 512, 0): "0 0 0", (8, 16400, 32, 8): "0 0 0",
    }
    text = "\n".join(" ".join(map(str, r)) for r in routes)
    run = subprocess.run([_program(tmp_path, TWO_PASSES, "two_passes")], input=text, capture_output=True, text=True, check=True)
    got = dict(zip(routes, run.stdout.strip().split("\n")))
    assert len(run.stdout.strip().split("\n")) == len(routes), run.stdout
    assert got == routes
