"""Lists that a kernel builds in LDS: every workgroup's entries fit the room its launcher gives it (CPU: the rules are host code)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PROGRAM = r"""
#include "conv_plan.h"
#include <vector>
using namespace dcnn;
static int bad = 0;
#define BAD(...) do { if (++bad < 10) printf(__VA_ARGS__); } while (0)

// the list that the plain convolution kernel cuts up (windows other than 1x1 and 3x3): entries of the groups a workgroup walks, by the
// kernel's rule, against the room that its launcher gives it
static void list(int px, int count, int slots, int grid, int spread) {
    const int64_t room = self_local_entries(px, slots * kTile, grid);
    const uint32_t ntiles = (uint32_t)cdiv(count, kTile);
    const int tiles = ws_slots(ntiles, spread, slots);
    const int64_t groups = cdiv(count, tiles * kTile);
    for (int b = 0; b < grid; ++b) {
        const WgTileRange r = tile_range(groups, b, grid);
        const int64_t mine = r.begin < r.end ? (r.end - r.begin + r.step - 1) / r.step : 0;
        if (mine * tiles * kTile > room)
            BAD("list of %d of %d pixels, workgroup %d of %d: %d entries, room for %d\n", count, px, b, grid, (int)(mine * tiles * kTile), (int)room);
    }
}
// blocks that workgroups compact for themselves: every pixel has one owner, within its slots, and the entries it walks have room
static void blocks(const char* what, int px, int shift, int cap, int group, int tiles) {
    const LocalShape s = local_shape(px, shift, cap, group);
    if (s.owners < 1 || s.owners > cap || s.entries < s.slots || s.entries % group != 0 || s.slots % (1 << shift) != 0)
        BAD("%s: %d pixels: %d owners, %d slots, %d entries\n", what, px, s.owners, s.slots, s.entries);
    std::vector<uint8_t> seen(px);
    for (int owner = 0; owner < s.owners; ++owner)
        for (int slot = 0; slot < s.slots; ++slot) {
            const int p = ((owner + (slot >> shift) * s.owners) << shift) + (slot & ((1 << shift) - 1));
            if (p < px) ++seen[p];
        }
    for (int p = 0; p < px; ++p)
        if (seen[p] != 1) { BAD("%s: pixel %d of %d has %d owners\n", what, p, px, seen[p]); break; }
    // (rounds of up to `tiles` tiles, fewer where the workgroup lists fewer)
    for (int count = 1; tiles > 0 && count <= s.slots; ++count) {
        const int n = (int)cdiv(count, kTile), per = n < tiles ? n : tiles;
        if ((int)cdiv(n, per) * per * kTile > s.entries) BAD("%s: %d entries in rounds of %d tiles, room for %d\n", what, count, per, s.entries);
    }
}
int main() {
    const int cus = 256;
    for (int px = 1; px <= 2500; px += px < 300 ? 1 : 13)
        for (int slots = 1; slots <= 8; slots *= 2)
            for (int cap : {cus, 2 * cus, 4 * cus}) {
                const int tiles = (int)cdiv(px, kTile), want = (int)cdiv(tiles, slots);
                const int spread_out = want < cus ? (tiles < cus ? tiles : cus) : want;           // (resident weights)
                for (int w : {want, spread_out}) {
                    const int grid = (int)(cdiv(w < cap ? w : cap, kXcd) * kXcd);
                    for (int count : {1, px / 3 + 1, px / 2 + 1, px - 1, px})
                        if (count >= 1 && count <= px) list(px, count, slots, grid, grid < cus ? grid : cus);
                }
            }
    for (int px = 1; px <= (int)kLocalMaxPixels; px += px < 1000 ? 1 : (px < 17000 ? 331 : 3989)) {
        for (int tiles = 1; tiles <= 8; tiles *= 2)
            for (int cap : {cus, 2 * cus, 4 * cus})
                for (int writers : {0, 1, 8})
                    blocks("convolution", px, conv_local_shift(px, cap), cap - writers, tiles * kTile, tiles);
        for (int run = 1; run <= kTile; run *= 2) blocks("activation, depthwise", px, tile_local_shift(px, kTileWaves * run), INT32_MAX, kTileWaves * run, 0);
        blocks("wide activation", px, tile_local_shift(px, kWideRun), INT32_MAX, kWideRun, 0);
        blocks("upsampling", px, tile_local_shift(px, 32), INT32_MAX, 32, 0);
    }
    return bad ? 1 : 0;
}
"""
RUNS = r"""
#include "common.h"
#include <vector>
using namespace dcnn;
int main() {
    int bad = 0;
    for (int cus : {256, 32})
        for (int rest : {1, 2, 3, 8, 16, 32})
            for (int px = 1; px <= (int)kSelfMaxPixels; px += px < 1500 ? 1 : 251) {
                const int runs = (int)cdiv(px, kRunPixels), parts = run_parts(px, rest, 4 * (int64_t)cus);
                std::vector<int> seen(runs * parts);
                for (int item = 0; item < runs * parts; ++item) {
                    const RunPart rp = run_part(item, runs, parts);
                    if (rp.run < 0 || rp.run >= runs || rp.part < 0 || rp.part >= parts || seen[rp.run * parts + rp.part]++) ++bad;
                }
                if (kRunTiles % parts != 0) ++bad;
            }
    for (int parts = 1; parts <= kRunTiles; parts *= 2)
        for (int even = 0; even < 2; ++even)
            for (int count = 0; count <= kRunPixels; ++count) {
                const int share = run_share(count, parts, even);
                if (share * parts < count || (!even && share % kTile != 0) || (count > 0 && share < 1)) ++bad;
                if (parts == kRunTiles && share > kTile) ++bad;         // a tile each
            }
    if (bad) printf("%d\n", bad);
    return bad ? 1 : 0;
}
"""


def test_every_run_and_share_has_one_workgroup(tmp_path):
    """Runs of pixels that several workgroups divide: each (run, part) belongs to one workgroup, and the shares hold all entries."""
    _run(tmp_path, RUNS)


def test_every_workgroups_entries_fit(tmp_path):
    _run(tmp_path, PROGRAM)


def _run(tmp_path, program):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "rooms.cpp", tmp_path / "rooms"
    src.write_text(program)
    inc = os.path.join(ROOT, "paper_2203_03996_amd", "csrc")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", f"-I{inc}", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
