"""Lists that a kernel builds in LDS: every workgroup's entries fit the room its launcher gives it (CPU: the rules are host code)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PROGRAM = r"""
#include "common.h"
using namespace dcnn;
static int bad = 0;
// the groups a workgroup walks, by the kernels' rules, against the entries there is room for
static void check(const char* what, int px, int count, int64_t room_groups, int64_t groups, int64_t entries, int grid, bool per_xcd) {
    const int64_t room = self_local_entries(room_groups * entries, entries, grid, per_xcd);
    for (int b = 0; b < grid; ++b) {
        int64_t mine = 0;
        if (per_xcd) {
            const WgTileRange r = tile_range(groups, b, grid);
            mine = r.begin < r.end ? (r.end - r.begin + r.step - 1) / r.step : 0;
        } else {
            mine = b < groups ? (groups - b + grid - 1) / grid : 0;
        }
        if (mine * entries > room && ++bad < 10)
            printf("%s: %d pixels, %d listed, workgroup %d of %d: %d entries, room for %d\n", what, px, count, b, grid, (int)(mine * entries), (int)room);
    }
}
int main() {
    const int num_cu = 256;
    auto up8 = [](int64_t g) { return (int)(cdiv(g, kXcd) * kXcd); };
    auto least = [](int64_t a, int64_t b) { return a < b ? a : b; };
    for (int px = 1; px <= (int)kSelfMaxPixels; px += px < 4096 ? 1 : 61) {
        const int counts[] = {1, px / 2, px - 1, px};
        for (int count : counts) {
            if (count < 1) continue;
            check("wide activation", px, count, wide_groups(px), wide_groups(count), kWideRun, (int)least(wide_groups(px), num_cu * 8), false);
            check("upsampling", px, count, cdiv(px, 32), cdiv(count, 32), 32, (int)least(cdiv(px, 32), num_cu * 4), false);
            for (int run = 8; run <= kTile; run *= 2)
                check("activation, depthwise", px, count, run_groups(px, run), run_groups(count, run), kTileWaves * run,
                      up8(least(cdiv(px, kTileWaves * run), num_cu * 4)), true);
            for (int tiles = 1; tiles <= 16; ++tiles)                        // convolutions: whole tiles, per XCD
                for (int cap : {num_cu, 2 * num_cu, 4 * num_cu})
                    check("convolution", px, count, cdiv(px, tiles * kTile), cdiv(cdiv(count, kTile), tiles), tiles * kTile,
                          up8(least(cdiv(px, tiles * kTile), cap)), true);
        }
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
