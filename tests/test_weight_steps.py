"""The wave-uniform part of a weight load's offset stays inside the packed weights, on padding steps too (CPU: the rule is plain C++)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <cstdio>
#include "kstep.h"
using namespace dcnn;
int main() {
    int bad = 0;
    for (int k = 1; k <= 7; k += 2)
        for (int kch = 1; kch <= 70; ++kch) {
            const int taps = k * k, ksteps = taps * kch;       // weights of one channel group: the least a descriptor covers
            for (int tap = 0; tap < taps; ++tap)               // groups of four K-steps of a tap
                for (int step = 0; step < (kch + 3) / 4 * 4; ++step) {
                    const int at = weight_step(tap, kch, step);
                    if (at < 0 || at >= ksteps || (step < kch && at != tap * kch + step)) ++bad;
                }
            if (kch > 1) continue;                             // groups of four taps of one K-step each
            for (int step = 0; step < (taps + 3) / 4 * 4; ++step) {
                const int at = weight_step(0, taps, step);
                if (at < 0 || at >= taps || (step < taps && at != step)) ++bad;
            }
        }
    printf("%d\n", bad);
    return bad != 0;
}
"""


def test_weight_steps_stay_inside_the_packed_weights(tmp_path):
    src = tmp_path / "steps.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "steps"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2203_03996_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, f"{r.stdout.strip()} steps outside"
