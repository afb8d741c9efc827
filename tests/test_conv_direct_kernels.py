"""The register-blocked convolution kernels that are built: those that a plan can ask for, fp16 ones within the registers (CPU: metadata of the
built library's code objects, and the host's rule for plans)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PLANS = r"""
#include "conv_plan.h"
using namespace dcnn;
int main() {
    int bad = 0, seen[4] = {};
    for (int dtype : {DCNN_F16, DCNN_F32})
        for (int k : {1, 3})
            for (int full = 0; full < 2; ++full)
                for (int cin = 4; cin <= 8192; cin += cin < 512 ? 4 : 260)
                    for (int cout = 4; cout <= 8192; cout += cout < 1100 ? 4 : 116) {
                        const ConvPlan p = conv_plan(dtype, k, cin, cout, full);
                        if (!p.ok || !p.stream || cout % (dtype == DCNN_F16 ? 8 : 4) != 0) continue;
                        ++seen[p.nb - 1];
                        if (p.nb > 3 || (p.nb == 1 && p.cs != 1) || (p.cs != 1 && p.cs != 2 && p.cs != 4)) {
                            if (++bad < 10) printf("%d: %dx%d %d->%d: %d blocks, %d waves\n", dtype, k, k, cin, cout, p.nb, p.cs);
                        }
                    }
    if (!seen[0] || !seen[1] || !seen[2]) { ++bad; printf("seen %d %d %d\n", seen[0], seen[1], seen[2]); }
    return bad != 0;
}
"""


def kernels(path):
    """Metadata of every kernel in the code objects that a library embeds."""
    data = open(path, "rb").read()
    for m in re.finditer(b"\x7fELF", data):
        elf = data[m.start():]
        if len(elf) < 64 or struct.unpack_from("<H", elf, 18)[0] != 224:     # EM_AMDGPU
            continue
        sections, count = struct.unpack_from("<Q", elf, 40)[0], struct.unpack_from("<H", elf, 60)[0]
        for i in range(count):
            kind = struct.unpack_from("<I", elf, sections + 64 * i + 4)[0]
            at, size = struct.unpack_from("<QQ", elf, sections + 64 * i + 24)
            end = at + size
            while kind == 7 and at < end:                                    # SHT_NOTE
                name, desc, note = struct.unpack_from("<III", elf, at)
                body = at + 12 + (name + 3) // 4 * 4
                if note == 32:                                               # NT_AMDGPU_METADATA
                    yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
                at = body + (desc + 3) // 4 * 4


def test_fp16_kernels_keep_their_sums_in_registers():
    import paper_2203_03996_amd as pkg
    if not os.path.exists(pkg.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    scratch = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels(pkg.LIB_PATH) if "conv_direct_kernelIDF16_" in k[".name"]}
    # <blocks, window, waves to a tile, list built in place>: one block 1, two and three blocks 1, 2, 4 waves
    assert len(scratch) == 7 * 2 * 2
    assert not {n: b for n, b in scratch.items() if b}


def test_streamed_plans_ask_for_kernels_that_are_built(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "plans.cpp", tmp_path / "plans"
    src.write_text(PLANS)
    inc = os.path.join(ROOT, "paper_2203_03996_amd", "csrc")
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", f"-I{inc}", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
