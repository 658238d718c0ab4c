"""The pointer block that the small-context kernels take by value (CPU only): every
64-bit address comes back as it went in, and a launch's addresses share their
upper 16 bits."""
import ctypes
import os
import subprocess

import pytest

from paper_2310_12298_amd import jorge as J

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PROGRAM = r"""
#include <cstdio>
#include "jorge_types.hpp"
using namespace jorge;
static const float* at(uint64_t v) { return reinterpret_cast<const float*>(v); }
static float* out(uint64_t v) { return reinterpret_cast<float*>(v); }
int main() {
    const uint64_t low[4] = {0x7f1234567890ull, 0x10ull, 0xfffffffffff0ull, 0x0000800000000000ull};
    for (uint64_t g : {0ull, 0x0100000000000000ull, 0xffff000000000000ull})
        for (uint64_t p : {0ull, 0x00ab000000000000ull}) {
            PtrPack pp{};
            for (int i = 0; i < kPtrBatch; ++i)
                if (!pp.set(i, at(g | low[i % 4]), out(p | low[(i + 1) % 4]))) return 1;
            for (int i = 0; i < kPtrBatch; ++i)
                if (pp.get(2 * i) != (g | low[i % 4]) || pp.get(2 * i + 1) != (p | low[(i + 1) % 4])) return 2;
            // Another upper part is for the next launch, and leaves this one's as they are.
            if (pp.set(3, at(g ^ 0x0001000000000000ull), out(p)) || pp.set(3, at(g), out(p ^ 0x0001000000000000ull)))
                return 3;
            if (pp.get(6) != (g | low[3]) || pp.get(7) != (p | low[0])) return 4;
        }
    static_assert(sizeof(PtrPack) + 128 <= 4096, "the block and a kernel's other arguments");
    std::puts("ok");
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="needs hipcc")
def test_every_address_survives_packing(tmp_path):
    src, exe = tmp_path / "pack.hip", tmp_path / "pack"
    src.write_text(PROGRAM)
    subprocess.run([HIPCC, "--offload-host-only", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2310_12298_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout == "ok\n", (res.returncode, res.stdout)


@pytest.mark.skipif(os.path.exists("/dev/kfd"), reason="made-up addresses: only where no GPU could follow them")
@pytest.mark.parametrize("shape", [(48, 40), (256, 300)])
def test_no_address_is_refused(shape):
    """The call gets past its checks, to the missing GPU, with addresses above 48 bits."""
    lib = J.load_library()
    high = [ctypes.c_void_p((0x0100 << 48) + 4096 * (i + 1)) for i in range(6)]
    args = (ctypes.byref(J.Shape(*shape)), None, 1, *high, 0.1, 0.9, 0.9, 0.0, None)
    assert lib.jorge_step_noalloc(*args) == -3      # a HIP error, not "unsupported"
