"""The packed count of a dotting stencil's partial sums (CPU): what its readers cannot add is refused, not dropped."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0910_1048_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r"""
#include "sgn_internal.h"
using namespace sgn;
static bool refused(int n, int width)
{
    try {
        const int p = pack_partials(n, width);
        return !(partial_count(p) == n && partial_width(p) == width);
    } catch (const Failure &) {
        return true;
    }
}
int main()
{
    const int most = 0xFFFFFF;
    if (refused(0, 1) || refused(1, 1) || refused(5, 3) || refused(most, kMaxPartialWidth)) return 1;
    return refused(most + 1, 1) && refused(1, kMaxPartialWidth + 1) && refused(1, 0) && refused(-1, 1) ? 0 : 2;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_packing_refuses_what_the_readers_would_drop(tmp_path):
    src, exe = str(tmp_path / "d.cpp"), str(tmp_path / "d")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, src, "-o", exe], check=True)
    assert subprocess.run([exe]).returncode == 0


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
@pytest.mark.parametrize("threads,fits", [(256, True), (704, True), (768, False)])
def test_a_block_of_more_wavefronts_does_not_compile(threads, fits):
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-fsyntax-only", "-std=c++17",
                        "-w", f"-DSGN_STENCIL_THREADS={threads}", "-I" + os.path.join(ROOT, "include"),
                        os.path.join(CSRC, "dslash.hip")], capture_output=True, text=True)
    assert (r.returncode == 0) == fits, r.stderr[-2000:]
    assert fits or "kMaxPartialWidth entries at most" in r.stderr
