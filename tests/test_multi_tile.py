"""The LDS tiles that the kernels of several steps per launch allocate hold every element that
their phases write, for each number of steps: checked by the compiler on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include <hip/hip_runtime.h>
#include "clbm_multi.h"
// A phase with ring r writes tile r & 1; the phase with r = 0 stores to memory instead.
template <int NS> constexpr unsigned written()
{
    int tiles = 0;
    for (int r = 1; r < NS; ++r)
        if ((r & 1) + 1 > tiles) tiles = (r & 1) + 1;
    return (unsigned)tiles * 14 * clbm::MultiTile<32, 16, NS>::P;
}
#define HOLDS(NS) static_assert(clbm::MultiTile<32, 16, NS>::elems >= written<NS>(), "LDS tile of " #NS " steps")
HOLDS(2);
HOLDS(3);
HOLDS(4);
HOLDS(6);
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_tiles_hold_what_is_written(tmp_path):
    src = tmp_path / "tiles.hip"
    src.write_text(SOURCE)
    r = subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "--offload-host-only",
                        "-I" + os.path.join(ROOT, "paper_1801_04577_amd", "csrc"), str(src)],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
