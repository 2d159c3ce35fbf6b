"""Host work of a launch: what the library asks the runtime for each time."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_COUNT = """
#include <dlfcn.h>
#include <stddef.h>
static int n;
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *fn, int threads, size_t lds) {
    static int (*real)(int *, const void *, int, size_t);
    if (!real) real = dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    ++n;
    return real(blocks, fn, threads, lds);
}
int queries(void) { return n; }
"""

_RUN = """
import ctypes, sys
# loaded before the HIP runtime, so that the library binds to this function
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import torch
from paper_0904_4887_amd import workloads as W
from paper_0904_4887_amd.binding import Solver
sizes = [(x, y, 48) for x in (32, 48, 64, 72, 96, 128, 144, 192) for y in (48, 64)]
again = 0
for n in sizes:
    L = (0.3 * n[0], 0.25 * n[1], 0.4 * n[2])
    eps, r = (torch.from_numpy(a).cuda() for a in W.random_fields(n, 31))
    for precision in (0, 1):
        s = Solver(0)
        s.set_grid(n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=precision)
        s.set_epsilon(eps)
        s.apply_split(r)
        first = shim.queries()
        s.apply_split(r)
        again += shim.queries() - first
        s.close()
assert first > 64, first
assert again == 0, again
print("ok")
"""


def test_occupancy_is_asked_for_once_a_block_shape(tmp_path):
    """Also in a process that has used more than a few grids."""
    src, so = tmp_path / "count.c", tmp_path / "count.so"
    src.write_text(_COUNT)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src), "-ldl"], check=True)
    p = subprocess.run([sys.executable, "-c", _RUN, str(so)], cwd=ROOT, capture_output=True, text=True, timeout=110)
    assert p.returncode == 0 and p.stdout.endswith("ok\n"), p.stdout + p.stderr
