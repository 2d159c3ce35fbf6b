"""The single-workgroup bottom of the V-cycle on sets of levels that do not fit
the LDS whole: with the first level's residual, or its residual and f, outside,
and out of global memory (thin levels, whose ghost planes weigh most)."""
import numpy as np
import pytest

from paper_0904_4887_amd import binding as B
from paper_0904_4887_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    return torch


def _opts(n, L, planes, **kw):
    return dict(z_wet_lo=L[2] * (n[2] - planes) / n[2], z_wet_hi=L[2], **kw)


def _lds_bytes(levels, elem, outside):
    """LDS bytes of a bottom set with the first level's residual (outside 1), or
    its residual and f (2), left in global memory."""
    total = 0
    for l, (nx, ny, nw) in enumerate(levels):
        ghosted, interior = nx * ny * (nw + 2), nx * ny * nw
        sizes = [ghosted, ghosted]
        if l > 0 or outside < 2:
            sizes.append(interior)
        if l + 1 < len(levels) and (l > 0 or outside < 1):
            sizes.append(interior)
        total += sum((x + 3) // 4 * 4 for x in sizes)
    return total * elem


def test_coarsest_sweeps_of_thin_sets_run_out_of_lds(torch):
    """(32, 32, 7) over (16, 16, 3) points miss the LDS in float64 and fit it in
    float32.  Either way a sweep of the coarsest level, staged in the LDS, costs
    barriers and LDS accesses: 0.27 us.  Out of global memory it took 1.9 us."""
    n, L = (64, 64, 32), (16.0, 16.0, 8.0)
    levels = B.plan(n, L, **_opts(n, L, 15))["levels"][-2:]
    assert levels == [(32, 32, 7), (16, 16, 3)]
    assert _lds_bytes(levels, 8, 2) > 160 * 1024 >= _lds_bytes(levels, 4, 0)
    eps, r = (torch.from_numpy(a).cuda() for a in W.random_fields(n, 31))
    sweep = {}
    for precision in (0, 1):
        us = {}
        for sweeps in (2, 66):
            s = B.Solver(0)
            s.set_grid(n, L, **_opts(n, L, 15, precision=precision, coarse_sweeps=sweeps, profile=1))
            s.set_epsilon(eps)
            s.apply_split(r)
            best = []
            for _ in range(20):
                s.profile_reset()
                s.apply_split(r)
                best.append(s.profile()["mg_bottom"]["ms"] * 1e3)
            us[sweeps] = min(best)
            s.close()
        sweep[precision] = (us[66] - us[2]) / 64
    assert sweep[0] <= 2 * sweep[1], sweep
