"""The single-workgroup bottom of the V-cycle on sets of levels that do not fit
the LDS whole: with the first level's residual, or its residual and f, outside,
and out of global memory (thin levels, whose ghost planes weigh most)."""
import numpy as np
import pytest

import oracle as O
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


# -------------------------------------------------- V-cycles written out
# Levels as (eps with the planes below and above, h); u and f hold the interior.

def _neighbours(m, below, above):
    return (np.roll(m, -1, 2), np.roll(m, 1, 2), np.roll(m, -1, 1), np.roll(m, 1, 1),
            np.concatenate([m[1:], above[None]]), np.concatenate([below[None], m[:-1]]))


def _weights(eps, h):
    return [0.5 / h[q // 2]**2 * (eps[1:-1] + e) for q, e in enumerate(_neighbours(eps[1:-1], eps[0], eps[-1]))]


def _off(w, u):
    zero = np.zeros_like(u[0])
    return sum(a * b for a, b in zip(w, _neighbours(u, zero, zero)))


def _sweeps(u, f, w, colours, times):
    k, j, i = np.indices(u.shape)
    for _ in range(times):
        for c in colours:
            u = np.where((i + j + k) % 2 == c, (_off(w, u) - f) / sum(w), u)
    return u


def _full_xy(a):
    """Full weighting over x and y, at the even nodes."""
    for axis in (1, 2):
        a = 0.25 * np.roll(a, 1, axis) + 0.5 * a + 0.25 * np.roll(a, -1, axis)
    return a[:, ::2, ::2]


def _full_z(a):
    return 0.25 * a[0:-2:2] + 0.5 * a[1:-1:2] + 0.25 * a[2::2]


def _interpolate(c, zc):
    if zc:
        p = np.zeros((2 * c.shape[0] + 1,) + c.shape[1:])
        p[1::2] = c
        z = np.zeros_like(c[:1])
        p[::2] = 0.5 * (np.concatenate([z, c]) + np.concatenate([c, z]))
        c = p
    for axis in (1, 2):
        p = np.repeat(c, 2, axis)
        odd = tuple(slice(1, None, 2) if q == axis else slice(None) for q in range(3))
        p[odd] = 0.5 * (c + np.roll(c, -1, axis))
        c = p
    return c


def _vcycle(u, f, eps, h, dims, o):
    w = _weights(eps, h)
    if len(dims) == 1:
        return _sweeps(u, f, w, (0, 1), o["coarse_sweeps"])
    u = _sweeps(u, f, w, (0, 1), o["pre"])
    zc = dims[1][2] != dims[0][2]
    r = _full_xy(f - (_off(w, u) - sum(w) * u))
    e = _full_xy(eps)
    if zc:
        r = _full_z(r)
        e = np.concatenate([e[:1], _full_z(e[1:-1]), e[-1:]])
    c = _vcycle(np.zeros_like(r), r, e, (2 * h[0], 2 * h[1], (2 if zc else 1) * h[2]), dims[1:], o)
    return _sweeps(u + _interpolate(c, zc), f, w, (1, 0), o["post"])


# outside: what the bottom set leaves in global memory in float64 (0 nothing, 1 the
# first level's residual, 2 its f too, 3 everything); above: levels over the set.
# Where levels lie over it, their sweeps interpolate the coarse correction (from
# 2^14 points on), with z halved and not, on bands of 4, 6, 8 and 12 rows
@pytest.mark.parametrize("n,planes,outside,above,opts", [
    ((16, 16, 16), 5, 0, 0, dict(max_levels=2)),
    ((16, 16, 32), 18, 1, 0, dict(max_levels=2)),
    ((16, 16, 32), 22, 2, 0, dict(max_levels=2)),
    ((16, 24, 32), 20, 3, 0, dict(max_levels=2)),
    ((96, 24, 32), 3, 3, 0, dict(max_levels=4)),
    ((16, 48, 64), 48, 1, 1, dict(max_levels=3, pre=1, post=3)),
    ((96, 64, 64), 7, 2, 1, dict(max_levels=4, cycles=2)),
    ((96, 96, 64), 7, 3, 1, dict(max_levels=4)),
    ((64, 96, 64), 48, 1, 2, dict(max_levels=4, post=1)),
    ((64, 96, 64), 56, 2, 2, dict(max_levels=4, pre=0)),
    ((64, 64, 48), 31, 0, 2, dict()),
    ((128, 128, 48), 31, 3, 2, dict(cycles=2)),
    ((96, 96, 96), 63, 0, 3, dict(semi=2.0)),
    ((72, 96, 64), 47, 0, 2, dict()),
    ((144, 48, 64), 31, 2, 2, dict(semi=1.6)),
    ((192, 48, 64), 47, 2, 2, dict()),
    ((216, 48, 48), 31, 0, 2, dict(pre=1, post=1))])
@pytest.mark.parametrize("precision", [0, 1])
def test_split_matches_written_out_vcycles(torch, n, planes, outside, above, opts, precision):
    opts = dict(dict(pre=2, post=2, coarse_sweeps=7, cycles=1), **opts)
    L = (0.25 * n[0], 0.25 * n[1], 0.25 * opts.pop("semi", 1.0) * n[2])
    opts = _opts(n, L, planes, **opts)
    pl = B.plan(n, L, **opts)
    k0, dims = pl["k_w0"], pl["levels"]
    bottom = next(l for l, d in enumerate(dims) if d[0] * d[1] * d[2] <= 8192)
    fits = [_lds_bytes(dims[bottom:], 8, q) <= 160 * 1024 for q in range(3)] + [True]
    assert (fits.index(True), bottom) == (outside, above), (fits.index(True), dims, bottom)
    eps, r = W.random_fields(n, 47)
    s = B.Solver(0)
    s.set_grid(n, L, precision=precision, **opts)
    s.set_epsilon(torch.from_numpy(eps).cuda())
    z = s.apply_split(torch.from_numpy(r).cuda()).cpu().numpy()
    ref = O.vacuum_solve(r, s.h)
    wet = [(k0 + q) % n[2] for q in range(dims[0][2])]
    ext = [(k0 - 1 + q) % n[2] for q in range(dims[0][2] + 2)]
    f = (r - O.apply_A(ref, eps, s.h))[wet]
    u = np.zeros_like(f)
    for _ in range(opts["cycles"]):
        u = _vcycle(u, f, eps[ext], s.h, dims, opts)
    ref[wet] += u
    # the bars of the coarsest sweeps against written-out ones
    assert np.abs(z - ref).max() <= (1e-12 if precision == 0 else 1e-4) * np.abs(ref).max()
    s.close()
