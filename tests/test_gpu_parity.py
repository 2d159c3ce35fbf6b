"""Parity of the HIP path (through the C ABI) with the FP64 oracle.

Sizes are chosen so the oracle finishes in seconds while the grids span
several tiles of every kernel and have ragged edges (x extents that are not
multiples of the 64-wide stencil tiles, radix-3 FFT lengths, a wet slab that
wraps through z = 0).
"""
import math

import numpy as np
import pytest

import oracle as O
from paper_0904_4887_amd import workloads as W

pytestmark = pytest.mark.gpu

FOUR_PI = 4.0 * math.pi


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def _solver(torch, n, L, **opts):
    from paper_0904_4887_amd.binding import Solver
    s = Solver(0)
    s.set_grid(n, L, **opts)
    return s


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _host(t):
    return t.detach().cpu().numpy()


def _rel(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


# ---------------------------------------------------------------- building blocks

@pytest.mark.parametrize("n", [(24, 36, 48), (32, 32, 64), (96, 16, 18)])
def test_apply_operator_matches_oracle(torch, n):
    L = (0.3 * n[0], 0.25 * n[1], 0.4 * n[2])
    eps, _ = W.random_fields(n, 7)
    rng = np.random.default_rng(8)
    phi = rng.normal(size=eps.shape)
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2])
    s.set_epsilon(_dev(torch, eps))
    out = _host(s.apply_operator(_dev(torch, phi)))
    ref = O.apply_A(phi, eps, s.h)
    assert _rel(out, ref) <= 1e-13


@pytest.mark.parametrize("n", [(24, 36, 48), (32, 32, 64), (96, 96, 192), (16, 8, 512), (12, 18, 384)])
def test_vacuum_solve_matches_oracle(torch, n):
    L = (0.2 * n[0], 0.3 * n[1], 0.1 * n[2])
    rng = np.random.default_rng(9)
    r = rng.normal(size=(n[2], n[1], n[0]))
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2])
    out = _host(s.vacuum_solve(_dev(torch, r)))
    ref = O.vacuum_solve(r, s.h)
    assert _rel(out, ref) <= 1e-12


def test_build_rho_matches_oracle(torch):
    w = W.slab(n=(48, 48, 96))
    s = _solver(torch, w.n, w.L)
    rho = _host(s.build_rho(w.xyz, w.q, w.sigma))
    ref = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    assert np.abs(rho - ref).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("exclusion", [False, True])
def test_build_epsilon_matches_oracle(torch, exclusion):
    w = W.slab(n=(48, 48, 96), exclusion=exclusion)
    s = _solver(torch, w.n, w.L)
    s.build_epsilon(w.xyz, w.radius, w.eps_params)
    eps = _host(s.get_epsilon())
    ref = O.eps_erf(w.n, w.L, w.xyz, w.radius, w.eps_params)
    assert np.abs(eps - ref).max() <= 1e-12 * 78.36


# four nodes a thread on 5166 tiles with remainders along x, y and z, one on 20;
# atoms past one batch of 256, around the whole cell and partly buried
@pytest.mark.parametrize("n", [(162, 162, 162), (36, 32, 18)])
def test_builders_on_ragged_tiles_and_many_atoms(torch, n):
    L = (12.0, 12.0, 12.0)
    rng = np.random.default_rng(41)
    m = 300
    xyz, q = rng.uniform(0.0, 12.0, (m, 3)), rng.normal(size=m)
    radius, sigma = rng.uniform(0.3, 0.5, m), rng.uniform(0.3, 0.6, m)
    p = dict(eps_inf=78.36, delta=0.1, exclusion=1, z_lim=0.1, delta_z=0.3)
    N = n[0] * n[1] * n[2]
    nodes = np.unique(np.r_[0:400, N - 400:N, rng.choice(N, 3000)])
    s = _solver(torch, n, L)
    s.build_epsilon(xyz, radius, p)
    at = torch.from_numpy(nodes).cuda()
    eps = _host(s.get_epsilon().reshape(-1)[at])
    rho = _host(s.build_rho(xyz, q, sigma).reshape(-1)[at])
    eps_ref = O.eps_erf(n, L, xyz, radius, p, nodes=nodes)
    rho_ref = O.rho_gauss(n, L, xyz, q, sigma, nodes=nodes)
    assert 10.0 < eps_ref.max() and eps_ref.min() < 1.01
    # the bars of the slab's builders
    assert np.abs(eps - eps_ref).max() <= 1e-12 * 78.36
    assert np.abs(rho - rho_ref).max() <= 1e-12 * np.abs(rho_ref).max()


# ---------------------------------------------------------------- full solve

def _check_solution(torch, s, rho, eps, phi, E, info, tol_E, tol_phi):
    ref_phi = O.solve(rho, eps, s.h, tol=1e-13)
    ref_E = O.energy(rho, ref_phi, s.h)
    assert info["rel_res"] <= s.opts.tol
    assert abs(E - ref_E) <= tol_E * abs(ref_E), (E, ref_E)
    assert _rel(phi, ref_phi) <= tol_phi
    assert abs(info["energy_eps_form"] - E) <= 1e-9 * abs(E)
    return ref_phi


def test_solve_tanh_box_fp64(torch):
    w = W.tanh_box()
    eps = w.eps_grid()
    rho = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    s = _solver(torch, w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], tol=1e-10)
    s.set_epsilon(_dev(torch, eps))
    phi, E, info = s.solve(_dev(torch, rho))
    _check_solution(torch, s, rho, eps, _host(phi), E, info, 1e-10, 1e-8)


@pytest.mark.parametrize("exclusion,precision", [(False, 0), (True, 0), (True, 1), (False, 1)])
def test_solve_small_slab(torch, exclusion, precision):
    w = W.slab(n=(48, 48, 96), exclusion=exclusion)
    s = _solver(torch, w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], tol=1e-10, precision=precision)
    s.build_epsilon(w.xyz, w.radius, w.eps_params)
    rho_d = s.build_rho(w.xyz, w.q, w.sigma)
    phi, E, info = s.solve(rho_d)
    eps = O.eps_erf(w.n, w.L, w.xyz, w.radius, w.eps_params)
    rho = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    _check_solution(torch, s, rho, eps, _host(phi), E, info, 1e-10, 1e-8)


@pytest.mark.parametrize("exclusion", [False, True])
def test_solve_small_slab_float32_dry_update(torch, exclusion):
    """Mixed precision with the float32 FFT dry update: the preconditioner
    changes, the float64 coupling still reaches the same solution."""
    w = W.slab(n=(48, 48, 96), exclusion=exclusion)
    s = _solver(torch, w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], tol=1e-10, precision=1, fft_fp32=1)
    s.build_epsilon(w.xyz, w.radius, w.eps_params)
    rho_d = s.build_rho(w.xyz, w.q, w.sigma)
    phi, E, info = s.solve(rho_d)
    eps = O.eps_erf(w.n, w.L, w.xyz, w.radius, w.eps_params)
    rho = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    _check_solution(torch, s, rho, eps, _host(phi), E, info, 1e-10, 1e-8)


# restart cycles whose new vectors the dry update rescales as it reads them: planes in
# one block and separate x passes (fewer than 64 planes of 96 x 96), with fewer blocks
# of reductions than usual and with all of them
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [(16, 32, 24), (96, 96, 32)])
def test_solve_with_rescaled_vectors(torch, n, precision):
    L = (0.25 * n[0], 0.25 * n[1], 0.4 * n[2])
    eps, rho = W.random_fields(n, 43)
    rho -= rho.mean()
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], tol=1e-10, precision=precision, fft_fp32=precision,
                krylov_fp32=precision, restart=8)
    s.set_epsilon(_dev(torch, eps))
    phi, E, info = s.solve(_dev(torch, rho))
    assert info["restarts"] >= 2
    # the bars of the other solves at this tolerance
    _check_solution(torch, s, rho, eps, _host(phi), E, info, 1e-9, 1e-7)


@pytest.mark.parametrize("exclusion", [False, True])
def test_forces_and_eps_gradient_match_oracle(torch, exclusion):
    w = W.slab(n=(48, 48, 96), exclusion=exclusion)
    s = _solver(torch, w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], tol=1e-12)
    s.build_epsilon(w.xyz, w.radius, w.eps_params)
    rho_d = s.build_rho(w.xyz, w.q, w.sigma)
    phi_d, E, info = s.solve(rho_d)
    g = _host(s.eps_gradient())
    F = s.forces(w.xyz, w.q, w.sigma, w.radius, w.eps_params)
    phi = _host(phi_d)
    # oracle gradient and forces evaluated on the GPU solution (isolates the kernels)
    g_ref = O.eps_gradient(phi, s.h)
    assert _rel(g, g_ref) <= 1e-12
    eps = O.eps_erf(w.n, w.L, w.xyz, w.radius, w.eps_params)
    F_ref = O.forces(w.n, w.L, w.xyz, w.radius, w.q, w.sigma, w.eps_params, phi, g_ref)
    assert np.abs(F - F_ref).max() <= 1e-10 * np.abs(F_ref).max()
    # and against the oracle's own solution
    rho = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    phi_o = O.solve(rho, eps, s.h, tol=1e-13)
    F_o = O.forces(w.n, w.L, w.xyz, w.radius, w.q, w.sigma, w.eps_params, phi_o, O.eps_gradient(phi_o, s.h))
    assert np.abs(F - F_o).max() <= 1e-8 * np.abs(F_o).max()
    # the switch term needs the atoms eps was built from
    from paper_0904_4887_amd.binding import DWPError, DWP_ESTATE
    moved = w.xyz.copy()
    moved[3, 0] += 0.01
    with pytest.raises(DWPError) as e:
        s.forces(moved, w.q, w.sigma, w.radius, w.eps_params)
    assert e.value.status == DWP_ESTATE


# ---------------------------------------------------------------- error paths

def test_error_paths(torch):
    from paper_0904_4887_amd.binding import DWPError, DWP_ESTATE, DWP_EINVAL, DWP_ENONFINITE, DWP_ENOCONV
    w = W.tanh_box(n=(16, 16, 32))
    s = _solver(torch, w.n, w.L, z_wet_lo=8.0, z_wet_hi=20.0)
    rho = O.rho_gauss(w.n, w.L, w.xyz, w.q, w.sigma)
    with pytest.raises(DWPError) as e:
        s.solve(_dev(torch, rho))
    assert e.value.status == DWP_ESTATE
    bad = w.eps_grid()
    bad[3, 2, 1] = 0.5
    with pytest.raises(DWPError) as e:
        s.set_epsilon(_dev(torch, bad))
    assert e.value.status == DWP_EINVAL
    s.set_epsilon(_dev(torch, w.eps_grid()))
    nan_rho = rho.copy()
    nan_rho[1, 1, 1] = np.nan
    with pytest.raises(DWPError) as e:
        s.solve(_dev(torch, nan_rho))
    assert e.value.status == DWP_ENONFINITE
    s.set_opts(max_outer=1)
    with pytest.raises(DWPError) as e:
        s.solve(_dev(torch, rho))
    assert e.value.status == DWP_ENOCONV
    s.set_opts(max_outer=600)
    phi, E, info = s.solve(_dev(torch, rho))
    assert info["rel_res"] <= 1e-10


@pytest.mark.parametrize("smoother", [1, 2])
@pytest.mark.parametrize("precision,cycles,pre,post", [(0, 1, 2, 2), (1, 1, 2, 2), (1, 2, 2, 2), (0, 1, 0, 1),
                                                    (1, 2, 0, 2)])
def test_fused_sweep_equals_colour_passes(torch, precision, cycles, pre, post, smoother):
    """The fused out-of-place sweep and the two in-place colour passes are the
    same Gauss-Seidel sweep: one application of the split agrees to rounding.
    The fine wet level of this grid (96 x 96 x 151) is above the size from
    which the fused kernel takes over, so both kernels really run: the fused
    one on bands of 12 whole rows (smoother 1) or on 32 x 16 tiles (smoother
    2).  Without pre-sweeps the first fused sweep follows the coarse-grid
    correction and must read it (its zero-input variant would drop it)."""
    from paper_0904_4887_amd.binding import plan
    w = W.slab(n=(96, 96, 192), exclusion=True)
    fine = plan(w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1])["levels"][0]
    assert fine[0] * fine[1] * fine[2] >= 1 << 20
    s = _solver(torch, w.n, w.L, z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], precision=precision, smoother=smoother,
                cycles=cycles, pre=pre, post=post)
    s.build_epsilon(w.xyz, w.radius, w.eps_params)
    rng = np.random.default_rng(3)
    r = _dev(torch, rng.normal(size=s.shape))
    z1 = _host(s.apply_split(r))
    s.set_opts(smoother=0)
    z0 = _host(s.apply_split(r))
    assert _rel(z1, z0) <= (1e-12 if precision == 0 else 2e-5)


@pytest.mark.parametrize("smoother", [1, 2])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n", [(216, 216, 48), (162, 108, 96)])
def test_fused_sweep_equals_colour_passes_ragged_tiles(torch, n, precision, smoother):
    """The fused sweep against the two colour passes on grids whose x and y
    extents are not multiples of its 32 x 16 tile (tiles overhang the
    periodic wrap in x and y).  On 162 x 108 nx is 2 mod 4, so the float32
    variant loads 8-byte vectors; x cannot be halved there, so that grid has
    a single multigrid level, smoothed by the grid-wide kernels.  With
    smoother 1 the row-band kernel takes these levels with bands of 12 rows
    (216, float32), 4 rows (216, float64) and 6 rows (108), with 4- and
    2-wide vectors."""
    from paper_0904_4887_amd.binding import plan
    L = (0.07 * n[0], 0.07 * n[1], 0.1 * n[2])
    opts = dict(z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=precision, smoother=smoother, coarse_sweeps=3)
    lv = plan(n, L, **opts)["levels"]
    assert lv[0][0] * lv[0][1] * lv[0][2] >= 1 << 20
    s = _solver(torch, n, L, **opts)
    eps, _ = W.random_fields(n, 17)
    s.set_epsilon(_dev(torch, eps))
    rng = np.random.default_rng(4)
    r = _dev(torch, rng.normal(size=s.shape))
    z1 = _host(s.apply_split(r))
    s.set_opts(smoother=0)
    z0 = _host(s.apply_split(r))
    assert np.isfinite(z1).all()
    assert _rel(z1, z0) <= (1e-12 if precision == 0 else 2e-5)


def test_bottom_vcycle_out_of_lds_matches_the_global_memory_one(torch):
    """The levels at the bottom of the hierarchy (12 x 12 x 37 and 6 x 6 x 18
    here) run in one workgroup; in float32 they fit its LDS (96 KB) and run out
    of it, in float64 (192 KB) they run from global memory.  One application
    of the split agrees between the two precisions to float32 rounding, while
    dropping the bottom levels changes it a hundred times more, so an error in
    either bottom kernel would show."""
    from paper_0904_4887_amd.binding import plan
    w = W.slab(n=(96, 96, 192), exclusion=True)
    opts = dict(z_wet_lo=w.z_wet[0], z_wet_hi=w.z_wet[1], pre=2, post=2, coarse_sweeps=8)
    lv = plan(w.n, w.L, **opts)["levels"]
    assert [tuple(x) for x in lv[-2:]] == [(12, 12, 37), (6, 6, 18)]
    rng = np.random.default_rng(5)
    r = rng.normal(size=(w.n[2], w.n[1], w.n[0]))
    z = {}
    for key, kw in (("lds", dict(precision=1)), ("global", dict(precision=0)),
                    ("no_bottom", dict(precision=0, max_levels=len(lv) - 2))):
        s = _solver(torch, w.n, w.L, **opts, **kw)
        s.build_epsilon(w.xyz, w.radius, w.eps_params)
        z[key] = _host(s.apply_split(_dev(torch, r)))
        s.close()
    d_lds, d_drop = _rel(z["lds"], z["global"]), _rel(z["no_bottom"], z["global"])
    assert d_lds <= 1e-4 and d_drop >= 100 * d_lds, (d_lds, d_drop)


def _rb_sweeps(f, eps, h, sweeps):
    """Red-black Gauss-Seidel sweeps from zero on a slab (zero data on the planes
    below and above it): f (nw, ny, nx), eps (nw + 2, ny, nx) with those planes."""
    u = np.zeros_like(eps)
    k, j, i = np.indices(f.shape)
    c = [1.0 / (x * x) for x in h]
    e0 = eps[1:-1]

    def nb(a):
        m = a[1:-1]
        return (np.roll(m, -1, 2), np.roll(m, 1, 2), np.roll(m, -1, 1), np.roll(m, 1, 1), a[2:], a[:-2])

    w = [0.5 * c[q // 2] * (e0 + e) for q, e in enumerate(nb(eps))]
    for _ in range(sweeps):
        for col in (0, 1):
            v = (sum(a * b for a, b in zip(w, nb(u))) - f) / sum(w)
            u[1:-1] = np.where((i + j + k) % 2 == col, v, u[1:-1])
    return u[1:-1]


# the sizes take the single-level bottom kernel through one, two and three points
# of a colour per thread and past its registers, with everything in LDS, with f
# outside and (the wide thin slabs) out of global memory; 9 sweeps of a level
# beyond those registers take the cooperative kernel, with tiles of one to three
# points of a colour per thread, rows whole and split, uneven tiles, one plane a tile
@pytest.mark.parametrize("n,planes,sweeps", [
    ((8, 8, 16), 3, 7), ((12, 18, 16), 9, 7), ((18, 16, 32), 13, 7), ((24, 16, 32), 15, 7), ((32, 16, 32), 16, 7),
    ((64, 64, 16), 3, 7), ((18, 16, 32), 25, 9), ((18, 18, 128), 111, 9), ((54, 48, 64), 41, 64), ((64, 96, 16), 3, 9),
    ((54, 108, 162), 127, 9), ((8, 8, 512), 400, 8), ((162, 16, 32), 20, 9)])
@pytest.mark.parametrize("precision", [0, 1])
def test_coarsest_sweeps_match_written_out_sweeps(torch, n, planes, sweeps, precision):
    from paper_0904_4887_amd import binding as B
    L = (0.3 * n[0], 0.25 * n[1], 0.4 * n[2])
    lo = L[2] * (n[2] - planes) / n[2]
    opts = dict(precision=precision, z_wet_lo=lo, z_wet_hi=L[2], max_levels=1, coarse_sweeps=sweeps, cycles=2)
    pl = B.plan(n, L, **opts)
    k0, nw = pl["k_w0"], pl["levels"][0][2]
    assert len(pl["levels"]) == 1
    eps, r = W.random_fields(n, 31)
    s = _solver(torch, n, L, **opts)
    s.set_epsilon(_dev(torch, eps))
    z = _host(s.apply_split(_dev(torch, r)))
    dry = O.vacuum_solve(r, s.h)
    rw = r - O.apply_A(dry, eps, s.h)
    wet = [(k0 + q) % n[2] for q in range(nw)]
    ext = [(k0 - 1 + q) % n[2] for q in range(nw + 2)]
    ref = dry.copy()
    # two cycles of one level: the second goes on from the first one's values
    ref[wet] += _rb_sweeps(rw[wet], eps[ext], s.h, 2 * sweeps)
    assert _rel(_host(s.apply_split(_dev(torch, r))), z) == 0.0
    # float32: the level's values and updates round at 6e-8; the bar of the
    # other bottom test
    assert _rel(z, ref) <= (1e-12 if precision == 0 else 1e-4)


def test_cooperative_sweeps_from_two_threads(torch):
    """Two contexts on streams of their own, driven by two threads, each with a
    coarsest level that takes the cooperative kernel on every CU: the results
    are those of the same calls one after the other."""
    import threading
    n, L = (108, 96, 96), (11.8, 11.8, 40.0)
    eps, r = W.random_fields(n, 37)
    de, dr = _dev(torch, eps), _dev(torch, r)
    torch.cuda.synchronize()
    out, alone = [[], []], None

    def work(q):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2])
            s.set_epsilon(de)
            z = [s.apply_split(dr) for _ in range(6)]
            st.synchronize()
            out[q] = [_host(t) for t in z]

    work(0)
    alone = out[0][0]
    threads = [threading.Thread(target=work, args=(q,)) for q in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for z in out[0] + out[1]:
        assert np.array_equal(z, alone)
    assert len(out[1]) == 6


@pytest.mark.parametrize("n", [(24, 36, 48), (96, 96, 192), (192, 192, 384), (256, 256, 32), (18, 54, 48),
                               (16, 8, 512)])
def test_float32_vacuum_solve_matches_oracle(torch, n):
    """The dry update with its spectrum in float32 (fft_fp32), as the
    building block runs it: agrees with the float64 oracle to float32
    rounding on grids with radix-2, 3, 4 and 8 stages and long z."""
    L = (0.2 * n[0], 0.3 * n[1], 0.1 * n[2])
    rng = np.random.default_rng(19)
    r = rng.normal(size=(n[2], n[1], n[0]))
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=1, fft_fp32=1)
    out = _host(s.vacuum_solve(_dev(torch, r)))
    ref = O.vacuum_solve(r, s.h)
    assert _rel(out, ref) <= 2e-5


# rows of 4 m and 4 m + 2 values, an odd and an even number of spectrum pairs, and a
# last block of lines that is not full
@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("n", [(18, 16, 24), (24, 18, 16), (54, 36, 18), (162, 8, 12), (96, 54, 24), (8, 8, 54)])
def test_scaled_dry_update_matches_oracle(torch, n, fp32):
    """s L^-1 (s r), s = eps^-1/2: the split without a wet correction."""
    L = (0.2 * n[0], 0.3 * n[1], 0.1 * n[2])
    eps, r = W.random_fields(n, 23)
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=fp32, fft_fp32=fp32, cycles=0, scaled_dry=1)
    s.set_epsilon(_dev(torch, eps))
    out = _host(s.apply_split(_dev(torch, r)))
    si = 1.0 / np.sqrt(eps)
    ref = si * O.vacuum_solve(si * r, s.h)
    # the bars of the unscaled solves
    assert _rel(out, ref) <= (2e-5 if fp32 else 1e-12)


# planes transformed in one block of 512 threads (3024 of at most 3072 values), of 1024
# (4704 and 5940 of 6144; fewer than 64 planes: separate passes), with up to ten values
# a thread (9360 and 10240 of 10240, the latter in float32 only: the LDS; fewer than 96
# planes or a last round of 32: separate passes), and past all of them
@pytest.mark.parametrize("fp32,scaled", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("n", [(54, 108, 8), (96, 96, 54), (96, 96, 64), (108, 108, 72), (128, 144, 96),
                               (128, 144, 72), (96, 128, 288), (8, 2048, 96), (162, 144, 96)])
def test_dry_update_by_planes_matches_oracle(torch, n, fp32, scaled):
    L = (0.2 * n[0], 0.2 * n[1], 0.2 * n[2])
    eps, r = W.random_fields(n, 29)
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=fp32, fft_fp32=fp32, cycles=0,
                scaled_dry=scaled)
    s.set_epsilon(_dev(torch, eps))
    out = _host(s.apply_split(_dev(torch, r)))
    si = 1.0 / np.sqrt(eps) if scaled else 1.0
    ref = si * O.vacuum_solve(si * r, s.h)
    # the bars of the other solves; a line of 2048 gains rounding as in the test of 4096
    long = max(n) / 512 if max(n) > 512 else 1.0
    assert _rel(out, ref) <= (2e-5 if fp32 else 1e-12) * long**2


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("n", [(4096, 8, 8), (8, 4096, 8), (8, 8, 4096)])
def test_vacuum_solve_at_the_longest_axis(torch, n, fp32):
    """The largest extent the planner accepts (4096) along each axis in turn: a
    line of 4096 values is one FFT block by itself (the x pass then stages 4097
    complex values in LDS).  The smallest eigenvalue of the 4096-long axis,
    (2 pi / 4096)^2 / h^2, amplifies rounding about 64 times more than on the
    512-long axes of the other tests, and the bars scale with it."""
    L = (0.05 * n[0], 0.05 * n[1], 0.05 * n[2])
    rng = np.random.default_rng(23)
    r = rng.normal(size=(n[2], n[1], n[0]))
    s = _solver(torch, n, L, z_wet_lo=0.3 * L[2], z_wet_hi=L[2], precision=fp32, fft_fp32=fp32)
    out = _host(s.vacuum_solve(_dev(torch, r)))
    ref = O.vacuum_solve(r, s.h)
    assert _rel(out, ref) <= (5e-4 if fp32 else 1e-10)
