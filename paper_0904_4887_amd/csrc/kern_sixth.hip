// The paper's sixth-order operator (Sec. II.F, Eqs. 16-18) on the full
// periodic box, its transpose, and the gradient kernels its adjoint needs.
//
//   A6 x   = sum_d G_d D1_d x + eps D2_d x,        G_d = D1_d eps,
//   A6^T y = sum_d -D1_d(G_d y) + D2_d(eps y),
// with the seven-point central stencils
//   D1 f_i = (1/h) sum_{n=1..3} a_n (f_{i+n} - f_{i-n}),   a = (3/4, -3/20, 1/60),
//   D2 f_i = (1/h^2) [b_0 f_i + sum_{n=1..3} b_n (f_{i+n} + f_{i-n})],
//   b = (-49/18, 3/2, -3/20, 1/90).
// G is computed once per permittivity.  The operators are LDS-tiled (below);
// the gradient kernel reads its wider stencil through the caches.  Every axis
// is periodic and at least 8 long, so a shift of up to 3 wraps at most once.
#include "dwp_internal.h"

#include <algorithm>

namespace dwp {

namespace {

constexpr int SX = 64, SY = 4;
constexpr double A1 = 0.75, A2 = -0.15, A3 = 1.0 / 60.0;
constexpr double B0 = -49.0 / 18.0, B1 = 1.5, B2 = -0.15, B3 = 1.0 / 90.0;
constexpr double FOUR_PI = 4.0 * 3.14159265358979323846;

__device__ __forceinline__ int wrap(int i, int n) { return i < 0 ? i + n : (i >= n ? i - n : i); }

struct Grid6 {
    int nx, ny, nz;
    size_t plane, N;
    double ihx, ihy, ihz;        // 1/h
    double ihx2, ihy2, ihz2;     // 1/h^2
};

Grid6 make_grid6(const Plan &p) {
    Grid6 g;
    g.nx = p.nx; g.ny = p.ny; g.nz = p.nz;
    g.plane = (size_t)p.nx * p.ny;
    g.N = p.N;
    g.ihx = 1.0 / p.h[0]; g.ihy = 1.0 / p.h[1]; g.ihz = 1.0 / p.h[2];
    g.ihx2 = g.ihx * g.ihx; g.ihy2 = g.ihy * g.ihy; g.ihz2 = g.ihz * g.ihz;
    return g;
}

// Offsets of the six neighbours at distance 1..3 along each axis, as flat
// index differences (periodic).
struct Star {
    long long xp[3], xm[3], yp[3], ym[3], zp[3], zm[3];
};

__device__ __forceinline__ Star star(const Grid6 &g, int i, int j, int k) {
    Star s;
#pragma unroll
    for (int n = 1; n <= 3; ++n) {
        s.xp[n - 1] = wrap(i + n, g.nx) - i;
        s.xm[n - 1] = wrap(i - n, g.nx) - i;
        s.yp[n - 1] = (long long)(wrap(j + n, g.ny) - j) * g.nx;
        s.ym[n - 1] = (long long)(wrap(j - n, g.ny) - j) * g.nx;
        s.zp[n - 1] = (long long)(wrap(k + n, g.nz) - k) * (long long)g.plane;
        s.zm[n - 1] = (long long)(wrap(k - n, g.nz) - k) * (long long)g.plane;
    }
    return s;
}

__device__ __forceinline__ double d1(const double *f, size_t c, const long long *p, const long long *m, double ih) {
    return ih * (A1 * (f[c + p[0]] - f[c + m[0]]) + A2 * (f[c + p[1]] - f[c + m[1]]) + A3 * (f[c + p[2]] - f[c + m[2]]));
}

__device__ __forceinline__ double d2(const double *f, size_t c, const long long *p, const long long *m, double ih2) {
    return ih2 * (B0 * f[c] + B1 * (f[c + p[0]] + f[c + m[0]]) + B2 * (f[c + p[1]] + f[c + m[1]]) +
                  B3 * (f[c + p[2]] + f[c + m[2]]));
}

// G_d = D1_d eps for the three directions
__global__ void __launch_bounds__(SX *SY) k_d1eps(Grid6 g, const double *__restrict__ eps, double *__restrict__ G) {
    const int i = blockIdx.x * SX + threadIdx.x, j = blockIdx.y * SY + threadIdx.y, k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const size_t c = (size_t)k * g.plane + (size_t)j * g.nx + i;
    const Star s = star(g, i, j, k);
    G[c] = d1(eps, c, s.xp, s.xm, g.ihx);
    G[g.N + c] = d1(eps, c, s.yp, s.ym, g.ihy);
    G[2 * g.N + c] = d1(eps, c, s.zp, s.zm, g.ihz);
}

// LDS-tiled form of the operator, its transpose and their residual forms.  A
// block owns a tile of ty rows of wp pairs of points (one 2-wide vector per
// thread; wp divides nx / 2 and ty divides ny, so no tile overhangs) for a
// chunk of kc planes.  It keeps the z neighbours (k - 3 .. k + 3) of its own
// points in registers and stages each plane with a halo of 4 columns and 3 rows
// in LDS (two slots): its own points from the registers, so that only the halo
// is loaded again.  Loads are issued one plane step ahead of their use; one
// barrier per step.
//   forward:    LDS and registers hold x and, in float64, eps; G = D1 eps is
//               formed from it, with the operations of k_d1eps, so that 24 bytes
//               per point move instead of 48 with G read back.  (On float32
//               vectors G is read: formed from eps in float32 it would lose
//               digits to cancellation.)
//   transposed: LDS holds eps y, Gx y, Gy y (the products the transpose
//               differentiates); registers hold eps y and Gz y.  G is read: it
//               is needed at the neighbours, where it would take eps 6 cells out.
// MODE 0: out = op x;  1: out = b - op x;  2: out (wet slab plane q, type T) =
// b - op x at box plane (k_w0 + q) mod nz.  AL: the box arrays are 16-byte
// aligned (a caller's may be aligned to 8 only: pairs are then loaded in halves).
// Bound by HBM, LDS reads and float64 arithmetic alike at large grids (a plane
// step spends about a microsecond of each per CU), by the latency of the steps
// at small ones.  A6 at 192 x 192 x 384 in float64: 176 us with 64 x 4 tiles, two
// barriers and unhidden loads a plane and G read; 91 us so.  On float32 vectors
// at 96 x 96 x 192 (kernel trace): 30.4 -> 14.0 us, transposed 36.2 -> 23.2 us.
constexpr int H6X = 4, H6Y = 3;             // halo columns (pair-aligned) and rows
constexpr int OP6_NT_FWD = 768, OP6_NT_TRANS = 512;  // most threads (168 and 256 registers)

struct Op6Shape {
    int k_w0, nplanes, wp, ty, tiles_x, tiles_y, kc, nb;
};

typedef double d2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));

template <bool AL> __device__ __forceinline__ d2v ldp(const double *p) {
    if constexpr (AL) return *(const d2v *)p;
    else return d2v{p[0], p[1]};
}
template <bool AL> __device__ __forceinline__ d2v ldp(const float *p) {
    const f2v v = *(const f2v *)p;  // the library's own arrays only
    return d2v{(double)v[0], (double)v[1]};
}
template <bool AL> __device__ __forceinline__ void stp(double *p, d2v v) {
    if constexpr (AL) *(d2v *)p = v;
    else { p[0] = v[0]; p[1] = v[1]; }
}
template <bool AL> __device__ __forceinline__ void stp(float *p, d2v v) {
    *(f2v *)p = f2v{(float)v[0], (float)v[1]};
}

// Where a block and a thread stand: tile origin, planes, the thread's own pair
// and its halo pair (in-plane element offset and LDS index, ylo: a row halo).
struct Op6Pos {
    int q0, q1, kb, own_l, halo_l, ls;
    bool own, halo, ylo;
    unsigned own_o, halo_o;
};
__device__ __forceinline__ bool op6_pos(const Grid6 &g, const Op6Shape &p, Op6Pos &t) {
    // each XCD (hardware block b runs on XCD b mod 8) gets a run of neighbouring tiles
    const int tile = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (tile >= p.nb) return false;
    const int x0 = (tile % p.tiles_x) * 2 * p.wp, y0 = ((tile / p.tiles_x) % p.tiles_y) * p.ty;
    t.q0 = (tile / (p.tiles_x * p.tiles_y)) * p.kc;
    t.q1 = min(p.nplanes, t.q0 + p.kc);
    t.ls = 2 * p.wp + 2 * H6X;  // LDS row length
    const int tid = threadIdx.x;
    const int r = tid / p.wp, c = tid - r * p.wp;
    t.own = r < p.ty;
    const int rr = t.own ? r : 0;
    t.own_o = (unsigned)((y0 + rr) * g.nx + x0 + 2 * c);
    t.own_l = (rr + H6Y) * t.ls + H6X + 2 * c;
    const int nhx = 4 * p.ty, nh = nhx + 2 * H6Y * p.wp;
    t.halo = tid < nh;
    const int h = t.halo ? tid : 0;
    int x, y, lx, ly;
    if (h < nhx) {  // two pairs left and two right of each row
        const int side = h & 3;
        ly = h >> 2;
        lx = side < 2 ? 2 * side - 4 : 2 * p.wp + 2 * (side - 2);
        t.ylo = false;
    } else {        // three rows below and three above
        const int q = h - nhx, row = q / p.wp;
        ly = row < H6Y ? row - H6Y : p.ty + row - H6Y;
        lx = 2 * (q - row * p.wp);
        t.ylo = true;
    }
    x = wrap(x0 + lx, g.nx);
    y = wrap(y0 + ly, g.ny);
    t.halo_o = (unsigned)(y * g.nx + x);
    t.halo_l = (ly + H6Y) * t.ls + H6X + lx;
    return true;
}

// ih sum_n A_n (f_{+n} - f_{-n}) and B_0 f_0 + sum_n B_n (f_{+n} + f_{-n})
__device__ __forceinline__ double d1v(double ih, double m3, double m2, double m1, double p1, double p2, double p3) {
    return ih * (A1 * (p1 - m1) + A2 * (p2 - m2) + A3 * (p3 - m3));
}
__device__ __forceinline__ double d2s(double m3, double m2, double m1, double c, double p1, double p2, double p3) {
    return B0 * c + B1 * (p1 + m1) + B2 * (p2 + m2) + B3 * (p3 + m3);
}
// the seven values -3 .. 3 along x around each of a pair, f[e .. e + 6]
struct Row8 {
    double f[8];
};
__device__ __forceinline__ Row8 row8(const double *l, d2v c) {
    const d2v a = *(const d2v *)(l - 4), b = *(const d2v *)(l - 2), d = *(const d2v *)(l + 2), e = *(const d2v *)(l + 4);
    return Row8{{a[1], b[0], b[1], c[0], c[1], d[0], d[1], e[0]}};
}

// G: null to form G from eps (float64 eps, staged like x), else read at the point
// with eps (float32 vectors: eps and G rounded to float32).
template <int MODE, class T, class TX, class TE, bool AL>
__global__ void __launch_bounds__(OP6_NT_FWD)
k_op6_fwd(Grid6 g, Op6Shape p, const TX *__restrict__ x, const TE *__restrict__ eps, const TE *__restrict__ G,
          const double *__restrict__ b, T *__restrict__ out) {
    extern __shared__ __align__(16) double op6_lds[];
    constexpr bool FORM = sizeof(TE) == 8;  // G is formed here
    Op6Pos t;
    if (!op6_pos(g, p, t)) return;
    const int field = (p.ty + 2 * H6Y) * t.ls;
    const int kb = MODE == 2 ? p.k_w0 : 0;
    auto zp = [&](int k) { return (size_t)wrap(k >= g.nz ? k - g.nz : k, g.nz) * g.plane; };
    // x (and eps) at planes k - 3 .. k + 3 and of the halo pair; with G read, eps and G at plane k
    d2v xq[7], eq[FORM ? 7 : 1], hx{0, 0}, he{0, 0}, gq[FORM ? 1 : 3];
    const int kf = kb + t.q0;
#pragma unroll
    for (int d = 0; d < 7; ++d) {
        const size_t o = zp(kf - 3 + d) + t.own_o;
        xq[d] = ldp<AL>(x + o);
        if constexpr (FORM) eq[d] = ldp<true>(eps + o);
    }
    auto halo = [&](int k) {
        if (t.halo) {
            const size_t o = zp(k) + t.halo_o;
            hx = ldp<AL>(x + o);
            if constexpr (FORM) he = ldp<true>(eps + o);
        }
    };
    auto stash = [&](int slot, d2v xv, d2v ev) {
        double *lx = op6_lds + slot * (FORM ? 2 : 1) * field, *le = lx + field;
        if (t.own) *(d2v *)(lx + t.own_l) = xv;
        if (t.halo) *(d2v *)(lx + t.halo_l) = hx;
        if constexpr (FORM) {
            if (t.own) *(d2v *)(le + t.own_l) = ev;
            if (t.halo) *(d2v *)(le + t.halo_l) = he;
        }
    };
    auto coefs = [&](int k) {
        if constexpr (!FORM) {
            const size_t o = zp(k) + t.own_o;
            eq[0] = ldp<true>(eps + o);
#pragma unroll
            for (int d = 0; d < 3; ++d) gq[d] = ldp<true>(G + d * g.N + o);
        }
    };
    halo(kf);
    stash(0, xq[3], FORM ? eq[FORM ? 3 : 0] : d2v{0, 0});
    halo(kf + 1);
    coefs(kf);
    __syncthreads();
    const double ihx = g.ihx, ihy = g.ihy, ihz = g.ihz, ihx2 = g.ihx2, ihy2 = g.ihy2, ihz2 = g.ihz2;
    const int ls = t.ls;
    for (int q = t.q0; q < t.q1; ++q) {
        const int k = kb + q, slot = (q - t.q0) & 1;
        const size_t o = zp(k) + t.own_o;
        d2v xn = xq[6], en = eq[FORM ? 6 : 0], bv{0, 0};
        const d2v ec = eq[FORM ? 3 : 0], g0 = gq[0], g1 = gq[FORM ? 0 : 1], g2 = gq[FORM ? 0 : 2];
        if (MODE != 0) bv = ldp<AL>(b + o);
        if (q + 1 < t.q1) {
            stash(slot ^ 1, xq[4], eq[FORM ? 4 : 0]);
            const size_t on = zp(k + 4) + t.own_o;
            xn = ldp<AL>(x + on);
            if constexpr (FORM) en = ldp<true>(eps + on);
            halo(k + 2);
            coefs(k + 1);
        }
        if (t.own) {
            const double *lx = op6_lds + slot * (FORM ? 2 : 1) * field + t.own_l, *le = lx + field;
            const Row8 fx = row8(lx, xq[3]);
            Row8 fe;
            d2v xy[6], ey[6];  // rows -3 .. -1, 1 .. 3
            if constexpr (FORM) fe = row8(le, ec);
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                xy[n] = *(const d2v *)(lx + (n - 3) * ls);
                xy[n + 3] = *(const d2v *)(lx + (n + 1) * ls);
                if constexpr (FORM) {
                    ey[n] = *(const d2v *)(le + (n - 3) * ls);
                    ey[n + 3] = *(const d2v *)(le + (n + 1) * ls);
                }
            }
            d2v v;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const double *f = fx.f + e;
                double Gx, Gy, Gz;
                if constexpr (FORM) {
                    const double *h = fe.f + e;
                    Gx = d1v(ihx, h[0], h[1], h[2], h[4], h[5], h[6]);
                    Gy = d1v(ihy, ey[0][e], ey[1][e], ey[2][e], ey[3][e], ey[4][e], ey[5][e]);
                    Gz = d1v(ihz, eq[0][e], eq[1][e], eq[2][e], eq[4][e], eq[5][e], eq[6][e]);
                } else {
                    Gx = g0[e];
                    Gy = g1[e];
                    Gz = g2[e];
                }
                const double xc = xq[3][e];
                const double d2 = ihx2 * d2s(f[0], f[1], f[2], xc, f[4], f[5], f[6]) +
                                  ihy2 * d2s(xy[0][e], xy[1][e], xy[2][e], xc, xy[3][e], xy[4][e], xy[5][e]) +
                                  ihz2 * d2s(xq[0][e], xq[1][e], xq[2][e], xc, xq[4][e], xq[5][e], xq[6][e]);
                v[e] = Gx * d1v(ihx, f[0], f[1], f[2], f[4], f[5], f[6]) +
                       Gy * d1v(ihy, xy[0][e], xy[1][e], xy[2][e], xy[3][e], xy[4][e], xy[5][e]) +
                       Gz * d1v(ihz, xq[0][e], xq[1][e], xq[2][e], xq[4][e], xq[5][e], xq[6][e]) + ec[e] * d2;
                if (MODE != 0) v[e] = bv[e] - v[e];
            }
            stp<AL>(out + (MODE == 2 ? (size_t)q * g.plane + t.own_o : o), v);
        }
#pragma unroll
        for (int d = 0; d < 6; ++d) {
            xq[d] = xq[d + 1];
            if constexpr (FORM) eq[d] = eq[d + 1];
        }
        xq[6] = xn;
        if constexpr (FORM) eq[6] = en;
        __syncthreads();
    }
}

template <int MODE, class T, class TX, class TE, bool AL>
__global__ void __launch_bounds__(OP6_NT_TRANS)
k_op6_trans(Grid6 g, Op6Shape p, const TX *__restrict__ y, const TE *__restrict__ eps, const TE *__restrict__ G,
            const double *__restrict__ b, T *__restrict__ out) {
    extern __shared__ __align__(16) double op6_lds[];
    Op6Pos t;
    if (!op6_pos(g, p, t)) return;
    const int field = (p.ty + 2 * H6Y) * t.ls;
    const int kb = MODE == 2 ? p.k_w0 : 0;
    const TE *Gx = G, *Gy = G + g.N, *Gz = G + 2 * g.N;
    auto zp = [&](int k) { return (size_t)wrap(k >= g.nz ? k - g.nz : k, g.nz) * g.plane; };
    // pq, zq: eps y and Gz y at planes k - 3 .. k + 3; yq: y at planes k + 1 .. k + 3;
    // ax, ay: Gx and Gy of plane k + 1; h0, h1: the halo pair's eps y and its G y
    d2v pq[7], zq[7], yq[3], ax, ay, hy{0, 0}, he{0, 0}, hg{0, 0};
    const int kf = kb + t.q0;
    d2v y0{0, 0};
#pragma unroll
    for (int d = 0; d < 7; ++d) {
        const size_t o = zp(kf - 3 + d) + t.own_o;
        const d2v yv = ldp<AL>(y + o);
        pq[d] = ldp<true>(eps + o) * yv;
        zq[d] = ldp<true>(Gz + o) * yv;
        if (d == 3) y0 = yv;
        if (d > 3) yq[d - 4] = yv;
    }
    auto halo = [&](int k) {
        if (t.halo) {
            const size_t o = zp(k) + t.halo_o;
            hy = ldp<AL>(y + o);
            he = ldp<true>(eps + o);
            hg = ldp<true>((t.ylo ? Gy : Gx) + o);
        }
    };
    auto grads = [&](int k) {
        const size_t o = zp(k) + t.own_o;
        ax = ldp<true>(Gx + o);
        ay = ldp<true>(Gy + o);
    };
    auto stash = [&](int slot, d2v pv, d2v yv) {
        double *l0 = op6_lds + slot * 3 * field, *l1 = l0 + field, *l2 = l1 + field;
        if (t.own) {
            *(d2v *)(l0 + t.own_l) = pv;
            *(d2v *)(l1 + t.own_l) = ax * yv;
            *(d2v *)(l2 + t.own_l) = ay * yv;
        }
        if (t.halo) {
            *(d2v *)(l0 + t.halo_l) = he * hy;
            *(d2v *)((t.ylo ? l2 : l1) + t.halo_l) = hg * hy;
        }
    };
    halo(kf);
    grads(kf);
    stash(0, pq[3], y0);
    halo(kf + 1);
    grads(kf + 1);
    __syncthreads();
    const double ihx = g.ihx, ihy = g.ihy, ihz = g.ihz, ihx2 = g.ihx2, ihy2 = g.ihy2, ihz2 = g.ihz2;
    const int ls = t.ls;
    for (int q = t.q0; q < t.q1; ++q) {
        const int k = kb + q, slot = (q - t.q0) & 1;
        const size_t o = zp(k) + t.own_o;
        d2v yn{0, 0}, en{0, 0}, zn{0, 0}, bv{0, 0};
        if (MODE != 0) bv = ldp<AL>(b + o);
        if (q + 1 < t.q1) {
            stash(slot ^ 1, pq[4], yq[0]);
            const size_t on = zp(k + 4) + t.own_o;
            yn = ldp<AL>(y + on);
            en = ldp<true>(eps + on);
            zn = ldp<true>(Gz + on);
            halo(k + 2);
            grads(k + 2);
        }
        if (t.own) {
            const double *l0 = op6_lds + slot * 3 * field + t.own_l, *l1 = l0 + field, *l2 = l1 + field;
            const Row8 f0 = row8(l0, pq[3]);
            // the middle pair of Gx y is not needed by the even stencil's own point,
            // but is by its neighbour's
            const Row8 f1 = row8(l1, *(const d2v *)l1);
            d2v p0[6], p2[6];  // rows -3 .. -1, 1 .. 3 of eps y and Gy y
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                p0[n] = *(const d2v *)(l0 + (n - 3) * ls);
                p0[n + 3] = *(const d2v *)(l0 + (n + 1) * ls);
                p2[n] = *(const d2v *)(l2 + (n - 3) * ls);
                p2[n + 3] = *(const d2v *)(l2 + (n + 1) * ls);
            }
            d2v v;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const double *f = f0.f + e, *h = f1.f + e;
                const double pc = pq[3][e];
                const double d1x = d1v(ihx, h[0], h[1], h[2], h[4], h[5], h[6]);
                const double d1y = d1v(ihy, p2[0][e], p2[1][e], p2[2][e], p2[3][e], p2[4][e], p2[5][e]);
                const double d1z = d1v(ihz, zq[0][e], zq[1][e], zq[2][e], zq[4][e], zq[5][e], zq[6][e]);
                const double d2 = ihx2 * d2s(f[0], f[1], f[2], pc, f[4], f[5], f[6]) +
                                  ihy2 * d2s(p0[0][e], p0[1][e], p0[2][e], pc, p0[3][e], p0[4][e], p0[5][e]) +
                                  ihz2 * d2s(pq[0][e], pq[1][e], pq[2][e], pc, pq[4][e], pq[5][e], pq[6][e]);
                v[e] = -(d1x + d1y + d1z) + d2;
                if (MODE != 0) v[e] = bv[e] - v[e];
            }
            stp<AL>(out + (MODE == 2 ? (size_t)q * g.plane + t.own_o : o), v);
        }
#pragma unroll
        for (int d = 0; d < 6; ++d) { pq[d] = pq[d + 1]; zq[d] = zq[d + 1]; }
        pq[6] = en * yn;
        zq[6] = zn * yn;
        yq[0] = yq[1];
        yq[1] = yq[2];
        yq[2] = yn;
        __syncthreads();
    }
}

// dE/d eps_n = sum_d D1_d(lam D1_d phi)_n - lam_n (sum_d D2_d phi)_n; the inner D1
// at a shifted node uses that node's own (wrapped) offsets.
__global__ void __launch_bounds__(SX *SY)
k_grad6(Grid6 g, const double *__restrict__ phi, const double *__restrict__ lam, double *__restrict__ out) {
    const int i = blockIdx.x * SX + threadIdx.x, j = blockIdx.y * SY + threadIdx.y, k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const size_t c = (size_t)k * g.plane + (size_t)j * g.nx + i;
    const double lc = lam[c];
    double s = 0.0;
    {
        // x
        const Star s0 = star(g, i, j, k);
        const double a[3] = {A1, A2, A3};
        double acc = 0.0;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            const Star sp = star(g, wrap(i + n + 1, g.nx), j, k), sm = star(g, wrap(i - n - 1, g.nx), j, k);
            const size_t cp = c + s0.xp[n], cm = c + s0.xm[n];
            double dp = 0.0, dm = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                dp += a[q] * (phi[cp + sp.xp[q]] - phi[cp + sp.xm[q]]);
                dm += a[q] * (phi[cm + sm.xp[q]] - phi[cm + sm.xm[q]]);
            }
            acc += a[n] * (lam[cp] * dp - lam[cm] * dm);
        }
        s += g.ihx * g.ihx * acc - lc * d2(phi, c, s0.xp, s0.xm, g.ihx2);
        // y
        acc = 0.0;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            const Star sp = star(g, i, wrap(j + n + 1, g.ny), k), sm = star(g, i, wrap(j - n - 1, g.ny), k);
            const size_t cp = c + s0.yp[n], cm = c + s0.ym[n];
            double dp = 0.0, dm = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                dp += a[q] * (phi[cp + sp.yp[q]] - phi[cp + sp.ym[q]]);
                dm += a[q] * (phi[cm + sm.yp[q]] - phi[cm + sm.ym[q]]);
            }
            acc += a[n] * (lam[cp] * dp - lam[cm] * dm);
        }
        s += g.ihy * g.ihy * acc - lc * d2(phi, c, s0.yp, s0.ym, g.ihy2);
        // z
        acc = 0.0;
#pragma unroll
        for (int n = 0; n < 3; ++n) {
            const Star sp = star(g, i, j, wrap(k + n + 1, g.nz)), sm = star(g, i, j, wrap(k - n - 1, g.nz));
            const size_t cp = c + s0.zp[n], cm = c + s0.zm[n];
            double dp = 0.0, dm = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                dp += a[q] * (phi[cp + sp.zp[q]] - phi[cp + sp.zm[q]]);
                dm += a[q] * (phi[cm + sm.zp[q]] - phi[cm + sm.zm[q]]);
            }
            acc += a[n] * (lam[cp] * dp - lam[cm] * dm);
        }
        s += g.ihz * g.ihz * acc - lc * d2(phi, c, s0.zp, s0.zm, g.ihz2);
    }
    out[c] = s;
}

// psi = phi / 2 - 4 pi lam / h^3 (h^3 psi = dE/d rho);  mode 1: out = g m / h^3 (+ psi if add)
__global__ void k_charge_potential(const double *__restrict__ phi, const double *__restrict__ lam, double s4pi_h3,
                                   double *__restrict__ psi, size_t n) {
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        psi[t] = 0.5 * phi[t] - s4pi_h3 * lam[t];
}

__global__ void k_scaled_product(const double *__restrict__ gr, const double *__restrict__ m, double inv_h3,
                                 const double *__restrict__ add, double *__restrict__ out, size_t n) {
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x)
        out[t] = gr[t] * m[t] * inv_h3 + (add ? add[t] : 0.0);
}

int grid1d6(size_t n) {
    size_t b = (n + 255) / 256;
    return (int)(b > 4096 ? 4096 : b);
}

// The sixth-order operator on the finest level of the wet multigrid: the
// slab's unknowns u (a ghosted level array, slab plane q at plane q + 1) are
// taken as zero on every plane outside the slab -- the Dirichlet data of the
// wet solve, reaching the three planes the seven-point stencils span beyond
// it -- and eps, G = D1 eps are the full-box arrays, slab plane q being box
// plane (k_w0 + q) mod nz.  MODE 0: one weighted-Jacobi sweep of A6_WW u = f,
// uout = u + omega (f - A6 u) / d, d = B0 eps sum_d 1/h_d^2 the diagonal of A6
// (the seven-point stencils couple points of equal red-black colour, so the
// colour ordering of the second-order smoother does not carry over); MODE 1:
// out = f - A6 u (slab planes, not ghosted).  Sums in float64.
template <class T, int MODE>
__global__ void __launch_bounds__(SX *SY)
k_wet6(const T *__restrict__ u, T *__restrict__ out, const T *__restrict__ f, const double *__restrict__ eps,
       const double *__restrict__ G, Grid6 g, int k_w0, int nw, double omega) {
    const int i = blockIdx.x * SX + threadIdx.x, j = blockIdx.y * SY + threadIdx.y, q = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const size_t pl = g.plane;
    const size_t c = (size_t)j * g.nx + i;
    const size_t cb = (size_t)((k_w0 + q) % g.nz) * pl + c;
    auto U = [&](int qq, size_t off) -> double {
        return (qq < 0 || qq >= nw) ? 0.0 : (double)u[(size_t)(qq + 1) * pl + off];
    };
    const size_t row = (size_t)j * g.nx;
    const double u0 = U(q, c);
    double xs[3], ys[3], zs[3], xd[3], yd[3], zd[3];
#pragma unroll
    for (int n = 1; n <= 3; ++n) {
        const double xp = U(q, row + wrap(i + n, g.nx)), xm = U(q, row + wrap(i - n, g.nx));
        const double yp = U(q, (size_t)wrap(j + n, g.ny) * g.nx + i), ym = U(q, (size_t)wrap(j - n, g.ny) * g.nx + i);
        const double zp = U(q + n, c), zm = U(q - n, c);
        xs[n - 1] = xp + xm; xd[n - 1] = xp - xm;
        ys[n - 1] = yp + ym; yd[n - 1] = yp - ym;
        zs[n - 1] = zp + zm; zd[n - 1] = zp - zm;
    }
    const double d1x = g.ihx * (A1 * xd[0] + A2 * xd[1] + A3 * xd[2]);
    const double d1y = g.ihy * (A1 * yd[0] + A2 * yd[1] + A3 * yd[2]);
    const double d1z = g.ihz * (A1 * zd[0] + A2 * zd[1] + A3 * zd[2]);
    const double d2x = g.ihx2 * (B0 * u0 + B1 * xs[0] + B2 * xs[1] + B3 * xs[2]);
    const double d2y = g.ihy2 * (B0 * u0 + B1 * ys[0] + B2 * ys[1] + B3 * ys[2]);
    const double d2z = g.ihz2 * (B0 * u0 + B1 * zs[0] + B2 * zs[1] + B3 * zs[2]);
    const double e = eps[cb];
    const double a6 = G[cb] * d1x + G[g.N + cb] * d1y + G[2 * g.N + cb] * d1z + e * (d2x + d2y + d2z);
    const double fv = (double)f[(size_t)q * pl + c];
    if (MODE == 0) {
        const double d = e * B0 * (g.ihx2 + g.ihy2 + g.ihz2);
        out[(size_t)(q + 1) * pl + c] = (T)(u0 + omega * (fv - a6) / d);
    } else {
        out[(size_t)q * pl + c] = (T)(fv - a6);
    }
}

}  // namespace

void launch_d1eps(hipStream_t s, const Plan &p, const double *eps, double *G) {
    const Grid6 g = make_grid6(p);
    dim3 gr((p.nx + SX - 1) / SX, (p.ny + SY - 1) / SY, p.nz), blk(SX, SY);
    k_d1eps<<<gr, blk, 0, s>>>(g, eps, G);
    DWP_LAUNCH_CHECK();
}

// Tile and chunk of the operator: the widest tile row of whole pairs up to 48
// that divides nx (48 pairs of 96 points, 32 of a power of two), as many rows
// as divide ny within the kernel's threads (32 at most), and the chunk length
// whose blocks fill whole rounds of the resident ones (a chunk costs its planes
// and about five steps to fill its registers).  Tall tiles save halo work:
// applied to the same arrays again and again, A6 at 192 x 192 x 384 takes 173 us
// with 4 rows of 48 pairs, 121 with 8, 86 with 16; 88 with 24 rows of 32 pairs,
// 91 with 32 rows of 24.  The transpose, whose registers allow 512 threads, is
// fastest at 8 rows of 48 (768 threads spill: 2 % more on the 128 x 128 x 256
// step).
static Op6Shape op6_shape(const Plan &p, int k_w0, int nplanes, const void *fn, int most, int fields, int &nt,
                          size_t &bytes) {
    Op6Shape s{};
    s.k_w0 = k_w0;
    s.nplanes = nplanes;
    for (int w = 1; w <= 48 && w <= p.nx / 2; ++w)
        if (p.nx / 2 % w == 0) s.wp = w;
    for (int t = 1; t <= 32 && t * s.wp <= most; ++t)
        if (p.ny % t == 0) s.ty = t;
    s.tiles_x = p.nx / 2 / s.wp;
    s.tiles_y = p.ny / s.ty;
    const int nh = 4 * s.ty + 2 * H6Y * s.wp;  // halo pairs, one per thread
    nt = (std::max(s.wp * s.ty, nh) + 63) / 64 * 64;
    bytes = sizeof(double) * 2 * fields * (size_t)(s.ty + 2 * H6Y) * (2 * s.wp + 2 * H6X);
    const long slots = (long)std::max(1, cu_count() * occupancy(fn, nt, bytes));
    const long tiles = (long)s.tiles_x * s.tiles_y;
    long best = -1;
    for (int c = 1; c <= 64; ++c) {
        const long blocks = tiles * ((nplanes + c - 1) / c), cost = (blocks + slots - 1) / slots * (c + 5);
        if (best < 0 || cost < best) { best = cost; s.kc = c; }
    }
    s.nb = (int)(tiles * ((nplanes + s.kc - 1) / s.kc));
    return s;
}

static bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <int MODE, class T, class TX, class TE, bool AL>
static void op6_fwd(hipStream_t s, const Plan &p, int k_w0, int nplanes, const TX *x, const TE *eps, const TE *G,
                    const double *b, T *out) {
    int nt = 0;
    size_t bytes = 0;
    const Op6Shape sh = op6_shape(p, k_w0, nplanes, reinterpret_cast<const void *>(&k_op6_fwd<MODE, T, TX, TE, AL>),
                                  OP6_NT_FWD, sizeof(TE) == 8 ? 2 : 1, nt, bytes);
    k_op6_fwd<MODE, T, TX, TE, AL><<<(sh.nb + 7) / 8 * 8, nt, bytes, s>>>(make_grid6(p), sh, x, eps, G, b, out);
    DWP_LAUNCH_CHECK();
}
template <int MODE, class T, class TX, class TE, bool AL>
static void op6_trans(hipStream_t s, const Plan &p, int k_w0, int nplanes, const TX *y, const TE *eps, const TE *G,
                      const double *b, T *out) {
    int nt = 0;
    size_t bytes = 0;
    const Op6Shape sh = op6_shape(p, k_w0, nplanes, reinterpret_cast<const void *>(&k_op6_trans<MODE, T, TX, TE, AL>),
                                  OP6_NT_TRANS, 3, nt, bytes);
    k_op6_trans<MODE, T, TX, TE, AL><<<(sh.nb + 7) / 8 * 8, nt, bytes, s>>>(make_grid6(p), sh, y, eps, G, b, out);
    DWP_LAUNCH_CHECK();
}
// the caller's arrays (x, b, out) may be aligned to 8 bytes only
template <int MODE, class T>
static void op6_any(hipStream_t s, const Plan &p, int k_w0, int nplanes, const double *x, const double *eps,
                    const double *G, const double *b, T *out, bool trans) {
    const bool al = aligned16(x) && aligned16(out) && (MODE == 0 || aligned16(b));
    if (trans) {
        if (al) op6_trans<MODE, T, double, double, true>(s, p, k_w0, nplanes, x, eps, G, b, out);
        else op6_trans<MODE, T, double, double, false>(s, p, k_w0, nplanes, x, eps, G, b, out);
    } else {
        if (al) op6_fwd<MODE, T, double, double, true>(s, p, k_w0, nplanes, x, eps, nullptr, b, out);
        else op6_fwd<MODE, T, double, double, false>(s, p, k_w0, nplanes, x, eps, nullptr, b, out);
    }
}

void launch_apply6_f32(hipStream_t s, const Plan &p, const float *x, const float *eps, const float *G, float *out,
                       bool trans) {
    if (trans) op6_trans<0, float, float, float, true>(s, p, 0, p.nz, x, eps, G, nullptr, out);
    else op6_fwd<0, float, float, float, true>(s, p, 0, p.nz, x, eps, G, nullptr, out);
}

void launch_apply6(hipStream_t s, const Plan &p, const double *x, const double *eps, const double *G,
                   const double *b, double *out, bool residual, bool trans) {
    if (residual) op6_any<1>(s, p, 0, p.nz, x, eps, G, b, out, trans);
    else op6_any<0>(s, p, 0, p.nz, x, eps, G, b, out, trans);
}

template <class T>
void launch_wet_residual6(hipStream_t s, const Plan &p, const double *v, const double *dD, const double *eps,
                          const double *G, T *fW, bool trans) {
    op6_any<2>(s, p, p.k_w0, p.nw, dD, eps, G, v, fW, trans);
}
template <class T>
void launch_wet6(hipStream_t s, const Plan &p, const Level &L, const T *u, T *out, const double *eps, const double *G,
                 bool smooth, double omega) {
    if (L.nx != p.nx || L.ny != p.ny || L.nw != p.nw) fail(DWP_EINVAL, "internal: not the finest wet level");
    dim3 gr((p.nx + SX - 1) / SX, (p.ny + SY - 1) / SY, L.nw), blk(SX, SY);
    if (smooth) k_wet6<T, 0><<<gr, blk, 0, s>>>(u, out, L.f.as<T>(), eps, G, make_grid6(p), p.k_w0, L.nw, omega);
    else k_wet6<T, 1><<<gr, blk, 0, s>>>(u, out, L.f.as<T>(), eps, G, make_grid6(p), p.k_w0, L.nw, omega);
    DWP_LAUNCH_CHECK();
}
template void launch_wet6<float>(hipStream_t, const Plan &, const Level &, const float *, float *, const double *,
                                 const double *, bool, double);
template void launch_wet6<double>(hipStream_t, const Plan &, const Level &, const double *, double *, const double *,
                                  const double *, bool, double);

template void launch_wet_residual6<float>(hipStream_t, const Plan &, const double *, const double *, const double *,
                                          const double *, float *, bool);
template void launch_wet_residual6<double>(hipStream_t, const Plan &, const double *, const double *,
                                           const double *, const double *, double *, bool);

void launch_grad6(hipStream_t s, const Plan &p, const double *phi, const double *lam, double *g_out) {
    const Grid6 g = make_grid6(p);
    dim3 gr((p.nx + SX - 1) / SX, (p.ny + SY - 1) / SY, p.nz), blk(SX, SY);
    k_grad6<<<gr, blk, 0, s>>>(g, phi, lam, g_out);
    DWP_LAUNCH_CHECK();
}

void launch_charge_potential(hipStream_t s, const Plan &p, const double *phi, const double *lam, double *psi) {
    const double h3 = p.h[0] * p.h[1] * p.h[2];
    k_charge_potential<<<grid1d6(p.N), 256, 0, s>>>(phi, lam, FOUR_PI / h3, psi, p.N);
    DWP_LAUNCH_CHECK();
}

void launch_scaled_product(hipStream_t s, const Plan &p, const double *gr, const double *m, const double *add,
                           double *out) {
    const double h3 = p.h[0] * p.h[1] * p.h[2];
    k_scaled_product<<<grid1d6(p.N), 256, 0, s>>>(gr, m, 1.0 / h3, add, out, p.N);
    DWP_LAUNCH_CHECK();
}

}  // namespace dwp
