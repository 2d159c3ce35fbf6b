// Host stepping of the row-band sweep that interpolates a coarse correction
// into its input (band_sweep.h with PRO): every access is checked against its
// buffer, and the output must equal the interpolation written out point by
// point, added to u, then two colour passes in place -- bit for bit, with the
// threads of a step in both orders.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <limits>
#include <random>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
#define BAND_CHECK(i, n) do { if (!((size_t)(i) < (size_t)(n))) { fprintf(stderr, "out of bounds, line %d: %zu >= %zu\n", __LINE__, (size_t)(i), (size_t)(n)); abort(); } } while (0)
namespace dwp {
inline float gs_value(float off, float f, float diag) { return (off - f) / diag; }
inline double gs_value(double off, double f, double diag) { return (off - f) / diag; }
}
#include "band_sweep.h"
using namespace dwp;

template <class T, int W, bool DOWN, int PD>
void march(const BandArgs<T> &a, T *lds, int band, int chunk, int nt, bool reverse) {
    std::vector<BandSweep<T, W, false, DOWN, PD, true>> th(nt);
    for (int t = 0; t < nt; ++t) { th[t].init(a, lds, band, chunk, t); th[t].prologue(); }
    const int m0 = th[0].first(), n = th[0].nsteps(), D = DOWN ? -1 : 1;
    for (int st = 0; st < n; st += 2) {
        for (int q = 0; q < nt; ++q) th[reverse ? nt - 1 - q : q].template step<0>(m0 + D * st);
        for (int q = 0; q < nt; ++q) th[reverse ? nt - 1 - q : q].template step<1>(m0 + D * (st + 1));
    }
}

template <class T, int W>
int run(int nx, int ny, int nw, int ty, int kc, int c0, bool reverse, int zc, int nzb = 0, int kw0 = 0) {
    const size_t plane = (size_t)nx * ny, planec = plane / 4;
    const int nxc = nx / 2, nyc = ny / 2, nwc = zc ? (nw - 1) / 2 : nw;
    std::mt19937 g(nx + 31 * ny + 977 * nw + 7 * kc);
    std::uniform_real_distribution<double> U(-0.5, 0.5);
    std::vector<T> u((nw + 2) * plane, T(0)), e((nw + 2) * plane), f(nw * plane), out((nw + 2) * plane, T(0));
    std::vector<T> uc((nwc + 2) * planec, T(0)), z(nzb * plane);
    for (auto &x : e) x = (T)(40.0 + 77.0 * U(g));
    for (auto &x : f) x = (T)(10.0 * U(g));
    for (auto &x : z) x = (T)U(g);
    for (size_t i = plane; i < (nw + 1) * plane; ++i) u[i] = (T)U(g);
    for (size_t i = planec; i < (nwc + 1) * planec; ++i) uc[i] = (T)U(g);
    const T cx = (T)1.3, cy = (T)0.7, cz = (T)0.4;
    // the interpolation: coarse rows in y, planes in z (ghosted), each with its weight
    std::vector<T> ref = u;
    for (int k = 0; k < nw; ++k)
        for (int j = 0; j < ny; ++j)
            for (int i = 0; i < nx; ++i) {
                T t = 0;
                const int p0 = zc ? (k + 1) / 2 : k + 1, p1 = zc ? k / 2 + 1 : k + 1;
                for (int pz = p0; pz <= p1; ++pz)
                    for (int d = 0; d <= (j & 1); ++d) {
                        const T *r = uc.data() + pz * planec + (size_t)((j / 2 + d) % nyc) * nxc;
                        const T w = (p1 > p0 ? T(0.5) : T(1)) * ((j & 1) ? T(0.5) : T(1));
                        t += w * ((i & 1) ? T(0.5) * (r[i / 2] + r[(i / 2 + 1) % nxc]) : r[i / 2]);
                    }
                ref[(k + 1) * plane + (size_t)j * nx + i] += t;
            }
    auto at = [&](int i, int j, int k) { return (size_t)(k + 1) * plane + (size_t)((j + ny) % ny) * nx + (i + nx) % nx; };
    for (int col = 0; col < 2; ++col)
        for (int k = 0; k < nw; ++k)
            for (int j = 0; j < ny; ++j)
                for (int i = 0; i < nx; ++i)
                    if (((i + j + k) & 1) == (col ? 1 - c0 : c0))
                        ref[at(i, j, k)] = band_point<T>(
                            cx, cy, cz, e[at(i, j, k)], e[at(i + 1, j, k)], e[at(i - 1, j, k)], e[at(i, j + 1, k)],
                            e[at(i, j - 1, k)], e[at(i, j, k + 1)], e[at(i, j, k - 1)], ref[at(i + 1, j, k)],
                            ref[at(i - 1, j, k)], ref[at(i, j + 1, k)], ref[at(i, j - 1, k)], ref[at(i, j, k + 1)],
                            ref[at(i, j, k - 1)], f[(size_t)k * plane + (size_t)j * nx + i]);
    std::vector<T> want = nzb ? z : ref;
    for (int k = 0; k < (nzb ? nw : 0); ++k)
        for (size_t q = 0; q < plane; ++q) want[(size_t)((kw0 + k) % nzb) * plane + q] += ref[(k + 1) * plane + q];
    const int bands = ny / ty, nchunks = (nw + kc - 1) / kc, nt = (ty + 4) * (nx / W);
    BandArgs<T> a{u.data(), out.data(), e.data(), f.data(), nx, ny, nw, ty, bands, kc, c0, cx, cy, cz,
                  nzb ? z.data() : nullptr, nzb, kw0, uc.data(), zc};
    for (int chunk = 0; chunk < nchunks; ++chunk)
        for (int band = 0; band < bands; ++band) {
            std::vector<T> lds(band_lds_elems_pro(nx, ty), std::numeric_limits<T>::quiet_NaN());
            if (chunk & 1) {
                if (band & 1) march<T, W, true, 1>(a, lds.data(), band, chunk, nt, reverse);
                else march<T, W, true, 2>(a, lds.data(), band, chunk, nt, reverse);
            } else {
                if (band & 1) march<T, W, false, 1>(a, lds.data(), band, chunk, nt, reverse);
                else march<T, W, false, 2>(a, lds.data(), band, chunk, nt, reverse);
            }
        }
    const std::vector<T> &got = nzb ? z : out;
    size_t bad = 0;
    for (size_t i = 0; i < got.size(); ++i) bad += !(got[i] == want[i]);
    if (bad) printf("W=%d %dx%dx%d ty=%d kc=%d c0=%d rev=%d zc=%d: %zu differ\n", W, nx, ny, nw, ty, kc, c0, (int)reverse, zc, bad);
    return bad != 0;
}

int main() {
    int bad = 0;
    for (int q = 0; q < 8; ++q) {
        const int zc = q & 1, c0 = q >> 1 & 1;
        const bool rev = q >> 2;
        bad += run<float, 4>(16, 24, 21, 12, 5, c0, rev, zc);
        bad += run<float, 4>(8, 8, 7, 4, 7, c0, rev, zc);
        bad += run<float, 4>(24, 16, 1, 8, 1, c0, rev, zc);
        bad += run<float, 4>(16, 24, 21, 12, 5, c0, rev, zc, 30, 17);
        bad += run<float, 2>(12, 20, 9, 4, 2, c0, rev, zc);
        bad += run<double, 2>(12, 24, 13, 8, 3, c0, rev, zc);
        bad += run<double, 2>(4, 16, 33, 4, 6, c0, rev, zc, 40, 37);
        bad += run<double, 2>(12, 12, 3, 4, 64, c0, rev, zc);
    }
    printf("%s (%d failing cases)\n", bad ? "FAILED" : "OK", bad);
    return bad != 0;
}
