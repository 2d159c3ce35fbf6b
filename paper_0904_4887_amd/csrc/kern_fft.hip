// Periodic vacuum Poisson solve by a hand-written mixed-radix 3-D FFT.
//
// psi = L^{-1} r with L the 7-point vacuum Laplacian: in Fourier space
// psi~(m) = -r~(m) / lambda(m), lambda(m) = sum_d 4 sin^2(pi m_d / n_d) / h_d^2,
// psi~(0) = 0 -- the grid counterpart of the paper's Eq. 15, with the discrete
// symbol in place of G^2 so that the dry update inverts exactly the operator
// the wet multigrid discretises.
//
// Five passes over HBM, each a batch of 1-D transforms staged in LDS:
//   x  : two real rows packed as one complex row, forward, split (R2C)
//   y  : forward along y on tiles of consecutive kx
//   z  : forward along z, multiply by -1/(N lambda), inverse along z
//   y  : inverse
//   x  : inverse of two rows at once (C2R)
// or three where a whole z plane fits a block (x and y, z, y and x).
// Each 1-D transform is a Stockham autosort FFT with radix-8, -6, -4, -3 and -2
// stages; a stage reads its inputs into registers, synchronises, and writes
// its outputs back in place.  The spectrum and the transforms run in float64,
// or in float32 (S = float) for the mixed-precision variant; the real input
// and output grids are float64 either way.
#include "dwp_internal.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

namespace dwp {

namespace {

constexpr int FFT_THREADS = 512;
constexpr int FFT_MAXE = 4096;   // complex values per block (lines x length) at most
// Lines per block: B * n within the budget (see tile_log2), never above the
// per-block maximum, with the lines of a block within 64 KB of LDS (the n
// twiddles of the axis follow them, up to 64 KB more for n = 4096 in float64,
// where the kernel's LDS limit is raised).  The float32 x
// passes take 16 lines of 192 (measured: 0.5 ms per step less than 8).  A
// float32 z pass of 16 lines of 384 (a per-block maximum of 8192 for that
// kernel alone: 124 VGPRs, half the waves) measured 40 % slower than 8.
constexpr int FFT_BUDGET_X = 2048, FFT_BUDGET_X32 = 4096, FFT_BUDGET_Y = 4096;
// z pass: threads, lines x length per block (16 lines of 384 with 1024
// threads measured 10 % slower than 8 lines with 512)
constexpr int FFT_Z_THREADS = 512, FFT_Z_MAXE = 4096;
static_assert(FFT_Z_THREADS >= FFT_THREADS, "a radix-6 line fits every pass");
constexpr int MAX_STAGES = 12;

// Division by a small positive d through one multiply-high: with
// m = floor(2^32 / d) + 1, floor(i * m / 2^32) = floor(i / d) whenever
// i * d < 2^32, which holds for every index here (i, d < 2^16).  d = 1 is
// handled by the callers.
struct Div {
    unsigned m;
    int d;
};
Div make_div(int d) { return Div{d > 1 ? (unsigned)(0xFFFFFFFFu / (unsigned)d + 1u) : 0u, d}; }
__device__ __forceinline__ int udiv(int i, Div q) { return q.d == 1 ? i : (int)__umulhi((unsigned)i, q.m); }

// Radix plan of one axis with the per-stage constants: radix r, product p of
// the earlier radices (and its divider), and the twiddle stride n / (p r).
struct Radices {
    int n;
    int nst;
    int r[MAX_STAGES];
    int p[MAX_STAGES];
    unsigned pm[MAX_STAGES];
    int tstride[MAX_STAGES];
};

// Complex arithmetic on double2 / float2.
template <class S> struct CT;
template <> struct CT<double> { using T = double2; };
template <> struct CT<float> { using T = float2; };
template <class S> using cplx = typename CT<S>::T;
template <class C> __device__ __forceinline__ C mk(decltype(C::x) a, decltype(C::x) b) { C r; r.x = a; r.y = b; return r; }

template <class C> __device__ __forceinline__ C cmul(C a, C b) {
    return mk<C>(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
template <class C> __device__ __forceinline__ C cadd(C a, C b) { return mk<C>(a.x + b.x, a.y + b.y); }
template <class C> __device__ __forceinline__ C csub(C a, C b) { return mk<C>(a.x - b.x, a.y - b.y); }
// multiply by -i (forward) or +i (inverse)
template <class C> __device__ __forceinline__ C rot(C a, bool inv) {
    return inv ? mk<C>(-a.y, a.x) : mk<C>(a.y, -a.x);
}

template <int R, class C> struct DFT;

template <class C> struct DFT<2, C> {
    static __device__ __forceinline__ void run(C *x, bool) {
        const C a = x[0], b = x[1];
        x[0] = cadd(a, b);
        x[1] = csub(a, b);
    }
};
template <class C> struct DFT<4, C> {
    static __device__ __forceinline__ void run(C *x, bool inv) {
        const C a = cadd(x[0], x[2]), b = csub(x[0], x[2]);
        const C c = cadd(x[1], x[3]), d = csub(x[1], x[3]);
        x[0] = cadd(a, c);
        x[2] = csub(a, c);
        const C rd = rot(d, inv);  // -i d (forward)
        x[1] = cadd(b, rd);
        x[3] = csub(b, rd);
    }
};
template <class C> struct DFT<3, C> {
    static __device__ __forceinline__ void run(C *x, bool inv) {
        using S = decltype(C::x);
        // w = exp(-2 pi i / 3) = -1/2 - i sqrt(3)/2
        const S s3 = (S)0.86602540378443864676;
        const C t1 = cadd(x[1], x[2]);
        const C t2 = mk<C>(x[0].x - (S)0.5 * t1.x, x[0].y - (S)0.5 * t1.y);
        const C d = csub(x[1], x[2]);
        const C rd = rot(mk<C>(s3 * d.x, s3 * d.y), inv);  // -i s3 d (forward)
        x[0] = cadd(x[0], t1);
        x[1] = cadd(t2, rd);
        x[2] = csub(t2, rd);
    }
};
template <class C> struct DFT<6, C> {
    static __device__ __forceinline__ void run(C *x, bool inv) {
        using S = decltype(C::x);
        // two radix-3 transforms of the even and odd inputs, then one radix-2
        // layer with the sixth roots of unity w6^k = exp(-+i pi k / 3):
        // X[k] = E[k] + w6^k O[k], X[k + 3] = E[k] - w6^k O[k]
        C ev[3] = {x[0], x[2], x[4]}, od[3] = {x[1], x[3], x[5]};
        DFT<3, C>::run(ev, inv);
        DFT<3, C>::run(od, inv);
        const S h = (S)0.5, sg = inv ? (S)0.86602540378443864676 : (S)-0.86602540378443864676;
        const C t1 = mk<C>(h * od[1].x - sg * od[1].y, h * od[1].y + sg * od[1].x);    // w6 = 1/2 + i sg
        const C t2 = mk<C>(-h * od[2].x - sg * od[2].y, sg * od[2].x - h * od[2].y);   // w6^2 = -1/2 + i sg
        x[0] = cadd(ev[0], od[0]);
        x[3] = csub(ev[0], od[0]);
        x[1] = cadd(ev[1], t1);
        x[4] = csub(ev[1], t1);
        x[2] = cadd(ev[2], t2);
        x[5] = csub(ev[2], t2);
    }
};
template <class C> struct DFT<8, C> {
    static __device__ __forceinline__ void run(C *x, bool inv) {
        using S = decltype(C::x);
        // two radix-4 transforms of the even and odd inputs, then one radix-2
        // layer with the eighth roots of unity w8^k = exp(-+i pi k / 4)
        C ev[4] = {x[0], x[2], x[4], x[6]}, od[4] = {x[1], x[3], x[5], x[7]};
        DFT<4, C>::run(ev, inv);
        DFT<4, C>::run(od, inv);
        const S c = (S)0.70710678118654752440;
        const C t1 = inv ? mk<C>(c * (od[1].x - od[1].y), c * (od[1].x + od[1].y))
                         : mk<C>(c * (od[1].x + od[1].y), c * (od[1].y - od[1].x));
        const C t2 = rot(od[2], inv);
        const C t3 = inv ? mk<C>(-c * (od[3].x + od[3].y), c * (od[3].x - od[3].y))
                         : mk<C>(c * (od[3].y - od[3].x), -c * (od[3].x + od[3].y));
        x[0] = cadd(ev[0], od[0]);
        x[4] = csub(ev[0], od[0]);
        x[1] = cadd(ev[1], t1);
        x[5] = csub(ev[1], t1);
        x[2] = cadd(ev[2], t2);
        x[6] = csub(ev[2], t2);
        x[3] = cadd(ev[3], t3);
        x[7] = csub(ev[3], t3);
    }
};

// The lines of a block, B = 2^lb of them or any number: work item w is
// butterfly i of line l with w = i B + l.
struct Pow2Lines {
    int lb;
    __device__ __forceinline__ int times(int i) const { return i << lb; }
    __device__ __forceinline__ void split(int w, int &l, int &i) const {
        l = w & ((1 << lb) - 1);
        i = w >> lb;
    }
};
struct AnyLines {
    Div d;
    __device__ __forceinline__ int times(int i) const { return i * d.d; }
    __device__ __forceinline__ void split(int w, int &l, int &i) const {
        i = udiv(w, d);
        l = w - i * d.d;
    }
};

// One Stockham stage of radix R on the B lines ln of length n held in LDS;
// element t of line l sits at buf[l * ls + t * es].  p = product of the
// radices of the earlier stages.  Butterfly i of a line reads
// x_q = buf[i + q n/R], twiddles x_q by exp(-+2 pi i q (i mod p) / (p R)),
// and writes output r to (i - i mod p) R + i mod p + r p.
// IL: the lines are interleaved (es = B, ls = 1: element t of line l at
// t B + l), so that work item w = i B + l reads x_q at w + q T B and writes
// output r at ((i - k) R + k) B + l + r p B without per-element multiplies.
template <int R, class C, int MAXE, int NT, bool IL, class LN>
__device__ void stage(C *buf, int n, int p, unsigned pm, int tstride, LN ln, int es, int ls,
                      const C *__restrict__ tw, bool inv) {
    // a block of 2^lb lines whose plan holds a radix-6 stage has at most 6 NT
    // values (the host's tile budget), so that the radix-6 stage is one
    // butterfly per thread
    constexpr int E = R == 6 && std::is_same_v<LN, Pow2Lines> && MAXE > 6 * NT ? 6 * NT : MAXE;
    constexpr int K = (E / R + NT - 1) / NT;
    const int T = n / R;
    const int items = ln.times(T);
    C x[K][R];
#pragma unroll
    for (int m = 0; m < K; ++m) {
        const int w = threadIdx.x + m * NT;
        if (w < items) {
            int l, i;
            ln.split(w, l, i);
#pragma unroll
            for (int q = 0; q < R; ++q) x[m][q] = IL ? buf[w + q * items] : buf[l * ls + (i + q * T) * es];
        }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < K; ++m) {
        const int w = threadIdx.x + m * NT;
        if (w < items) {
            int l, i;
            ln.split(w, l, i);
            const int k = p > 1 ? i - p * (int)__umulhi((unsigned)i, pm) : 0;
            if (p > 1) {
                const int kt = k * tstride;
#pragma unroll
                for (int q = 1; q < R; ++q) {
                    C t = tw[q * kt];
                    if (inv) t.y = -t.y;
                    x[m][q] = cmul(x[m][q], t);
                }
            }
            DFT<R, C>::run(x[m], inv);
            const int j = (i - k) * R + k;
            const int jb = ln.times(j) + l, pb = ln.times(p);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (IL) buf[jb + r * pb] = x[m][r];
                else buf[l * ls + (j + r * p) * es] = x[m][r];
            }
        }
    }
    __syncthreads();
}

// R6: the plan may hold a radix-6 stage (a kernel built without it keeps the
// registers the radix-6 stage would need)
template <bool R6, bool IL, class C, int MAXE, int NT, class LN>
__device__ void fft_lines_of(C *buf, const Radices &rd, LN ln, int es, int ls, const C *__restrict__ tw, bool inv) {
    for (int s = 0; s < rd.nst; ++s) {
        const int R = rd.r[s];
        if (R == 8) stage<8, C, MAXE, NT, IL>(buf, rd.n, rd.p[s], rd.pm[s], rd.tstride[s], ln, es, ls, tw, inv);
        else if (R6 && R == 6) stage<6, C, MAXE, NT, IL>(buf, rd.n, rd.p[s], rd.pm[s], rd.tstride[s], ln, es, ls, tw, inv);
        else if (R == 4) stage<4, C, MAXE, NT, IL>(buf, rd.n, rd.p[s], rd.pm[s], rd.tstride[s], ln, es, ls, tw, inv);
        else if (R == 3) stage<3, C, MAXE, NT, IL>(buf, rd.n, rd.p[s], rd.pm[s], rd.tstride[s], ln, es, ls, tw, inv);
        else stage<2, C, MAXE, NT, IL>(buf, rd.n, rd.p[s], rd.pm[s], rd.tstride[s], ln, es, ls, tw, inv);
    }
}
template <bool R6, bool IL, class C, int MAXE = FFT_MAXE, int NT = FFT_THREADS>
__device__ void fft_lines(C *buf, const Radices &rd, int lb, int es, int ls, const C *__restrict__ tw, bool inv) {
    fft_lines_of<R6, IL, C, MAXE, NT>(buf, rd, Pow2Lines{lb}, es, ls, tw, inv);
}

// A block's loads of n_el values from global memory: KL per thread issued
// together, then stored (ld(e) gives value e, st(e, v) puts it in LDS), so a
// thread waits once per KL values instead of once per value.  With ntw > 0
// the ntw twiddles tw_g[] come along into tw_l[] (LDS), so that the stages
// read them from LDS.
template <int KL, int NT, class V, class Ld, class St>
__device__ __forceinline__ void load_batched(int n_el, Ld ld, St st, const V *__restrict__ tw_g = nullptr,
                                             V *tw_l = nullptr, int ntw = 0) {
    const int tot = n_el + ntw;
    for (int e0 = 0; e0 < tot; e0 += KL * NT) {
        V v[KL];
#pragma unroll
        for (int m = 0; m < KL; ++m) {
            const int e = e0 + threadIdx.x + m * NT;
            if (e < n_el) v[m] = ld(e);
            else if (e < tot) v[m] = tw_g[e - n_el];
        }
#pragma unroll
        for (int m = 0; m < KL; ++m) {
            const int e = e0 + threadIdx.x + m * NT;
            if (e < n_el) st(e, v[m]);
            else if (e < tot) tw_l[e - n_el] = v[m];
        }
    }
}
constexpr int FFT_KL = FFT_MAXE / FFT_THREADS;  // one batch covers a block of the separate passes

// ---------------------------------------------------------------- rescaling of the input
// The divisor's reciprocal of a pending rescaling (0: none), in every thread;
// the partials are added in the order of the separate kernel (256 threads, then
// four waves).  sh: four doubles.
__device__ double rescale_factor(const Rescale &rs, double *sh) {
    double v = 0.0;
    if (threadIdx.x < RED_THREADS)
        for (int b = threadIdx.x; b < rs.nparts; b += RED_THREADS) v += rs.partial[b];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (threadIdx.x < RED_THREADS && (threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double tot = 0.0;
    for (int q = 0; q < RED_THREADS / 64; ++q) tot += sh[q];
    if (blockIdx.x == 0 && threadIdx.x == 0) *rs.nu2 = tot;
    const double nu = sqrt(tot);
    return nu == 0.0 || fabs(nu - 1.0) <= rs.tol ? 0.0 : 1.0 / nu;
}
template <class V> __device__ __forceinline__ void rescale(V &v, double f, int n) {
    for (int q = 0; q < n; ++q) v[q] = (decltype(v[q] + v[q]))((double)v[q] * f);
}

// W values of a row, and the same as they lie in memory: the rows of float64
// arrays may be a caller's, which are aligned to 8 bytes only (gfx950 loads 16
// bytes from any 4-byte boundary, so the code is that of aligned vectors).
template <class T, int W> struct RowVec {
    typedef T V __attribute__((ext_vector_type(W)));
    typedef T M __attribute__((ext_vector_type(W), aligned(sizeof(T) == 8 ? 8 : W * sizeof(T))));
};
static_assert(alignof(RowVec<double, 2>::M) == 8 && alignof(RowVec<double, 4>::M) == 8);

// ---------------------------------------------------------------- x passes
// Rows are the nx-long x lines of the [nz][ny][nx] grid; B = 2^lb complex
// lines per block carry 2B real rows.  LDS lines are padded to n + 1 elements.
// The real rows move W values of both rows of a line per access, W = 4 or, for
// rows of 4 m + 2 values, 2 (single values took 96 us where pairs take 65 us,
// 162 x 216 x 432 in float64).  SC: scaled by sinv, whose rows are loaded the
// same way (value by value: 47.6 us, now 42.0 us at 192 x 192 x 384 from float32).
template <class S, class TI, bool R6, bool SC, int W>
__global__ void __launch_bounds__(FFT_THREADS)
k_fft_x_fwd(TI *in, const double *__restrict__ sinv, cplx<S> *__restrict__ out,
            Radices rd, const cplx<S> *__restrict__ tw, int lb, int nrows, int nkx, int ldc, Div dw, Div dk,
            Div dk2, Rescale rs) {
    using C = cplx<S>;
    typedef RowVec<std::remove_const_t<TI>, W> RI;
    typedef typename RI::V TIW;
    typedef double DW __attribute__((ext_vector_type(W)));
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int n = rd.n, ls = n + 1, B = 1 << lb;
    const int r0 = blockIdx.x * 2 * B;
    C *twl = lds + B * ls;
    {
        const int nw = n / W;  // dw divides by it
        for (int e = threadIdx.x; e < n; e += FFT_THREADS) twl[e] = tw[e];
        constexpr int KV = SC ? 2 : (FFT_MAXE / W + FFT_THREADS - 1) / FFT_THREADS;
        constexpr bool RS = !std::is_const<TI>::value;  // a float16 vector comes out unit
        double *rsh = reinterpret_cast<double *>(twl + n);
        double fac = 0.0;
        for (int e0 = 0; e0 < B * nw; e0 += KV * FFT_THREADS) {
            TIW va[KV], vb[KV];
            DW sa[SC ? KV : 1], sb[SC ? KV : 1];
#pragma unroll
            for (int m = 0; m < KV; ++m) {
                const int e = e0 + threadIdx.x + m * FFT_THREADS;
                if (e < B * nw) {
                    const int l = udiv(e, dw), t = e - l * nw;
                    const int ra = r0 + 2 * l;
                    if (ra + 1 < nrows) {
                        const size_t ia = (size_t)ra * n + W * t;
                        va[m] = *reinterpret_cast<const typename RI::M *>(in + ia);
                        vb[m] = *reinterpret_cast<const typename RI::M *>(in + ia + n);
                        if constexpr (SC) {
                            sa[m] = *reinterpret_cast<const DW *>(sinv + ia);
                            sb[m] = *reinterpret_cast<const DW *>(sinv + ia + n);
                        }
                    } else {
                        va[m] = vb[m] = TIW(0);
                        if constexpr (SC) sa[m] = sb[m] = DW(0);
                    }
                }
            }
            if constexpr (RS) {
                if (rs.partial) {
                    if (e0 == 0) fac = rescale_factor(rs, rsh);
                    if (fac != 0.0) {
#pragma unroll
                        for (int m = 0; m < KV; ++m) {
                            const int e = e0 + threadIdx.x + m * FFT_THREADS;
                            if (e >= B * nw) continue;
                            const int l = udiv(e, dw), t = e - l * nw, ra = r0 + 2 * l;
                            if (ra + 1 >= nrows) continue;
                            TI *x = in + (size_t)ra * n + W * t;
                            rescale(va[m], fac, W);
                            rescale(vb[m], fac, W);
                            *reinterpret_cast<typename RI::M *>(x) = va[m];
                            *reinterpret_cast<typename RI::M *>(x + n) = vb[m];
                        }
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < KV; ++m) {
                const int e = e0 + threadIdx.x + m * FFT_THREADS;
                if (e < B * nw) {
                    const int l = udiv(e, dw), t = e - l * nw;
#pragma unroll
                    for (int q = 0; q < W; ++q) {
                        double a = (double)va[m][q], b = (double)vb[m][q];
                        if constexpr (SC) { a *= sa[m][q]; b *= sb[m][q]; }
                        lds[l * ls + W * t + q] = mk<C>((S)a, (S)b);
                    }
                }
            }
        }
    }
    __syncthreads();
    fft_lines<R6, false>(lds, rd, lb, 1, ls, twl, false);
    if constexpr (sizeof(S) == 4) {
        // two neighbouring kx per thread, stored as 16-byte pairs (ldc even)
        const int nk2 = (nkx + 1) >> 1;
        const S h = (S)0.5;
        for (int e = threadIdx.x; e < B * nk2; e += FFT_THREADS) {
            const int l = udiv(e, dk2), k = 2 * (e - l * nk2);
            const int ra = r0 + 2 * l, rb = ra + 1;
            if (rb >= nrows) continue;
            float4 A, Bq;
            {
                const C z = lds[l * ls + k], zc = lds[l * ls + (k == 0 ? 0 : n - k)];  // Z[k], Z[-k]
                A.x = h * (z.x + zc.x); A.y = h * (z.y - zc.y);
                Bq.x = h * (z.y + zc.y); Bq.y = -h * (z.x - zc.x);
            }
            if (k + 1 < nkx) {
                const C z = lds[l * ls + k + 1], zc = lds[l * ls + n - k - 1];
                A.z = h * (z.x + zc.x); A.w = h * (z.y - zc.y);
                Bq.z = h * (z.y + zc.y); Bq.w = -h * (z.x - zc.x);
                *reinterpret_cast<float4 *>(out + (size_t)ra * ldc + k) = A;
                *reinterpret_cast<float4 *>(out + (size_t)rb * ldc + k) = Bq;
            } else {
                out[(size_t)ra * ldc + k] = mk<C>(A.x, A.y);
                out[(size_t)rb * ldc + k] = mk<C>(Bq.x, Bq.y);
            }
        }
        return;
    }
    for (int e = threadIdx.x; e < B * nkx; e += FFT_THREADS) {
        const int l = udiv(e, dk), k = e - l * nkx;
        const int ra = r0 + 2 * l, rb = ra + 1;
        if (rb >= nrows) continue;
        const C z = lds[l * ls + k];
        const C zc = lds[l * ls + (k == 0 ? 0 : n - k)];  // Z[-k]
        // A = (Z + conj Z[-k]) / 2, B = (Z - conj Z[-k]) / (2 i)
        const S h = (S)0.5;
        out[(size_t)ra * ldc + k] = mk<C>(h * (z.x + zc.x), h * (z.y - zc.y));
        out[(size_t)rb * ldc + k] = mk<C>(h * (z.y + zc.y), -h * (z.x - zc.x));
    }
}

// The half spectrum of a line's two rows is read once, 16 bytes at a time (KN
// values of kx), and each value k also gives the value n - k of the Hermitian
// extension; the real rows leave as in the forward pass.  (Reading every value
// twice, once per row value: 28.9 us, now 23.9 at 192 x 192 x 384 in float32,
// 15.9 -> 9.8 at 96 x 96 x 192 and 90 -> 56 at 162 x 216 x 432 in float64.)
template <class S, class TO, bool R6, bool SC, int W>
__global__ void __launch_bounds__(FFT_THREADS)
k_fft_x_inv(const cplx<S> *__restrict__ in, const double *__restrict__ sinv, TO *__restrict__ out,
            Radices rd, const cplx<S> *__restrict__ tw, int lb, int nrows, int nkx, int ldc, Div dw, Div dk) {
    using C = cplx<S>;
    constexpr int KN = 16 / sizeof(C);
    typedef S SV __attribute__((ext_vector_type(2 * KN)));
    typedef RowVec<TO, W> RO;
    typedef double DW __attribute__((ext_vector_type(W)));
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int n = rd.n, ls = n + 1, B = 1 << lb;
    const int r0 = blockIdx.x * 2 * B;
    C *twl = lds + B * ls;
    for (int e = threadIdx.x; e < n; e += FFT_THREADS) twl[e] = tw[e];
    const int nk = (nkx + KN - 1) / KN;  // dk divides by it
    constexpr int KL = FFT_MAXE / 2 / KN / FFT_THREADS;
    for (int e0 = 0; e0 < B * nk; e0 += KL * FFT_THREADS) {
        SV va[KL], vb[KL];
#pragma unroll
        for (int m = 0; m < KL; ++m) {
            const int e = e0 + threadIdx.x + m * FFT_THREADS;
            va[m] = vb[m] = SV(0);
            if (e < B * nk) {
                const int l = udiv(e, dk), k = KN * (e - l * nk), ra = r0 + 2 * l;
                if (ra + 1 < nrows) {  // rows are padded to a multiple of 8 values
                    va[m] = *reinterpret_cast<const SV *>(in + (size_t)ra * ldc + k);
                    vb[m] = *reinterpret_cast<const SV *>(in + (size_t)(ra + 1) * ldc + k);
                }
            }
        }
#pragma unroll
        for (int m = 0; m < KL; ++m) {
            const int e = e0 + threadIdx.x + m * FFT_THREADS;
            if (e < B * nk) {
                const int l = udiv(e, dk), k0 = KN * (e - l * nk);
#pragma unroll
                for (int q = 0; q < KN; ++q) {
                    const int k = k0 + q;
                    if (k >= nkx) continue;
                    C A = mk<C>(va[m][2 * q], va[m][2 * q + 1]), Bv = mk<C>(vb[m][2 * q], vb[m][2 * q + 1]);
                    const bool self = k == 0 || 2 * k == n;
                    if (self) { A.y = 0; Bv.y = 0; }
                    lds[l * ls + k] = mk<C>(A.x - Bv.y, A.y + Bv.x);                  // A + i B
                    if (!self) lds[l * ls + n - k] = mk<C>(A.x + Bv.y, Bv.x - A.y);   // conj A + i conj B
                }
            }
        }
    }
    __syncthreads();
    fft_lines<R6, false>(lds, rd, lb, 1, ls, twl, true);
    const int nw = n / W;  // dw divides by it
    for (int e = threadIdx.x; e < B * nw; e += FFT_THREADS) {
        const int l = udiv(e, dw), t = e - l * nw;
        const int ra = r0 + 2 * l;
        if (ra + 1 >= nrows) continue;
        const size_t ia = (size_t)ra * n + W * t;
        DW sa, sb;
        if constexpr (SC) {
            sa = *reinterpret_cast<const DW *>(sinv + ia);
            sb = *reinterpret_cast<const DW *>(sinv + ia + n);
        }
        typename RO::V a, b;
#pragma unroll
        for (int q = 0; q < W; ++q) {
            const C z = lds[l * ls + W * t + q];
            if constexpr (SC) {
                a[q] = (TO)((double)z.x * sa[q]);
                b[q] = (TO)((double)z.y * sb[q]);
            } else {
                a[q] = (TO)z.x;
                b[q] = (TO)z.y;
            }
        }
        *reinterpret_cast<typename RO::M *>(out + ia) = a;
        *reinterpret_cast<typename RO::M *>(out + ia + n) = b;
    }
}

// Block -> (line tile, row) of the y and z passes, XCD-aware: the grid is
// one-dimensional and padded to a multiple of 8; hardware block b runs on XCD
// b mod 8, which gets the contiguous run of tiles [xcd * per, (xcd + 1) * per),
// so the line tiles of one row (which share the 128-byte cache lines at their
// edges) run side by side on one XCD and its L2 serves the shared lines once.
// Returns false for the padding blocks.  (Tiles that leave out the columns
// beyond the last full group of B, with those columns' lines grouped along
// the rows instead, measured slower: their scattered accesses form a tail.)
__device__ __forceinline__ bool xcd_tile2(int ntx, int nty, int &tx, int &ty) {
    const int per = gridDim.x / 8;
    const int t = (blockIdx.x % 8) * per + blockIdx.x / 8;
    if (t >= ntx * nty) return false;
    ty = t / ntx;
    tx = t - ty * ntx;
    return true;
}
inline int xcd_grid(int n) { return (n + 7) / 8 * 8; }

// Float32 spectrum, lines interleaved in LDS (element t of line l at t B + l,
// B = 2^lb >= 2): the block's B n values move between the spectrum (element
// t of line l at base + t stride + l) and LDS two neighbouring lines per
// 16-byte access; lines from bw on are zero in LDS and are not written back.
// pair_load also brings the n twiddles into twl.
__device__ __forceinline__ void pair_load(float2 *lds, const float2 *__restrict__ c, size_t base, size_t stride,
                                          int lb, int n, int bw, const float2 *__restrict__ tw, float2 *twl) {
    for (int e = threadIdx.x; e < n; e += FFT_THREADS) twl[e] = tw[e];
    constexpr int KP = FFT_MAXE / 2 / FFT_THREADS;
    const int np = (n << lb) >> 1, hmask = (1 << (lb - 1)) - 1;
    for (int e0 = 0; e0 < np; e0 += KP * FFT_THREADS) {
        float4 v[KP];
#pragma unroll
        for (int m = 0; m < KP; ++m) {
            const int e = e0 + threadIdx.x + m * FFT_THREADS;
            if (e < np) {
                const int t = e >> (lb - 1), l = (e & hmask) << 1;
                const float2 *src = c + base + (size_t)t * stride + l;
                if (l + 1 < bw) v[m] = *reinterpret_cast<const float4 *>(src);
                else if (l < bw) v[m] = make_float4(src->x, src->y, 0.0f, 0.0f);
                else v[m] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        }
#pragma unroll
        for (int m = 0; m < KP; ++m) {
            const int e = e0 + threadIdx.x + m * FFT_THREADS;
            if (e < np) reinterpret_cast<float4 *>(lds)[e] = v[m];
        }
    }
}
__device__ __forceinline__ void pair_store(const float2 *lds, float2 *__restrict__ c, size_t base, size_t stride,
                                           int lb, int n, int bw) {
    const int np = (n << lb) >> 1, hmask = (1 << (lb - 1)) - 1;
    for (int e = threadIdx.x; e < np; e += FFT_THREADS) {
        const int t = e >> (lb - 1), l = (e & hmask) << 1;
        float2 *dst = c + base + (size_t)t * stride + l;
        const float4 v = reinterpret_cast<const float4 *>(lds)[e];
        if (l + 1 < bw) *reinterpret_cast<float4 *>(dst) = v;
        else if (l < bw) *dst = make_float2(v.x, v.y);
    }
}

// ---------------------------------------------------------------- y pass
// Block (tile of B = 2^lb consecutive kx, plane z): lines along y, LDS
// element (y, l) at y * B + l.
// INV: the inverse transform (a template argument, so that the butterflies'
// direction is fixed at compile time).
template <class S, bool R6, bool INV>
__global__ void __launch_bounds__(FFT_THREADS)
k_fft_y(cplx<S> *__restrict__ c, Radices rd, const cplx<S> *__restrict__ tw, int lb, int nkx, int ldc, int nz) {
    using C = cplx<S>;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int ny = rd.n, B = 1 << lb, bmask = B - 1;
    int bt, z;
    if (!xcd_tile2((nkx + B - 1) / B, nz, bt, z)) return;
    const int kx0 = bt * B;
    const int bw = min(B, nkx - kx0);
    const size_t base = (size_t)z * ny * ldc + kx0;
    C *twl = lds + B * ny;
    constexpr bool PAIRS = sizeof(S) == 4;
    if (PAIRS && lb >= 1) {
        pair_load(reinterpret_cast<float2 *>(lds), reinterpret_cast<const float2 *>(c), base, ldc, lb, ny, bw,
                  reinterpret_cast<const float2 *>(tw), reinterpret_cast<float2 *>(twl));
    } else {
        load_batched<FFT_KL, FFT_THREADS, C>(
            B * ny,
            [&](int e) {
                const int y = e >> lb, l = e & bmask;
                return (l < bw) ? c[base + (size_t)y * ldc + l] : mk<C>(0, 0);
            },
            [&](int e, C v) { lds[e] = v; }, tw, twl, ny);
    }
    __syncthreads();
    fft_lines<R6, true>(lds, rd, lb, B, 1, twl, INV);
    if (PAIRS && lb >= 1) {
        pair_store(reinterpret_cast<const float2 *>(lds), reinterpret_cast<float2 *>(c), base, ldc, lb, ny, bw);
        return;
    }
    for (int e = threadIdx.x; e < B * ny; e += FFT_THREADS) {
        const int y = e >> lb, l = e & bmask;
        if (l < bw) c[base + (size_t)y * ldc + l] = lds[e];
    }
}

// ---------------------------------------------------------------- x and y passes of a small plane
// One block of NT threads transforms a whole z plane along x and along y, so
// the half spectrum does not go to memory in between: the ny / 2 packed lines
// of the x pass (padded to n + 1), split in registers into the ny x nkx values
// of the y pass (interleaved: value (y, k) at y nkx + k) in the same LDS.  The
// arithmetic is that of the separate passes.  At most PE NT values of either
// form (PE per thread; what a stage keeps in registers).  Bound by the LDS
// traffic and the barriers of a block's own chain of stages, the memory idle
// meanwhile; the separate passes overlap their blocks but move the spectrum
// four more times.  Whole solve, five passes against three, us: 25.5 -> 18.4 at
// 32 x 32 x 64, 70 -> 51 at 96 x 96 x 192, 106 -> 84 at 128 x 128 x 256 in
// float64; 51.5 -> 40, 74 -> 55 in float32.  (Planes of up to 192 x 192 in
// float32, 20 values a thread: 157 -> 187 us at 192 x 192 x 384, one block a
// CU and nothing to overlap with.)
template <class S, class TI, bool SC, int NT, int PE>
__global__ void __launch_bounds__(NT)
k_fft_xy_fwd(TI *in, const double *__restrict__ sinv, cplx<S> *__restrict__ out, Radices rx,
             Radices ry, const cplx<S> *__restrict__ twx, const cplx<S> *__restrict__ twy, int ldc, Div dl, Div dw,
             Div dk, Rescale rs) {
    using C = cplx<S>;
    constexpr int MAXE = PE * NT;
    typedef RowVec<std::remove_const_t<TI>, 2> RI;
    typedef typename RI::V TIW;
    typedef double DW __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int n = rx.n, ls = n + 1, ny = ry.n, nl = ny >> 1, nkx = dk.d;
    const size_t z = blockIdx.x;
    C *tx = lds + max(nl * ls, ny * nkx), *ty = tx + n;
    for (int e = threadIdx.x; e < n + ny; e += NT) tx[e] = e < n ? twx[e] : twy[e - n];
    {
        const int nw = n >> 1;  // dw divides by it
        constexpr int KV = (PE + 1) / 2;
        TIW va[KV], vb[KV];
        DW sa[SC ? KV : 1], sb[SC ? KV : 1];
#pragma unroll
        for (int m = 0; m < KV; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nw) {
                const int l = udiv(e, dw), t = e - l * nw;
                const size_t ia = (z * ny + 2 * l) * n + 2 * t;
                va[m] = *reinterpret_cast<const typename RI::M *>(in + ia);
                vb[m] = *reinterpret_cast<const typename RI::M *>(in + ia + n);
                if constexpr (SC) {
                    sa[m] = *reinterpret_cast<const DW *>(sinv + ia);
                    sb[m] = *reinterpret_cast<const DW *>(sinv + ia + n);
                }
            }
        }
        if constexpr (!std::is_const<TI>::value) {  // a float16 vector comes out unit
            if (rs.partial) {
                const double fac = rescale_factor(rs, reinterpret_cast<double *>(ty + ny));
                if (fac != 0.0) {
#pragma unroll
                    for (int m = 0; m < KV; ++m) {
                        const int e = threadIdx.x + m * NT;
                        if (e >= nl * nw) continue;
                        const int l = udiv(e, dw), t = e - l * nw;
                        TI *x = in + (z * ny + 2 * l) * n + 2 * t;
                        rescale(va[m], fac, 2);
                        rescale(vb[m], fac, 2);
                        *reinterpret_cast<typename RI::M *>(x) = va[m];
                        *reinterpret_cast<typename RI::M *>(x + n) = vb[m];
                    }
                }
            }
        }
#pragma unroll
        for (int m = 0; m < KV; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nw) {
                const int l = udiv(e, dw), t = e - l * nw;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    double a = (double)va[m][q], b = (double)vb[m][q];
                    if constexpr (SC) { a *= sa[m][q]; b *= sb[m][q]; }
                    lds[l * ls + 2 * t + q] = mk<C>((S)a, (S)b);
                }
            }
        }
    }
    __syncthreads();
    fft_lines_of<true, false, C, MAXE, NT>(lds, rx, AnyLines{dl}, 1, ls, tx, false);
    {
        constexpr int KS = (PE + 1) / 2;
        C A[KS], Bv[KS];
        const S h = (S)0.5;
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nkx) {
                const int l = udiv(e, dk), k = e - l * nkx;
                const C v = lds[l * ls + k], vc = lds[l * ls + (k == 0 ? 0 : n - k)];
                A[m] = mk<C>(h * (v.x + vc.x), h * (v.y - vc.y));
                Bv[m] = mk<C>(h * (v.y + vc.y), -h * (v.x - vc.x));
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nkx) {
                const int l = udiv(e, dk);
                lds[e + l * nkx] = A[m];           // (2 l) nkx + k
                lds[e + (l + 1) * nkx] = Bv[m];
            }
        }
    }
    __syncthreads();
    fft_lines_of<true, true, C, MAXE, NT>(lds, ry, AnyLines{dk}, nkx, 1, ty, false);
    for (int e = threadIdx.x; e < ny * nkx; e += NT) {
        const int y = udiv(e, dk), k = e - y * nkx;
        out[(z * ny + y) * ldc + k] = lds[e];
    }
}

template <class S, class TO, bool SC, int NT, int PE>
__global__ void __launch_bounds__(NT)
k_fft_xy_inv(const cplx<S> *__restrict__ in, const double *__restrict__ sinv, TO *__restrict__ out, Radices rx,
             Radices ry, const cplx<S> *__restrict__ twx, const cplx<S> *__restrict__ twy, int ldc, Div dl, Div dw,
             Div dk) {
    using C = cplx<S>;
    constexpr int MAXE = PE * NT;
    typedef RowVec<TO, 2> RO;
    typedef double DW __attribute__((ext_vector_type(2)));
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int n = rx.n, ls = n + 1, ny = ry.n, nl = ny >> 1, nkx = dk.d;
    const size_t z = blockIdx.x;
    C *tx = lds + max(nl * ls, ny * nkx), *ty = tx + n;
    for (int e = threadIdx.x; e < n + ny; e += NT) tx[e] = e < n ? twx[e] : twy[e - n];
    load_batched<6, NT, C>(
        ny * nkx,
        [&](int e) {
            const int y = udiv(e, dk), k = e - y * nkx;
            return in[(z * ny + y) * ldc + k];
        },
        [&](int e, C v) { lds[e] = v; });
    __syncthreads();
    fft_lines_of<true, true, C, MAXE, NT>(lds, ry, AnyLines{dk}, nkx, 1, ty, true);
    {
        constexpr int KS = (PE + 1) / 2;
        C A[KS], Bv[KS];
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nkx) {
                const int l = udiv(e, dk);
                A[m] = lds[e + l * nkx];
                Bv[m] = lds[e + (l + 1) * nkx];
            }
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < KS; ++m) {
            const int e = threadIdx.x + m * NT;
            if (e < nl * nkx) {
                const int l = udiv(e, dk), k = e - l * nkx;
                C a = A[m], b = Bv[m];
                const bool self = k == 0 || 2 * k == n;
                if (self) { a.y = 0; b.y = 0; }
                lds[l * ls + k] = mk<C>(a.x - b.y, a.y + b.x);
                if (!self) lds[l * ls + n - k] = mk<C>(a.x + b.y, b.x - a.y);
            }
        }
    }
    __syncthreads();
    fft_lines_of<true, false, C, MAXE, NT>(lds, rx, AnyLines{dl}, 1, ls, tx, true);
    const int nw = n >> 1;  // dw divides by it
    for (int e = threadIdx.x; e < nl * nw; e += NT) {
        const int l = udiv(e, dw), t = e - l * nw;
        const size_t ia = (z * ny + 2 * l) * n + 2 * t;
        const C v0 = lds[l * ls + 2 * t], v1 = lds[l * ls + 2 * t + 1];
        typename RO::V a, b;
        if constexpr (SC) {
            const DW sa = *reinterpret_cast<const DW *>(sinv + ia), sb = *reinterpret_cast<const DW *>(sinv + ia + n);
            a[0] = (TO)((double)v0.x * sa[0]);
            a[1] = (TO)((double)v1.x * sa[1]);
            b[0] = (TO)((double)v0.y * sb[0]);
            b[1] = (TO)((double)v1.y * sb[1]);
        } else {
            a[0] = (TO)v0.x;
            a[1] = (TO)v1.x;
            b[0] = (TO)v0.y;
            b[1] = (TO)v1.y;
        }
        *reinterpret_cast<typename RO::M *>(out + ia) = a;
        *reinterpret_cast<typename RO::M *>(out + ia + n) = b;
    }
}

// ---------------------------------------------------------------- z pass + Green
// -1 / lambda through the hardware reciprocal (two Newton steps in float64).
__device__ __forceinline__ double neg_recip(double d) {
    double r = __builtin_amdgcn_rcp(d);
    double e = __builtin_fma(-d, r, 1.0);
    r = __builtin_fma(r, e, r);
    e = __builtin_fma(-d, r, 1.0);
    r = __builtin_fma(r, e, r);
    return -r;
}
__device__ __forceinline__ float neg_recip(float d) { return -__builtin_amdgcn_rcpf(d); }

// Block (tile of B = 2^lb consecutive kx, row y): lines along z, LDS element
// (z, l) at z * B + l.
template <class S, bool R6, int MAXE = FFT_MAXE, int NT = FFT_THREADS>
__global__ void __launch_bounds__(NT)
k_fft_z_green(cplx<S> *__restrict__ c, Radices rd, const cplx<S> *__restrict__ tw, int lb, int nkx, int ldc, int ny,
              const S *__restrict__ lamx, const S *__restrict__ lamy, const S *__restrict__ lamz, S inv_n,
              int lam_lds) {
    using C = cplx<S>;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    C *lds = reinterpret_cast<C *>(lds_raw);
    const int nz = rd.n, B = 1 << lb, bmask = B - 1;
    int bt, y;
    if (!xcd_tile2((nkx + B - 1) / B, ny, bt, y)) return;
    const int kx0 = bt * B;
    const int bw = min(B, nkx - kx0);
    const size_t zstride = (size_t)ny * ldc;
    const size_t base = (size_t)y * ldc + kx0;
    C *twl = lds + B * nz;
    // with lam_lds the symbol's z values and the block's kx values follow
    // the twiddles, loaded with the lines (the Green step then reads LDS only)
    S *lz = reinterpret_cast<S *>(twl + nz), *lx = lz + nz;
    if (lam_lds) {
        for (int e = threadIdx.x; e < nz + B; e += NT) {
            if (e < nz) lz[e] = lamz[e];
            else if (kx0 + e - nz < nkx) lx[e - nz] = lamx[kx0 + e - nz];
        }
    }
    constexpr bool PAIRS = sizeof(S) == 4 && NT == FFT_THREADS && MAXE == FFT_MAXE;
    if (PAIRS && lb >= 1) {
        pair_load(reinterpret_cast<float2 *>(lds), reinterpret_cast<const float2 *>(c), base, zstride, lb, nz, bw,
                  reinterpret_cast<const float2 *>(tw), reinterpret_cast<float2 *>(twl));
    } else {
        load_batched<(MAXE + NT - 1) / NT, NT, C>(
            B * nz,
            [&](int e) {
                const int z = e >> lb, l = e & bmask;
                return (l < bw) ? c[base + (size_t)z * zstride + l] : mk<C>(0, 0);
            },
            [&](int e, C v) { lds[e] = v; }, tw, twl, nz);
    }
    __syncthreads();
    fft_lines<R6, true, C, MAXE, NT>(lds, rd, lb, B, 1, twl, false);
    const S ly = lamy[y];
    for (int e = threadIdx.x; e < B * nz; e += NT) {
        const int z = e >> lb, l = e & bmask;
        const int kx = kx0 + l;
        S g = 0;
        if (l < bw && (kx | y | z) != 0)
            g = inv_n * neg_recip((lam_lds ? lx[l] : lamx[kx]) + ly + (lam_lds ? lz[z] : lamz[z]));
        const C v = lds[e];
        lds[e] = mk<C>(v.x * g, v.y * g);
    }
    __syncthreads();
    fft_lines<R6, true, C, MAXE, NT>(lds, rd, lb, B, 1, twl, true);
    if (PAIRS && lb >= 1) {
        pair_store(reinterpret_cast<const float2 *>(lds), reinterpret_cast<float2 *>(c), base, zstride, lb, nz, bw);
        return;
    }
    for (int e = threadIdx.x; e < B * nz; e += NT) {
        const int z = e >> lb, l = e & bmask;
        if (l < bw) c[base + (size_t)z * zstride + l] = lds[e];
    }
}

// Raise a kernel's dynamic LDS limit to 160 KB, once per device (bit d of
// `done`), when a launch asks for more than the default 64 KB.
void lds_attr(const void *fn, std::atomic<unsigned> &done, size_t bytes) {
    if (bytes <= 64 * 1024) return;
    int dev = 0;
    DWP_HIP(hipGetDevice(&dev));
    const unsigned bit = 1u << (dev & 31);
    if (done.load() & bit) return;
    DWP_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    done.fetch_or(bit);
}
template <class F> const void *fptr(F *f) { return reinterpret_cast<const void *>(f); }

Radices radices_of(const FFTAxis &ax) {
    Radices r{};
    r.n = ax.n;
    r.nst = (int)ax.radices.size();
    int p = 1;
    for (int s = 0; s < r.nst; ++s) {
        r.r[s] = ax.radices[s];
        r.p[s] = p;
        r.pm[s] = make_div(p).m;
        r.tstride[s] = ax.n / (p * ax.radices[s]);
        p *= ax.radices[s];
    }
    return r;
}

// Lines per block: the largest power of two with B * n <= budget, capped at
// 16 (16 lines of the padded spectrum are 256 contiguous bytes).
int tile_log2(int n, int budget) {
    int lb = 0;
    while (lb < 4 && (2 << lb) * n <= budget) ++lb;
    return lb;
}

// Whether the x and y passes of a plane of pv values run in one block (bytes
// of LDS), nz blocks in all.  Small planes always do (8 x 8 x 8: 22 -> 16 us).
// Larger ones need the planes to occupy the chip: a block's chain of stages
// takes what it takes however few there are (96 x 96 in float64: 29 us by
// separate passes and 31 in one at nz = 8, 39 and 37.5 at 64, 70 and 51 at
// 192).  Past PLANE_MID one block fills a CU, so the last round over the (256)
// CUs has to be worth it (128 x 128: 112 and 114 us at nz = 288, 138 and 127
// at 384, 182 and 185 at 576; 40 and 48 at 32, 54 and 54 at 64).
constexpr int PLANE_SMALL = 6 * 512, PLANE_MID = 6 * 1024, PLANE_MAX = 10 * 1024;
bool plane_pass(int pv, size_t bytes, int nz) {
    if (pv <= PLANE_SMALL) return true;
    if (pv <= PLANE_MID) return nz >= 64;
    if (pv > PLANE_MAX || bytes > 160 * 1024) return false;
    const int cus = cu_count(), last = nz % cus;
    return last == 0 || 8 * last >= 3 * cus;
}

}  // namespace

// Radix plan, twiddles and the discrete symbol 4 sin^2(pi m / n) / h^2 of one
// axis (m < n / 2 + 1 when `half`).  Twiddles and symbol are evaluated in long
// double on the host.
void fft_plan_axis(FFTAxis &ax, int n, double h, bool half, int order) {
    ax.n = n;
    ax.radices.clear();
    int m = n, a = 0, b = 0;
    while (m % 3 == 0) { ++a; m /= 3; }
    while (m % 2 == 0) { ++b; m /= 2; }
    // radix 8 for the power of two as far as it goes; a lone factor 2 left
    // over pairs with a factor 3 into one radix-6 stage (384 = 6 8 8: three
    // stages instead of four) on lines short enough for one radix-6
    // butterfly per thread of a block
    const bool six = a > 0 && b % 3 == 1 && n <= 6 * FFT_THREADS;
    for (int i = 0; i < a - (six ? 1 : 0); ++i) ax.radices.push_back(3);
    if (six) ax.radices.push_back(6);
    for (int i = 0; i < b / 3; ++i) ax.radices.push_back(8);
    if (b % 3 == 2) ax.radices.push_back(4);
    if (b % 3 == 1 && !six) ax.radices.push_back(2);
    if (m != 1 || (int)ax.radices.size() > MAX_STAGES) fail(DWP_EINVAL, "grid size must be 2^a 3^b");
    const long double pi = 3.141592653589793238462643383279502884L;
    std::vector<double2> tw(n);
    std::vector<float2> tw32(n);
    for (int t = 0; t < n; ++t) {
        const long double a = -2.0L * pi * (long double)t / (long double)n;
        tw[t] = make_double2((double)cosl(a), (double)sinl(a));
        tw32[t] = make_float2((float)cosl(a), (float)sinl(a));
    }
    const int nl = half ? n / 2 + 1 : n;
    std::vector<double> lam(nl);
    std::vector<float> lam32(nl);
    for (int k = 0; k < nl; ++k) {
        if (order == 6) {
            // minus the eigenvalue of the seven-point second derivative (Eq. 18)
            const long double th = 2.0L * pi * (long double)k / (long double)n;
            const long double v = -(-49.0L / 18.0L) - 2.0L * (1.5L * cosl(th) - 0.15L * cosl(2.0L * th) +
                                                                 cosl(3.0L * th) / 90.0L);
            lam[k] = (double)(v / ((long double)h * (long double)h));
        } else {
            const long double s = sinl(pi * (long double)k / (long double)n);
            lam[k] = (double)(4.0L * s * s / ((long double)h * (long double)h));
        }
        lam32[k] = (float)lam[k];
    }
    ax.tw.alloc(sizeof(double2) * n);
    ax.lam.alloc(sizeof(double) * nl);
    ax.tw32.alloc(sizeof(float2) * n);
    ax.lam32.alloc(sizeof(float) * nl);
    DWP_HIP(hipMemcpy(ax.tw.p, tw.data(), sizeof(double2) * n, hipMemcpyHostToDevice));
    DWP_HIP(hipMemcpy(ax.lam.p, lam.data(), sizeof(double) * nl, hipMemcpyHostToDevice));
    DWP_HIP(hipMemcpy(ax.tw32.p, tw32.data(), sizeof(float2) * n, hipMemcpyHostToDevice));
    DWP_HIP(hipMemcpy(ax.lam32.p, lam32.data(), sizeof(float) * nl, hipMemcpyHostToDevice));
}

template <class S, class TI, class TO>
static void vacuum_solve_t(hipStream_t st, const Plan &p, const FFTAxis &ax, const FFTAxis &ay, const FFTAxis &az,
                           TI *r, const double *sinv, void *cbuf_v, TO *out, Profiler *prof, const Rescale &rs) {
    using C = cplx<S>;
    C *cbuf = static_cast<C *>(cbuf_v);
    auto TW = [](const FFTAxis &a) { return sizeof(S) == 8 ? a.tw.as<C>() : a.tw32.as<C>(); };
    auto LAM = [](const FFTAxis &a) { return sizeof(S) == 8 ? a.lam.as<S>() : a.lam32.as<S>(); };
    // algorithmic bytes of each pass: the real grid (8 B / point, twice when
    // scaled) and the half-spectrum (one complex value) read and written once
    const double Cn = (double)p.nkx * p.ny * p.nz, cb = (double)sizeof(C);
    const double bx = (sinv ? 8.0 + sizeof(TI) : (double)sizeof(TI)) * p.N + cb * Cn;
    const double bxi = (sinv ? 8.0 + sizeof(TO) : (double)sizeof(TO)) * p.N + cb * Cn;
    auto pb = [&](int g) { return prof ? prof->begin(st, g) : -1; };
    auto pe = [&](int ev, int g, double b) { if (prof) prof->end(st, ev, g, b); };
    int ev;
    // each pass in the variant with or without a radix-6 stage, as its axis'
    // plan needs (the radix-6 code costs registers where it is not used)
    auto has6 = [](const FFTAxis &a) { return std::find(a.radices.begin(), a.radices.end(), 6) != a.radices.end(); };
    auto RD = [](const FFTAxis &a) { return radices_of(a); };
    // a pass with a radix-6 stage takes at most 6 values per thread in a block
    auto budget = [&](const FFTAxis &a, int b, int nt) { return has6(a) ? std::min(b, 6 * nt) : b; };
    auto with6 = [](bool six, auto &&f) {
        if (six) f(std::true_type{});
        else f(std::false_type{});
    };
    const int nrows = p.ny * p.nz;
    const int lbx = tile_log2(p.nx, budget(ax, sizeof(S) == 4 ? FFT_BUDGET_X32 : FFT_BUDGET_X, FFT_THREADS));
    const int Bx = 1 << lbx;
    const int gx = (nrows + 2 * Bx - 1) / (2 * Bx);
    constexpr size_t RSB = sizeof(double) * (RED_THREADS / 64);  // of a pending rescaling
    const size_t ldsx = sizeof(C) * ((size_t)Bx * (p.nx + 1) + p.nx) + RSB;
    constexpr int KN = 16 / sizeof(C);
    const Div dk = make_div(p.nkx), dk2 = make_div((p.nkx + 1) / 2), dkn = make_div((p.nkx + KN - 1) / KN);
    // the variant of an x pass: scaled or not, rows of 4 m or 4 m + 2 values
    auto with_rows = [&](auto &&f) {
        auto wide = [&](auto sc) {
            if (p.nx % 4 == 0) f(sc, std::integral_constant<int, 4>{});
            else f(sc, std::integral_constant<int, 2>{});
        };
        if (sinv) wide(std::true_type{});
        else wide(std::false_type{});
    };
    const int lby = tile_log2(p.ny, budget(ay, FFT_BUDGET_Y, FFT_THREADS)), By = 1 << lby;
    const int gy = xcd_grid((p.nkx + By - 1) / By * p.nz);
    const size_t ldsy = sizeof(C) * ((size_t)By * p.ny + p.ny);
    auto y_pass = [&](auto inv) {
        constexpr bool INV = decltype(inv)::value;
        with6(has6(ay), [&](auto r6) {
            constexpr bool R6 = decltype(r6)::value;
            static std::atomic<unsigned> attr{0};
            lds_attr(fptr(&k_fft_y<S, R6, INV>), attr, ldsy);
            k_fft_y<S, R6, INV><<<gy, FFT_THREADS, ldsy, st>>>(cbuf, RD(ay), TW(ay), lby, p.nkx, p.ldc, p.nz);
            DWP_LAUNCH_CHECK();
        });
    };
    // both passes of a plane in one block
    const int pv = std::max(p.ny / 2 * (p.nx + 1), p.ny * p.nkx);
    const size_t ldsp = sizeof(C) * ((size_t)pv + p.nx + p.ny) + RSB;
    const bool plane = plane_pass(pv, ldsp, p.nz);
    const Div dl = make_div(p.ny / 2), dw2 = make_div(p.nx / 2);
    auto with_plane = [&](auto &&f) {
        auto size = [&](auto sc) {
            using std::integral_constant;
            if (pv <= PLANE_SMALL) f(sc, integral_constant<int, 512>{}, integral_constant<int, 6>{});
            else if (pv <= PLANE_MID) f(sc, integral_constant<int, 1024>{}, integral_constant<int, 6>{});
            else f(sc, integral_constant<int, 1024>{}, integral_constant<int, 10>{});
        };
        if (sinv) size(std::true_type{});
        else size(std::false_type{});
    };
    ev = pb(PG_FFT_X);
    if (plane) with_plane([&](auto sc, auto nt, auto pe_) {
        constexpr bool SC = decltype(sc)::value;
        constexpr int NT = decltype(nt)::value, PE = decltype(pe_)::value;
        static std::atomic<unsigned> attr{0};
        lds_attr(fptr(&k_fft_xy_fwd<S, TI, SC, NT, PE>), attr, ldsp);
        k_fft_xy_fwd<S, TI, SC, NT, PE><<<p.nz, NT, ldsp, st>>>(r, sinv, cbuf, RD(ax), RD(ay), TW(ax), TW(ay), p.ldc, dl,
                                                            dw2, dk, rs);
        DWP_LAUNCH_CHECK();
    });
    else with6(has6(ax), [&](auto r6) {
        with_rows([&](auto sc, auto w) {
            constexpr bool R6 = decltype(r6)::value, SC = decltype(sc)::value;
            constexpr int W = decltype(w)::value;
            static std::atomic<unsigned> attr{0};
            lds_attr(fptr(&k_fft_x_fwd<S, TI, R6, SC, W>), attr, ldsx);
            k_fft_x_fwd<S, TI, R6, SC, W><<<gx, FFT_THREADS, ldsx, st>>>(r, sinv, cbuf, RD(ax), TW(ax), lbx, nrows,
                                                                        p.nkx, p.ldc, make_div(p.nx / W), dk, dk2, rs);
            DWP_LAUNCH_CHECK();
        });
    });
    pe(ev, PG_FFT_X, bx);
    if (!plane) {
        ev = pb(PG_FFT_Y);
        y_pass(std::false_type{});
        pe(ev, PG_FFT_Y, 2.0 * cb * Cn);
    }
    // z pass with the Green's function (lines of 8 kx; the twiddles follow
    // the lines in LDS)
    ev = pb(PG_FFT_Z);
    with6(has6(az), [&](auto r6) {
        constexpr bool R6 = decltype(r6)::value;
        const int lbz = tile_log2(p.nz, budget(az, FFT_Z_MAXE, FFT_Z_THREADS)), Bz = 1 << lbz;
        const int gz = xcd_grid((p.nkx + Bz - 1) / Bz * p.ny);
        // the symbol staged in LDS too where it fits
        const size_t base_bytes = sizeof(C) * ((size_t)Bz * p.nz + p.nz);
        const size_t lam_bytes = sizeof(S) * ((size_t)p.nz + Bz);
        const int lam_lds = base_bytes + lam_bytes <= 160 * 1024 ? 1 : 0;
        const size_t bytes = base_bytes + (lam_lds ? lam_bytes : 0);
        static std::atomic<unsigned> attr{0};
        lds_attr(fptr(&k_fft_z_green<S, R6, FFT_Z_MAXE, FFT_Z_THREADS>), attr, bytes);
        k_fft_z_green<S, R6, FFT_Z_MAXE, FFT_Z_THREADS><<<gz, FFT_Z_THREADS, bytes, st>>>(
            cbuf, RD(az), TW(az), lbz, p.nkx, p.ldc, p.ny, LAM(ax), LAM(ay), LAM(az), (S)(1.0 / (double)p.N), lam_lds);
        DWP_LAUNCH_CHECK();
    });
    pe(ev, PG_FFT_Z, 2.0 * cb * Cn);
    if (!plane) {
        ev = pb(PG_FFT_Y);
        y_pass(std::true_type{});
        pe(ev, PG_FFT_Y, 2.0 * cb * Cn);
    }
    ev = pb(PG_FFT_X);
    if (plane) with_plane([&](auto sc, auto nt, auto pe_) {
        constexpr bool SC = decltype(sc)::value;
        constexpr int NT = decltype(nt)::value, PE = decltype(pe_)::value;
        static std::atomic<unsigned> attr{0};
        lds_attr(fptr(&k_fft_xy_inv<S, TO, SC, NT, PE>), attr, ldsp);
        k_fft_xy_inv<S, TO, SC, NT, PE><<<p.nz, NT, ldsp, st>>>(cbuf, sinv, out, RD(ax), RD(ay), TW(ax), TW(ay), p.ldc, dl,
                                                            dw2, dk);
        DWP_LAUNCH_CHECK();
    });
    else with6(has6(ax), [&](auto r6) {
        with_rows([&](auto sc, auto w) {
            constexpr bool R6 = decltype(r6)::value, SC = decltype(sc)::value;
            constexpr int W = decltype(w)::value;
            static std::atomic<unsigned> attr{0};
            lds_attr(fptr(&k_fft_x_inv<S, TO, R6, SC, W>), attr, ldsx);
            k_fft_x_inv<S, TO, R6, SC, W><<<gx, FFT_THREADS, ldsx, st>>>(cbuf, sinv, out, RD(ax), TW(ax), lbx, nrows,
                                                                        p.nkx, p.ldc, make_div(p.nx / W), dkn);
            DWP_LAUNCH_CHECK();
        });
    });
    pe(ev, PG_FFT_X, bxi);
}

void launch_vacuum_solve(hipStream_t st, const Plan &p, const FFTAxis &ax, const FFTAxis &ay, const FFTAxis &az,
                         double *r, const double *sinv, void *cbuf, double *out, Profiler *prof, bool fp32,
                         const Rescale &rs) {
    if (fp32) vacuum_solve_t<float, double, double>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, rs);
    else vacuum_solve_t<double, double, double>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, rs);
}
void launch_vacuum_solve(hipStream_t st, const Plan &p, const FFTAxis &ax, const FFTAxis &ay, const FFTAxis &az,
                         float *r, const double *sinv, void *cbuf, float *out, Profiler *prof, bool fp32,
                         const Rescale &rs) {
    if (fp32) vacuum_solve_t<float, float, float>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, rs);
    else vacuum_solve_t<double, float, float>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, rs);
}
void launch_vacuum_solve(hipStream_t st, const Plan &p, const FFTAxis &ax, const FFTAxis &ay, const FFTAxis &az,
                         const _Float16 *r, const double *sinv, void *cbuf, float *out, Profiler *prof, bool fp32) {
    if (fp32) vacuum_solve_t<float, const _Float16, float>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, Rescale{});
    else vacuum_solve_t<double, const _Float16, float>(st, p, ax, ay, az, r, sinv, cbuf, out, prof, Rescale{});
}

}  // namespace dwp
