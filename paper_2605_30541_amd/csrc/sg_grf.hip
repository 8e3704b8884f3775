// The random field of SaltSDT (SubsurfaceGen, arXiv 2605.30541, App. B,
// Alg. 4): white noise on a periodic grid of powers of two shaped in Fourier
// space by sqrt(P(k)), P(k) = (1 + sum_k (k_k l_k)^2)^-p, cropped to the
// volume and scaled to zero mean and unit variance.
//
// The noise is real, so only half of its spectrum along x is held: kx = 0 ..
// Px/2, rows of Q values.  Five passes over that half spectrum, in place:
//   1. x forward, real to complex (two real lines per complex line);
//   2. y forward (strided lines);
//   3. z forward, times the spectral factor, z inverse: one pass, the line
//      stays in registers in between; only the volume's nz planes are written;
//   4. y inverse on those planes; only ny rows are written;
//   5. x inverse, complex to real, straight into the cropped volume, with the
//      sums for its mean and variance;
// then the normalisation.  Neither direction is scaled (the normalisation
// removes every constant factor).
//
// Bound: memory, about 38 GB for the 1024^3 grid of a 619 x 1000 x 1000
// volume.  Measured there: 52.1 ms with full complex transforms written
// transposed (six passes of 16 GB in 32-byte pieces), 9.9 ms in this form.
#include "sg_internal.h"

#include <algorithm>
#include <type_traits>

namespace sg {

namespace {

// The spectral factor sqrt(P(k)); k in radians per cell in the FFT's frequency
// order (0, 1, .., P/2-1, -P/2, .., -1) / P.
struct Spectrum {
    int Pz, Py, Px;
    double lz, ly, lx, half_p;
};

// (k l)^2 of position i on an axis of n cells with correlation length l
__device__ inline double wavenumber2(int i, int n, double l)
{
    const double two_pi = 6.283185307179586;
    const double f = (i < (n + 1) / 2 ? i : i - n) / (double)n;
    const double k = two_pi * f * l;
    return k * k;
}

// q^-half_p for q >= 1: log2 q = e + log2 m with q = m 2^e, the
// product with half_p in FP64, of which only the fraction goes through the
// FP32 exponential.  (FP32 throughout, the rounding of log2 q ~ 14 alone
// moved the field by 1e-7 of its norm.)  q and half_p log2 q must be finite:
// spectrum() sees to it.
__device__ inline float spectral_amp(double q, double half_p)
{
    int e;
    const float m = (float)frexp(q, &e);   // in [1/2, 1)
    const double s = half_p * ((double)e + (double)log2f(m)), n = rint(s);
    return ldexpf(exp2f((float)(n - s)), -(int)fmin(n, 1000.0));
}

// Lengths and exponents so large that (k l)^2 or the power would leave FP64 are
// taken smaller: the factor is then at most (1e147)^-p on that axis.
// (Clamped in the kernel, per value, the z pass lost a wave per SIMD: 9.8 -> 11.1
// ms for a 619 x 1000 x 1000 field.)
Spectrum spectrum(const int P[3], double lz, double ly, double lx, double p)
{
    const double most = 1e150;
    return Spectrum{P[0], P[1], P[2], std::min(lz, most), std::min(ly, most), std::min(lx, most),
                    std::min(0.5 * p, 1e300)};
}

// Where the half spectrum lives: row (z, y) of Px/2 + 1 values starts at z *
// plane + y * Q.  Rows are whole 128-byte lines and the plane stride an odd
// number of them, so lines along y and z spread over the memory channels
// (small grids are stored densely: the workspace is two full complex grids).
struct HalfGrid {
    int Pz, Py, Px, nkx, Q;
    int64_t plane;
};

HalfGrid half_grid(const int P[3])
{
    HalfGrid G{P[0], P[1], P[2], P[2] / 2 + 1, P[2] / 2 + 1, 0};
    if (G.Px >= 64) {
        G.Q = (G.nkx + 15) / 16 * 16;
        G.plane = (int64_t)G.Py * G.Q + 16;
    } else {
        G.plane = (int64_t)G.Py * G.Q;
    }
    return G;
}

// Complex values of either width.
template <class F>
struct Cx {
    F x, y;
};
template <class F>
__device__ __forceinline__ Cx<F> operator+(Cx<F> a, Cx<F> b) { return {a.x + b.x, a.y + b.y}; }
template <class F>
__device__ __forceinline__ Cx<F> operator-(Cx<F> a, Cx<F> b) { return {a.x - b.x, a.y - b.y}; }
template <class F>
__device__ __forceinline__ Cx<F> operator*(Cx<F> a, Cx<F> w) { return {a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x}; }
__device__ __forceinline__ float2 cswap(float2 a) { return make_float2(a.y, a.x); }

// Forward DFTs of 1, 2, 4, 8 and 16 values in registers, results in order.
template <int R, class F>
__device__ __forceinline__ void dft(Cx<F> (&v)[R])
{
    if constexpr (R == 2) {
        const Cx<F> a = v[0], b = v[1];
        v[0] = a + b;
        v[1] = a - b;
    } else if constexpr (R == 4) {
        const Cx<F> t0 = v[0] + v[2], t1 = v[0] - v[2], t2 = v[1] + v[3], d = v[1] - v[3];
        const Cx<F> t3{d.y, -d.x};   // -i d
        v[0] = t0 + t2;
        v[1] = t1 + t3;
        v[2] = t0 - t2;
        v[3] = t1 - t3;
    } else if constexpr (R == 8) {
        const F h = (F)0.70710678118654752440;
        Cx<F> e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft<4>(e);
        dft<4>(o);
        o[1] = {h * (o[1].x + o[1].y), h * (o[1].y - o[1].x)};
        o[2] = {o[2].y, -o[2].x};
        o[3] = {h * (o[3].y - o[3].x), -h * (o[3].x + o[3].y)};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = e[k] + o[k];
            v[k + 4] = e[k] - o[k];
        }
    } else if constexpr (R == 16) {
        // cos and sin of 2 pi m / 16, m = 0 .. 9
        constexpr F c1 = (F)0.92387953251128674, s1 = (F)0.38268343236508977, h = (F)0.70710678118654752;
        constexpr F wc[10] = {1, c1, h, s1, 0, -s1, -h, -c1, -1, -c1};
        constexpr F ws[10] = {0, s1, h, c1, 1, c1, h, s1, 0, -s1};
        Cx<F> a[4][4];
#pragma unroll
        for (int n = 0; n < 4; ++n) {
#pragma unroll
            for (int m = 0; m < 4; ++m) a[n][m] = v[n + 4 * m];
            dft<4>(a[n]);
        }
#pragma unroll
        for (int n = 1; n < 4; ++n)
#pragma unroll
            for (int m = 1; m < 4; ++m) a[n][m] = a[n][m] * Cx<F>{wc[n * m], -ws[n * m]};
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            Cx<F> b[4] = {a[0][m], a[1][m], a[2][m], a[3][m]};
            dft<4>(b);
#pragma unroll
            for (int k = 0; k < 4; ++k) v[m + 4 * k] = b[k];
        }
    }
}

// A workgroup transforms kC lines of length L = 2^LOG together: Stockham
// passes of radix up to 16, each thread holding its butterflies' values in
// registers, LDS only to exchange them between passes.  X: the lines are
// contiguous in memory (lanes along the line), else neighbouring lines are
// neighbours in memory (kC lanes across the lines, 64-byte pieces; the two
// pieces of a 128-byte line go to neighbouring workgroups of one XCD).
// kC = 8 lines of 1024 take 70 KB of LDS, so two workgroups share a CU and one's
// loads and stores overlap the other's butterflies.
constexpr int kC = 8;

template <int LOG, bool X>
struct Lines {
    static constexpr int L = 1 << LOG, kWork = kC * L;
    static constexpr int NT = kWork / 16 < 64 ? 64 : (kWork / 16 > 512 ? 512 : kWork / 16);
    static constexpr int kPad = L + L / 16 + 1;      // a line in LDS (X), one pad value per 16
    static constexpr int kLds = X ? kC * kPad : kC * (L + L / 16);
    // radices of the passes (LOG = their sum of logarithms); the last first when REV
    static constexpr int kPasses = LOG <= 4 ? 1 : (LOG <= 7 ? 2 : 3);
    static constexpr int radix(int p, bool rev)
    {
        if (kPasses == 1) return L;
        const int q = rev ? kPasses - 1 - p : p;
        return q > 0 ? 8 : (kPasses == 2 ? L / 8 : L / 64);
    }
    // The pass (of radix 8) whose butterflies run in FP64; none in the z
    // inverse, whose pass is bound by the vector unit.  The complex transforms
    // of a whole real grid leave half of their rounding error in the imaginary
    // part, which is dropped; the half spectrum has no such part and, in FP32
    // throughout, was 1.07 times as far from the exact field (2.57e-7 against
    // 2.42e-7 at 619 x 1000 x 1000).  In this form it is 2.3e-7, for 0.4 ms.
    template <bool REV>
    static constexpr int kWide = kPasses == 1 || REV ? -1 : kPasses - 1;
    static constexpr int most(int r) { return (kWork / r + NT - 1) / NT * r; }
    static constexpr int E = most(radix(0, false)) > most(radix(kPasses - 1, false)) ? most(radix(0, false))
                                                                                  : most(radix(kPasses - 1, false));

    __device__ static __forceinline__ int at(int c, int pos)
    {
        return X ? c * kPad + pos + (pos >> 4) : (pos + (pos >> 4)) * kC + c;
    }
    // butterfly b of a pass of radix R takes values j + k L / R, k < R, of line c
    template <int R>
    __device__ static __forceinline__ bool butterfly(int i, int &c, int &j)
    {
        const int b = (int)threadIdx.x + i * NT;
        if (X) {
            c = b / (L / R);
            j = b % (L / R);
        } else {
            c = b % kC;
            j = b / kC;
        }
        return kWork / R % NT == 0 || b < kWork / R;
    }
    // f(value, line, position) over the values this thread holds in the layout of radix R
    template <int R, class F>
    __device__ static __forceinline__ void each(float2 (&v)[E], F f)
    {
#pragma unroll
        for (int i = 0; i < (kWork / R + NT - 1) / NT; ++i) {
            int c, j;
            if (!butterfly<R>(i, c, j)) continue;
#pragma unroll
            for (int k = 0; k < R; ++k) f(v[i * R + k], c, j + k * (L / R));
        }
    }
    __device__ static void twiddles(float2 *tw)
    {
        if (kPasses == 1) return;
        for (int m = threadIdx.x; m < L; m += NT) {
            float sn, cs;
            sincospif(-2.f * (float)m / (float)L, &sn, &cs);
            tw[m] = make_float2(cs, sn);
        }
    }
    // Forward transform of v (in the layout of the first pass's radix; the
    // result in that of the last).  Uses buf between passes; the caller
    // separates it from its own use of buf by a barrier.
    template <bool REV, int P = 0, int S = 1>
    __device__ static __forceinline__ void run(float2 (&v)[E], float2 *buf, const float2 *tw)
    {
        constexpr int R = radix(P, REV);
#pragma unroll
        for (int i = 0; i < (kWork / R + NT - 1) / NT; ++i) {
            int c, j;
            if (!butterfly<R>(i, c, j)) continue;
            using F = std::conditional_t<P == kWide<REV>, double, float>;
            Cx<F> u[R];
#pragma unroll
            for (int k = 0; k < R; ++k) u[k] = {(F)v[i * R + k].x, (F)v[i * R + k].y};
            if (S > 1) {
                const int m = (j % S) * (L / (S * R));
#pragma unroll
                for (int k = 1; k < R; ++k) {
                    const float2 w = tw[m * k];
                    u[k] = u[k] * Cx<F>{(F)w.x, (F)w.y};
                }
            }
            dft<R>(u);
#pragma unroll
            for (int k = 0; k < R; ++k) v[i * R + k] = make_float2((float)u[k].x, (float)u[k].y);
        }
        if constexpr (P + 1 < kPasses) {
            if (P > 0) __syncthreads();   // the reads of the exchange before
#pragma unroll
            for (int i = 0; i < (kWork / R + NT - 1) / NT; ++i) {
                int c, j;
                if (!butterfly<R>(i, c, j)) continue;
                const int o = (j / S) * (S * R) + j % S;
#pragma unroll
                for (int k = 0; k < R; ++k) buf[at(c, o + k * S)] = v[i * R + k];
            }
            __syncthreads();
            each<radix(P + 1, REV)>(v, [&](float2 &x, int c, int pos) { x = buf[at(c, pos)]; });
            run<REV, P + 1, S * R>(v, buf, tw);
        }
    }
    static constexpr int kFirst = radix(0, false), kLast = radix(kPasses - 1, false);
};

// Consecutive blocks of work go to one XCD (the hardware deals workgroups to
// the 8 XCDs in turn), so the halves of a memory line that neighbouring
// workgroups touch meet in one L2.
__device__ __forceinline__ unsigned xcd_order(unsigned bid, unsigned n)
{
    const unsigned per = n >> 3;
    return bid >= per * 8 ? bid : (bid & 7) * per + (bid >> 3);
}

// Pass 1: lines 2q and 2q+1 of the real noise as the real and imaginary part
// of complex line q; their half spectra from its spectrum C as
// (C(k) + conj C(-k)) and -i (C(k) - conj C(-k)) (twice the spectra).
template <int LOG>
__global__ void __launch_bounds__((Lines<LOG, true>::NT)) k_fft_x(const float *__restrict__ noise, HalfGrid G,
                                                                float2 *__restrict__ out)
{
    using T = Lines<LOG, true>;
    __shared__ float2 buf[T::kLds], tw[T::L];
    const int64_t q0 = (int64_t)xcd_order(blockIdx.x, gridDim.x) * kC, lines = (int64_t)G.Pz * G.Py;
    float2 v[T::E];
    T::template each<T::kFirst>(v, [&](float2 &x, int c, int pos) {
        const int64_t l = 2 * (q0 + c);
        x.x = l < lines ? __builtin_nontemporal_load(noise + l * T::L + pos) : 0.f;
        x.y = l + 1 < lines ? __builtin_nontemporal_load(noise + (l + 1) * T::L + pos) : 0.f;
    });
    T::twiddles(tw);
    __syncthreads();
    T::template run<false>(v, buf, tw);
    __syncthreads();
    T::template each<T::kLast>(v, [&](float2 &x, int c, int pos) { buf[T::at(c, pos)] = x; });
    __syncthreads();
    constexpr int H = T::L / 2 + 1;
    for (int i = threadIdx.x; i < kC * H; i += T::NT) {
        const int c = i / H, k = i % H;
        const int64_t l = 2 * (q0 + c);
        if (l >= lines) break;
        const float2 a = buf[T::at(c, k)], b = buf[T::at(c, (T::L - k) & (T::L - 1))];
        out[l / G.Py * G.plane + l % G.Py * G.Q + k] = make_float2(a.x + b.x, a.y - b.y);
        if (l + 1 < lines)
            out[(l + 1) / G.Py * G.plane + (l + 1) % G.Py * G.Q + k] = make_float2(a.y + b.y, b.x - a.x);
    }
}

// Passes 2 and 4: the lines along y of every plane, in place; rows below
// `keep` are written.
template <int LOG, bool INV>
__global__ void __launch_bounds__((Lines<LOG, false>::NT)) k_fft_y(float2 *__restrict__ a, HalfGrid G, int keep)
{
    using T = Lines<LOG, false>;
    __shared__ float2 buf[T::kLds], tw[T::L];
    const unsigned blk = xcd_order(blockIdx.x, gridDim.x), nt = (unsigned)((G.nkx + kC - 1) / kC);
    const int x0 = (int)(blk % nt) * kC, cols = min(kC, G.nkx - x0);
    float2 *p = a + (int64_t)(blk / nt) * G.plane + x0;
    float2 v[T::E];
    T::template each<T::kFirst>(v, [&](float2 &x, int c, int pos) {
        x = c < cols ? p[(int64_t)pos * G.Q + c] : make_float2(0.f, 0.f);
        if (INV) x = cswap(x);
    });
    T::twiddles(tw);
    __syncthreads();
    T::template run<false>(v, buf, tw);
    T::template each<T::kLast>(v, [&](float2 &x, int c, int pos) {
        if (c < cols && pos < keep) p[(int64_t)pos * G.Q + c] = INV ? cswap(x) : x;
    });
}

// Pass 3: the lines along z, forward, times the spectral factor, inverse (the
// radices in reverse order, so the forward result is already laid out for the
// inverse's first pass), in place; planes below `keep` are written.
template <int LOG>
__global__ void __launch_bounds__((Lines<LOG, false>::NT)) k_fft_z(float2 *__restrict__ a, HalfGrid G, Spectrum S,
                                                                 int keep)
{
    using T = Lines<LOG, false>;
    __shared__ float2 buf[T::kLds], tw[T::L];
    const unsigned blk = xcd_order(blockIdx.x, gridDim.x), nt = (unsigned)((G.nkx + kC - 1) / kC);
    const int x0 = (int)(blk % nt) * kC, cols = min(kC, G.nkx - x0), y = (int)(blk / nt);
    float2 *p = a + (int64_t)y * G.Q + x0;
    float2 v[T::E];
    T::template each<T::kFirst>(v, [&](float2 &x, int c, int pos) {
        x = c < cols ? p[(int64_t)pos * G.plane + c] : make_float2(0.f, 0.f);
    });
    T::twiddles(tw);
    __syncthreads();
    T::template run<false>(v, buf, tw);
    const double kyx = 1.0 + wavenumber2(y, S.Py, S.ly) + wavenumber2(x0 + (int)threadIdx.x % kC, S.Px, S.lx);
    T::template each<T::kLast>(v, [&](float2 &x, int, int pos) {
        const float amp = spectral_amp(kyx + wavenumber2(pos, S.Pz, S.lz), S.half_p);
        x = make_float2(x.y * amp, x.x * amp);   // swapped: the inverse transform is a forward one of swapped values
    });
    __syncthreads();
    T::template run<true>(v, buf, tw);
    T::template each<T::kFirst>(v, [&](float2 &x, int c, int pos) {
        if (c < cols && pos < keep) p[(int64_t)pos * G.plane + c] = cswap(x);
    });
}

// Pass 5: rows 2q and 2q+1 of a plane (A and B) as one complex line A + i B,
// whose inverse transform has the two real lines as real and imaginary part;
// per-workgroup FP64 sums of v and v^2.
template <int LOG>
__global__ void __launch_bounds__((Lines<LOG, true>::NT)) k_ifft_x(const float2 *__restrict__ a, HalfGrid G, int nz,
                                                                 int ny, int nx, float *__restrict__ out,
                                                                 double *__restrict__ partials)
{
    using T = Lines<LOG, true>;
    __shared__ float2 buf[T::kLds], tw[T::L];
    const int64_t ppz = (ny + 1) / 2, q0 = (int64_t)xcd_order(blockIdx.x, gridDim.x) * kC, npair = ppz * nz;
    constexpr int H = T::L / 2 + 1;
    for (int i = threadIdx.x; i < kC * H; i += T::NT) {
        const int c = i / H, k = i % H;
        const int64_t q = q0 + c;
        float2 A = make_float2(0.f, 0.f), B = A;
        if (q < npair) {
            const int64_t z = q / ppz;
            const int y = 2 * (int)(q % ppz);
            const float2 *r = a + z * G.plane + (int64_t)y * G.Q + k;
            A = r[0];
            if (y + 1 < ny) B = r[G.Q];
        }
        // (stored swapped, for the inverse)
        if (k == 0 || 2 * k == T::L) {
            buf[T::at(c, k)] = make_float2(B.x, A.x);   // real there
        } else {
            buf[T::at(c, k)] = make_float2(A.y + B.x, A.x - B.y);
            buf[T::at(c, T::L - k)] = make_float2(B.x - A.y, A.x + B.y);
        }
    }
    T::twiddles(tw);
    __syncthreads();
    float2 v[T::E];
    T::template each<T::kFirst>(v, [&](float2 &x, int c, int pos) { x = buf[T::at(c, pos)]; });
    __syncthreads();
    T::template run<false>(v, buf, tw);
    double s1 = 0.0, s2 = 0.0;
    T::template each<T::kLast>(v, [&](float2 &x, int c, int pos) {
        const int64_t q = q0 + c;
        if (q >= npair || pos >= nx) return;
        const int64_t z = q / ppz;
        const int y = 2 * (int)(q % ppz);
        float *o = out + (z * ny + y) * nx + pos;
        o[0] = x.y;
        s1 += x.y;
        s2 += (double)x.y * x.y;
        if (y + 1 < ny) {
            o[nx] = x.x;
            s1 += x.x;
            s2 += (double)x.x * x.x;
        }
    });
    for (int o = 32; o > 0; o >>= 1) {
        s1 += __shfl_xor(s1, o);
        s2 += __shfl_xor(s2, o);
    }
    __shared__ double r1[T::NT / 64], r2[T::NT / 64];
    if ((threadIdx.x & 63) == 0) {
        r1[threadIdx.x >> 6] = s1;
        r2[threadIdx.x >> 6] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < T::NT / 64; ++w) {
            s1 += r1[w];
            s2 += r2[w];
        }
        partials[2 * (int64_t)blockIdx.x] = s1;
        partials[2 * (int64_t)blockIdx.x + 1] = s2;
    }
}

// One workgroup: mean and 1/std from the partial sums, in a fixed order (four
// pairs in flight per thread).
__global__ void __launch_bounds__(1024) k_grf_stats(const double2 *partials, int64_t nblocks, int64_t n, double *stats)
{
    __shared__ double r1[16], r2[16];
    double s1 = 0.0, s2 = 0.0;
    for (int64_t b = threadIdx.x; b < nblocks; b += 4096) {
        double2 p[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) p[u] = b + 1024 * u < nblocks ? partials[b + 1024 * u] : make_double2(0.0, 0.0);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            s1 += p[u].x;
            s2 += p[u].y;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        s1 += __shfl_xor(s1, o);
        s2 += __shfl_xor(s2, o);
    }
    if ((threadIdx.x & 63) == 0) {
        r1[threadIdx.x >> 6] = s1;
        r2[threadIdx.x >> 6] = s2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) {
            s1 += r1[w];
            s2 += r2[w];
        }
        const double mean = s1 / (double)n;
        const double var = s2 / (double)n - mean * mean;
        stats[0] = mean;
        stats[1] = var > 0.0 ? 1.0 / sqrt(var) : 0.0;
    }
}

__global__ void __launch_bounds__(256) k_grf_normalize(float *out, int64_t n, const double *stats)
{
    const double mean = stats[0], inv = stats[1];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = (float)(((double)out[i] - mean) * inv);
}

int log2i(int v)
{
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
}

unsigned grid1d(int64_t n)
{
    int64_t b = (n + 255) / 256;
    return (unsigned)(b > 65536 ? 65536 : (b < 1 ? 1 : b));
}

constexpr int kStatBlocks = 2048;   // (room for as many pairs of sums is part of the workspace)

// Calls f(std::integral_constant<int, log>) for log = 0 .. 10.
template <class F>
hipError_t with_log(int log, F f)
{
    switch (log) {
    case 0: f(std::integral_constant<int, 0>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    case 3: f(std::integral_constant<int, 3>{}); break;
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

void grf_grid(int nz, int ny, int nx, int P[3])
{
    const int n[3] = {nz, ny, nx};
    for (int k = 0; k < 3; ++k) P[k] = 1 << log2i(n[k]);
}

size_t grf_workspace_bytes(int nz, int ny, int nx)
{
    int P[3];
    grf_grid(nz, ny, nx, P);
    const size_t n = (size_t)P[0] * P[1] * P[2];
    return 2 * n * sizeof(float2) + (size_t)kStatBlocks * 2 * sizeof(double) + 256;
}

hipError_t launch_grf(const float *noise, int nz, int ny, int nx, double lz, double ly, double lx, double p, float *out,
                      void *ws, hipStream_t st)
{
    int P[3];
    grf_grid(nz, ny, nx, P);
    const HalfGrid G = half_grid(P);
    const Spectrum S = spectrum(P, lz, ly, lx, p);
    // the half spectrum, the result's statistics and the sums per workgroup of pass 5
    float2 *a = (float2 *)ws;
    const int64_t npair = (int64_t)nz * ((ny + 1) / 2), blocks = (npair + kC - 1) / kC;
    double *stats = (double *)(a + (G.plane * G.Pz + 31) / 32 * 32), *partials = stats + 2;
    if ((char *)(partials + 2 * blocks) > (char *)ws + grf_workspace_bytes(nz, ny, nx)) return hipErrorInvalidValue;
    const unsigned tiles = (unsigned)((G.nkx + kC - 1) / kC);
    hipError_t e = with_log(log2i(P[2]), [&](auto lg) {
        constexpr int LOG = decltype(lg)::value;
        const int64_t pairs = ((int64_t)G.Pz * G.Py + 1) / 2;
        hipLaunchKernelGGL(k_fft_x<LOG>, dim3((unsigned)((pairs + kC - 1) / kC)), dim3((Lines<LOG, true>::NT)), 0, st,
                           noise, G, a);
    });
    if (e != hipSuccess) return e;
    if (G.Py > 1) {
        e = with_log(log2i(P[1]), [&](auto lg) {
            constexpr int LOG = decltype(lg)::value;
            hipLaunchKernelGGL((k_fft_y<LOG, false>), dim3(tiles * G.Pz), dim3((Lines<LOG, false>::NT)), 0, st, a, G,
                               G.Py);
        });
        if (e != hipSuccess) return e;
    }
    e = with_log(log2i(P[0]), [&](auto lg) {
        constexpr int LOG = decltype(lg)::value;
        hipLaunchKernelGGL(k_fft_z<LOG>, dim3(tiles * G.Py), dim3((Lines<LOG, false>::NT)), 0, st, a, G, S, nz);
    });
    if (e != hipSuccess) return e;
    if (G.Py > 1) {
        e = with_log(log2i(P[1]), [&](auto lg) {
            constexpr int LOG = decltype(lg)::value;
            hipLaunchKernelGGL((k_fft_y<LOG, true>), dim3(tiles * nz), dim3((Lines<LOG, false>::NT)), 0, st, a, G, ny);
        });
        if (e != hipSuccess) return e;
    }
    e = with_log(log2i(P[2]), [&](auto lg) {
        constexpr int LOG = decltype(lg)::value;
        hipLaunchKernelGGL(k_ifft_x<LOG>, dim3((unsigned)blocks), dim3((Lines<LOG, true>::NT)), 0, st, a, G, nz, ny, nx,
                           out, partials);
    });
    if (e != hipSuccess) return e;
    const int64_t m = (int64_t)nz * ny * nx;
    hipLaunchKernelGGL(k_grf_stats, dim3(1), dim3(1024), 0, st, (const double2 *)partials, blocks, m, stats);
    hipLaunchKernelGGL(k_grf_normalize, dim3(grid1d(m)), dim3(256), 0, st, out, m, stats);
    return hipGetLastError();
}

}  // namespace sg
