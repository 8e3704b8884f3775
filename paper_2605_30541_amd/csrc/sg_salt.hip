// SaltSDT (SubsurfaceGen, arXiv 2605.30541, App. B, Alg. 4): salt bodies from
// rotated ellipsoids whose signed distance is perturbed by a random field,
// merged, opened and closed, cleared of small components and written over
// the model below the water.  Volumes are [nz][ny][nx], x fastest.
//
// Sets of voxels are kept as bits, a 64-bit word per 64 voxels of a row (word
// x / 64 of row z ny + y; bits past the row's end are 0): one wave's ballot.
//
// Kernels, in launch order:
//  * k_field_extremes: max(xi, 0) and max(-xi, 0) of every body's field,
//    read back once so the host can bound each body's reach (below);
//  * k_raster: the ellipsoid's voxel centres, as bits over the body's box;
//  * k_dist_x, k_dist_z, k_dist_y: the exact squared Euclidean distances to the
//    nearest voxel outside and the nearest one inside, as three separable
//    passes: the 1D distance along x from the bits, then along z and y the
//    least of (w k)^2 + f(k cells away).  The search goes outward and ends
//    where (w k)^2 alone exceeds the least so far, which is exact (the paper
//    names Meijster's algorithm, which yields the same distances) -- or where
//    the decision it is for is made: phi' = d_in - d_out + a rbar xi > 0
//    needs d_out only where a rbar xi > 0 and only up to that, d_in only where
//    a rbar xi < 0 and only up to its negative (k_field_bounds: the extremes of
//    xi over the rows y, for the pass along z).  k_dist_y sets K.  Where a body
//    reaches far, k_envelope_z takes k_dist_z's place: the same distances from
//    the lower envelope of the parabolas, linear in a line's length.  A body
//    covering no voxel gives d_out = infinity everywhere (phi' = -inf), one
//    covering all gives d_in = infinity (phi' = +inf): no special cases;
//  * k_morph x4: opening then closing with the 6-neighbour cross, a voxel
//    outside the volume counting as empty;
//  * k_cc_init, k_cc_merge, k_cc_count: 6-connected components by a
//    lock-free union-find (runs along x inside a word are labelled from the
//    word; the rest is joined by atomicMin on the roots; then every label is
//    pointed at its root and counted), so each component ends labelled by its
//    smallest voxel index;
//  * k_salt_write: the final write.
//
// Each body is processed on boxes only.  d_out and phi' on the raster's
// bounding box widened by B = max over the volume of (a rbar xi) plus two
// voxels: outside it every voxel is outside the body and more than B from it,
// so phi' < 0 and the body adds nothing there, and inside it d_out is exact
// (every inside voxel is in the box).  d_in on the raster's bounding box plus
// two voxels: it is needed only at inside voxels (it is 0 at outside ones),
// and the nearest outside voxel of an inside voxel, clamped into that box, is
// still outside and no farther.  Decisions (inside the ellipsoid, phi' > 0)
// are taken in FP64 without fused multiply-adds, so they round as the plain
// definitions do.
//
// Bound: the distance passes by FP64 issue (about 12 operations per voxel and
// cell of distance), the rest by memory (the fields read once for their
// extremes, the model read and written).  Measured for three bodies in 619 x
// 1000 x 1000 voxels: 28.7 ms with lower envelopes of parabolas (one thread
// and a stack in memory per line), sets as bytes and a label for every
// voxel; 8.6 ms in this form.
#include "sg_internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#pragma clang fp contract(off)

namespace sg {

namespace {

constexpr int kSaltThreads = 256;
constexpr int kWaves = kSaltThreads / 64;

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kSaltThreads - 1) / kSaltThreads); }

__device__ inline double inf_d() { return __builtin_huge_val(); }

// Voxels [z0, z0 + bz) x [y0, y0 + by) x [x0, x0 + bx) of the volume.
struct Box {
    int z0, y0, x0, bz, by, bx;
};

// Words of a row that hold voxels of the box: x0 / 64 .. (x0 + bx - 1) / 64.
__host__ __device__ inline int box_words(const Box &b) { return (b.x0 + b.bx - 1) / 64 - b.x0 / 64 + 1; }

__host__ __device__ inline int row_words(int nx) { return (nx + 63) / 64; }

// Index of this wave in the launch (uniform over the wave).
__device__ inline int64_t wave_index()
{
    return (int64_t)blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}
inline unsigned wave_blocks(int64_t waves) { return (unsigned)((waves + kWaves - 1) / kWaves); }

__device__ inline float wave_max(float v)
{
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    return v;
}

// ext[2 b] = max(xi_b, 0), ext[2 b + 1] = max(-xi_b, 0) as float bits (a
// non-negative float orders as its bits); NaN values are ignored.  ext must
// start at zero.  Body b = blockIdx.y.
__global__ void __launch_bounds__(kSaltThreads) k_field_extremes(int64_t n, const float *grf, unsigned *ext)
{
    const float *xi = grf + (int64_t)blockIdx.y * n;
    float hi = 0.0f, lo = 0.0f;
    const int64_t stride = (int64_t)gridDim.x * kSaltThreads;
    int64_t q = (int64_t)blockIdx.x * kSaltThreads + threadIdx.x;
    if (n % 4 == 0 && ((uintptr_t)grf & 15) == 0) {   // every field 16-byte aligned: four values per load
        const float4 *x4 = (const float4 *)xi;
        for (; q < n / 4; q += stride) {
            const float4 v = x4[q];
            hi = fmaxf(hi, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
            lo = fmaxf(lo, fmaxf(fmaxf(-v.x, -v.y), fmaxf(-v.z, -v.w)));
        }
    } else {
        for (; q < n; q += stride) {
            const float v = xi[q];
            hi = fmaxf(hi, v);
            lo = fmaxf(lo, -v);
        }
    }
    hi = wave_max(hi);
    lo = wave_max(lo);
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&ext[2 * blockIdx.y], __float_as_uint(hi));
        atomicMax(&ext[2 * blockIdx.y + 1], __float_as_uint(lo));
    }
}

// Raster of the ellipsoid over the box, one wave per word: bits[row of the
// box][word of the row], 0 outside the box.
__global__ void __launch_bounds__(kSaltThreads) k_raster(Box b, double dz, double dy, double dx, SaltBody B,
                                                         uint64_t *bits)
{
    const int nw = box_words(b);
    const int64_t w = wave_index();
    if (w >= (int64_t)b.bz * b.by * nw) return;
    const int64_t row = w / nw;
    const int iz = b.z0 + (int)(row / b.by), iy = b.y0 + (int)(row % b.by);
    const int ix = (b.x0 / 64 + (int)(w % nw)) * 64 + (int)(threadIdx.x & 63);
    const double p0 = iz * dz - B.c[0], p1 = iy * dy - B.c[1], p2 = ix * dx - B.c[2];
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double u = (B.R[3 * k] * p0 + B.R[3 * k + 1] * p1 + B.R[3 * k + 2] * p2) / B.r[k];
        s += u * u;
    }
    const uint64_t set = __ballot(s <= 1.0 && ix >= b.x0 && ix < b.x0 + b.bx);
    if ((threadIdx.x & 63) == 0) bits[w] = set;
}

// Along x, one wave per row (z, y) of box r: k[row][x - x0], x over [x0, x0 +
// bx), = cells to the nearest voxel of the row inside r that is a feature (set
// in `bits`, the raster over r, or not set when `outside`), -1 if the row has
// none; rows in [z][y], or with `by_y` in [y][z].  The words of r's part are
// walked upwards with the last feature before the word and the first one after
// it (a second index into the row).
__global__ void __launch_bounds__(kSaltThreads) k_dist_x(Box r, int x0, int bx, const uint64_t *__restrict__ bits,
                                                         int outside, bool by_y, int32_t *__restrict__ k)
{
    const int64_t row = wave_index();
    if (row >= (int64_t)r.bz * r.by) return;
    int32_t *kr = k + (by_y ? row % r.by * r.bz + row / r.by : row) * bx;
    const int lane = threadIdx.x & 63;
    const int w0 = r.x0 / 64, w1 = (r.x0 + r.bx - 1) / 64;
    const uint64_t *rw = bits + row * box_words(r) - w0;
    auto feature = [&](int w) -> uint64_t {   // of word w, inside r
        if (w < w0 || w > w1) return 0;
        uint64_t m = ~0ull;
        if (w == w0) m &= ~0ull << (r.x0 & 63);
        if (w == w1 && ((r.x0 + r.bx) & 63)) m &= ~(~0ull << ((r.x0 + r.bx) & 63));
        return (outside ? ~rw[w] : rw[w]) & m;
    };
    const uint64_t upto = ~0ull >> (63 - lane), from = ~0ull << lane;   // bits 0..lane, lane..63
    int last = -1, ahead = x0 / 64;
    uint64_t fa = feature(ahead);
    for (int w = x0 / 64; w <= (x0 + bx - 1) / 64; ++w) {
        const uint64_t f = feature(w);
        while (ahead <= w || fa == 0) {   // the first word past w that has a feature
            if (++ahead > w1) break;
            fa = feature(ahead);
        }
        const int next = ahead <= w1 ? ahead * 64 + __ffsll((unsigned long long)fa) - 1 : -1;
        const int x = w * 64 + lane;
        const uint64_t below = f & upto, above = f & from;
        const int l = below ? w * 64 + 63 - __clzll((long long)below) : last;
        const int n = above ? w * 64 + __ffsll((unsigned long long)above) - 1 : next;
        int d = -1;
        if (l >= 0) d = x - l;
        if (n >= 0 && (d < 0 || n - x < d)) d = n - x;
        if (x >= x0 && x < x0 + bx) kr[x - x0] = d;
        if (f) last = w * 64 + 63 - __clzll((long long)f);
    }
}

// Least and largest xi of every (z, x) of the box over its rows y (NaN ignored).
__global__ void __launch_bounds__(kSaltThreads) k_field_bounds(Box b, int ny, int nx, const float *__restrict__ xi,
                                                               float2 *__restrict__ lohi)
{
    const int nw = (b.bx + 63) / 64;
    const int64_t w = wave_index();
    if (w >= (int64_t)nw * b.bz) return;
    const int lx = (int)(w % nw) * 64 + (int)(threadIdx.x & 63), lz = (int)(w / nw);
    if (lx >= b.bx) return;
    const float *x = xi + ((int64_t)(b.z0 + lz) * ny + b.y0) * nx + b.x0 + lx;
    float lo = INFINITY, hi = -INFINITY;
    constexpr int kFlight = 8;
    for (int y = 0; y < b.by; y += kFlight) {
        float v[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) v[u] = x[(int64_t)min(y + u, b.by - 1) * nx];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            lo = fminf(lo, v[u]);
            hi = fmaxf(hi, v[u]);
        }
    }
    lohi[(int64_t)lz * b.bx + lx] = make_float2(lo, hi);
}

// best[i] <- min over k >= k0 of f(i - k) + (w k)^2, f(i + k) + (w k)^2 and
// itself, i = 0 .. N-1, for f >= 0: outward in steps of four cells, until for
// every i (w k)^2 exceeds best[i] or lim[i], or best[i] is no more than
// lim[i] * enough (or the line ends, kmax cells away).  A result above lim[i]
// is only known to be above it; one up to lim[i] * enough is an upper bound.
// N neighbouring outputs share their samples: L and H hold those below and
// above that the four steps need, so a step loads one value of each for N
// outputs.
template <int N, class F>
__device__ __forceinline__ void search(double (&best)[N], const double (&lim)[N], double enough, double w, int k0,
                                       int kmax, F f)
{
    auto open = [&](int k) {   // a step k can still matter
        const double d = w * (double)k;
        double far = -1.0;
#pragma unroll
        for (int i = 0; i < N; ++i) far = fmax(far, best[i] <= lim[i] * enough ? -1.0 : fmin(best[i], lim[i]));
        return k <= kmax && d * d < far;
    };
    if (!open(k0)) return;
    double L[N + 3], H[N + 3];   // f(i - k0 - 3 + ..), f(i + k0 + ..)
#pragma unroll
    for (int j = 0; j < N + 3; ++j) {
        L[j] = f(j - k0 - 3);
        H[j] = f(j + k0);
    }
    for (;; k0 += 4) {
        double nl[4], nh[4];   // the next steps' new samples, in flight meanwhile
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            nl[j] = f(j - k0 - 7);
            nh[j] = f(k0 + N + 3 + j);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const double d = w * (double)(k0 + s), kk = d * d;
#pragma unroll
            for (int i = 0; i < N; ++i) best[i] = fmin(best[i], fmin(L[i - s + 3], H[i + s]) + kk);
        }
        if (!open(k0 + 4)) return;
#pragma unroll
        for (int j = N + 2; j >= 4; --j) L[j] = L[j - 4];
#pragma unroll
        for (int j = 0; j < 4; ++j) L[j] = nl[j];
#pragma unroll
        for (int j = 0; j < N - 1; ++j) H[j] = H[j + 4];
#pragma unroll
        for (int j = 0; j < 4; ++j) H[N - 1 + j] = nh[j];
    }
}

// The rows of the volume that an ellipsoid can reach at depth rows of one y:
// z = c + slope (y - cy) +- (sqrt(hz2 (1 - (y - cy)^2 / cyy)) + extra) in metres
// (the projection of the ellipsoid onto z and y), widened by two cells.
struct ZSpan {
    double c, cy, slope, hz2, cyy, extra;
};

// Along z, in [z][y][x]: g = min over z' of (dz (z - z'))^2 + (dx k)^2 with k
// the x distance (infinite where -1) over the rows of box r; g over r's rows y,
// and the planes and columns of box b, which k's rows cover too.  Only values
// up to the largest a rbar xi (of -a rbar xi, when `inner`) of the (z, x) are
// needed.  The features of a body's inside lie in the span of its y: the
// search starts there.  A wave takes kOutZ planes of 64 columns.
constexpr int kOutZ = 8, kOutY = 4;
__global__ void __launch_bounds__(kSaltThreads) k_dist_z(Box r, Box b, double dz, double dy, double dx, ZSpan S,
                                                         int inner, double a_rbar, Box fb,
                                                         const float2 *__restrict__ lohi,
                                                         const int32_t *__restrict__ k, double *__restrict__ g)
{
    const int nw = (b.bx + 63) / 64, nb = (b.bz + kOutZ - 1) / kOutZ;
    const int64_t w = wave_index();
    if (w >= (int64_t)nw * r.by * nb) return;
    const int lx = (int)(w % nw) * 64 + (int)(threadIdx.x & 63);
    const int64_t rest = w / nw;
    const int ly = (int)(rest % r.by), z0 = b.z0 + (int)(rest / r.by) * kOutZ;   // (z0 in the volume)
    if (lx >= b.bx) return;
    // planes that can hold features of this y
    int zlo = r.z0, zhi = r.z0 + r.bz - 1;
    if (!inner) {
        const double d = (r.y0 + ly) * dy - S.cy, c = S.c + S.slope * d;
        const double h = sqrt(S.hz2 * fmax(1.0 - d * d / S.cyy, 0.0)) + S.extra + 2.0 * dz;
        const double lo = floor((c - h) / dz), hi = ceil((c + h) / dz);
        if (lo > zlo) zlo = lo < zhi ? (int)lo : zhi;
        if (hi < zhi) zhi = hi > zlo ? (int)hi : zlo;
    }
    const int64_t stride = (int64_t)r.by * b.bx, at = (int64_t)ly * b.bx + lx;
    auto f = [&](int i) {
        const int z = z0 + i;   // (loaded from a clamped place, so that no load waits for a branch)
        const int32_t c = k[at + (min(max(z, zlo), zhi) - r.z0) * stride];
        const double d = dx * (double)c;
        return c < 0 || z < zlo || z > zhi ? inf_d() : d * d;
    };
    constexpr int kOut = kOutZ;
    double best[kOut], lim[kOut];
    const int zend = b.z0 + b.bz;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const float2 lh = lohi[(int64_t)(min(z0 + i, zend - 1) - fb.z0) * fb.bx + (b.x0 + lx - fb.x0)];
        const double t0 = a_rbar * (double)lh.x, t1 = a_rbar * (double)lh.y;
        const double cap = fmax(inner ? fmax(-t0, -t1) : fmax(t0, t1), 0.0);
        best[i] = f(i);
        lim[i] = z0 + i < zend ? cap * cap * (1.0 + 1e-9) : -1.0;   // (infinite: nothing is cut off)
    }
    const int k0 = z0 + kOut - 1 < zlo ? zlo - (z0 + kOut - 1) : (z0 > zhi ? z0 - zhi : 1);
    search(best, lim, 0.0, dz, k0, max(zhi - z0, z0 + kOut - 1 - zlo), f);
#pragma unroll
    for (int i = 0; i < kOut; ++i)
        if (z0 + i < zend) g[at + (z0 + i - b.z0) * stride] = best[i];
}

// Along y, and the union.  gin (over box r, the raster's) and gout (over the
// rows y of r, the planes and columns of b) hold the distances over z and x.
// An outside voxel is salt where d_out < t = a rbar xi, an inside one where
// d_in > -t: the search ends as soon as that is decided, and is not begun where
// the sign of t decides it.  A wave takes kOutY rows of a word of K and sets its
// bits (no other wave of the launch has that word).
__global__ void __launch_bounds__(kSaltThreads) k_dist_y(Box r, Box b, int ny, int nx, double dy,
                                                         const uint64_t *__restrict__ raster,
                                                         const double *__restrict__ gin,
                                                         const double *__restrict__ gout,
                                                         const float *__restrict__ xi, double a_rbar, uint64_t *K)
{
    constexpr int kOut = kOutY;
    const int nw = box_words(b), nb = (b.by + kOut - 1) / kOut;
    const int64_t w = wave_index();
    if (w >= (int64_t)nw * b.bz * nb) return;
    const int word = b.x0 / 64 + (int)(w % nw), lane = threadIdx.x & 63, ix = word * 64 + lane;
    const int64_t rest = w / nw;
    const int y0 = b.y0 + (int)(rest % nb) * kOut, lz = (int)(rest / nb), yend = b.y0 + b.by;   // (y0 in the volume)
    const int iz = b.z0 + lz;
    // inside voxels of the rows (the raster's box may miss the plane, a row or the word)
    uint64_t inside[kOut];
    const int rw = word - r.x0 / 64;
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int y = y0 + i - r.y0, z = iz - r.z0;
        const bool hit = z >= 0 && z < r.bz && y >= 0 && y < r.by && rw >= 0 && rw < box_words(r);
        inside[i] = hit ? raster[((int64_t)z * r.by + y) * box_words(r) + rw] : 0;
    }
    unsigned salt = 0;   // bit i: row y0 + i
    if (ix >= b.x0 && ix < b.x0 + b.bx) {
        float x[kOut];
#pragma unroll
        for (int i = 0; i < kOut; ++i) x[i] = xi[((int64_t)iz * ny + min(y0 + i, yend - 1)) * nx + ix];
        auto t = [&](int i) { return a_rbar * (double)x[i]; };
        auto in = [&](int i) { return (inside[i] >> lane & 1) != 0; };
        // a squared distance from (1 + 1e-12) t^2 is above the threshold, one up to (1 - 1.5e-12) t^2 below it
        const double enough = 1.0 - 2.5e-12;
        // (kept finite where t^2 overflows: a best value is infinite until a feature is met, and must not pass for decided)
        auto limit = [&](int i, bool wanted) {
            return wanted && y0 + i < yend ? fmin(t(i) * t(i) * (1.0 + 1e-12), 1.7976931348623157e308) : -1.0;
        };
        double best[kOut], lim[kOut];
        const double *go = gout + (int64_t)lz * r.by * b.bx + (ix - b.x0);
        auto fo = [&](int i) {
            const int y = y0 + i - r.y0;
            const double d = go[(int64_t)min(max(y, 0), r.by - 1) * b.bx];
            return y >= 0 && y < r.by ? d : inf_d();
        };
#pragma unroll
        for (int i = 0; i < kOut; ++i) {
            best[i] = fo(i);
            lim[i] = limit(i, !in(i) && t(i) > 0.0);
        }
        const int ylast = r.y0 + r.by - 1;
        const int k0 = y0 + kOut - 1 < r.y0 ? r.y0 - (y0 + kOut - 1) : (y0 > ylast ? y0 - ylast : 1);
        search(best, lim, enough, dy, k0, max(ylast - y0, y0 + kOut - 1 - r.y0), fo);
        bool any = false;
#pragma unroll
        for (int i = 0; i < kOut; ++i) {
            any |= in(i);
            if (!in(i) && -sqrt(best[i]) + t(i) > 0.0) salt |= 1u << i;
        }
        if (any) {   // every inside voxel is in r
            const double *gi = gin + (int64_t)(iz - r.z0) * r.by * r.bx + (ix - r.x0);
            auto fi = [&](int i) {
                const int y = y0 + i - r.y0;
                const double d = gi[(int64_t)min(max(y, 0), r.by - 1) * r.bx];
                return y >= 0 && y < r.by ? d : inf_d();
            };
#pragma unroll
            for (int i = 0; i < kOut; ++i) {
                best[i] = fi(i);
                lim[i] = limit(i, in(i) && t(i) < 0.0);
            }
            search(best, lim, enough, dy, 1, r.by, fi);
#pragma unroll
            for (int i = 0; i < kOut; ++i)
                if (in(i) && sqrt(best[i]) + t(i) > 0.0) salt |= 1u << i;
        }
    }
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const uint64_t set = __ballot((salt >> i & 1u) && y0 + i < yend);
        if (set && lane == 0) K[((int64_t)iz * ny + y0 + i) * row_words(nx) + word] |= set;
    }
}

// g[p] = min over q of (w (p0 + p - q))^2 + f(q), p = 0 .. m-1, q = 0 .. n-1:
// the lower envelope of the parabolas rooted at the finite samples.  v holds
// the envelope's roots (stride vs), g's stride is gs.  The top two roots also
// live in registers; where neighbouring parabolas meet is computed again when
// it is needed (kept in memory, it would be the largest array).  f is read four
// samples ahead.
template <class F>
__device__ __forceinline__ void envelope(int n, int p0, int m, double w, F f, int32_t *v, int64_t vs, double *g, int64_t gs)
{
    const double w2 = w * w;
    auto height = [&](int q, double fq) { return fq + w2 * ((double)q * q); };
    // abscissa where the parabola of root b starts to lie below that of a < b
    auto meet = [&](int a, double ha, int b, double hb) { return (hb - ha) / (2.0 * w2 * (double)(b - a)); };
    int k = -1;                    // index of the last parabola of the envelope
    int vk = 0, vl = 0;            // its root, and that of the one before
    double hk = 0.0, hl = 0.0;     // their heights
    double zk = 0.0;               // where it starts
    double f0 = f(0), f1 = n > 1 ? f(1) : 0.0, f2 = n > 2 ? f(2) : 0.0, f3 = n > 3 ? f(3) : 0.0;
    for (int q = 0; q < n; ++q) {
        const double fq = f0;
        f0 = f1;
        f1 = f2;
        f2 = f3;
        f3 = q + 4 < n ? f(q + 4) : 0.0;
        if (!(fq < inf_d())) continue;
        const double hq = height(q, fq);
        double s = 0.0;
        while (k >= 0) {
            s = meet(vk, hk, q, hq);
            if (k == 0 || s > zk) break;
            --k;
            vk = vl;
            hk = hl;
            if (k > 0) {
                vl = v[(k - 1) * vs];
                hl = height(vl, f(vl));
                zk = meet(vl, hl, vk, hk);
            }
        }
        if (++k > 0) {
            vl = vk;
            hl = hk;
            zk = s;
        }
        vk = q;
        hk = hq;
        v[k * vs] = q;
    }
    if (k < 0) {
        for (int p = 0; p < m; ++p) g[p * gs] = inf_d();
        return;
    }
    int j = 0, vj = v[0], vn = 0;
    double fj = f(vj), fn = 0.0, zn = inf_d();   // (zn: where parabola j + 1 starts)
    auto look_ahead = [&]() {
        zn = inf_d();
        if (j < k) {
            vn = v[(j + 1) * vs];
            fn = f(vn);
            zn = meet(vj, height(vj, fj), vn, height(vn, fn));
        }
    };
    look_ahead();
    for (int p = 0; p < m; ++p) {
        const double at = (double)(p0 + p);
        while (zn < at) {
            ++j;
            vj = vn;
            fj = fn;
            look_ahead();
        }
        const double d = w * (at - (double)vj);
        g[p * gs] = d * d + fj;
    }
}

// The pass along z where k_dist_z's searches would go far: the same distances,
// none of them cut off, one thread per line of box r's rows y, the transforms of
// d_in (on r) and d_out (on box `outer`, from r) side by side (blockIdx.y).  The
// x distances k come with rows in [y][z], so that a line's samples lie close.
struct EnvelopeSide {
    const int32_t *k;
    double *g;
    int32_t *v;   // room for the roots
};
__global__ void __launch_bounds__(kSaltThreads) k_envelope_z(Box r, Box outer, double dz, double dx, EnvelopeSide in,
                                                             EnvelopeSide out)
{
    const Box b = blockIdx.y == 0 ? r : outer;
    const EnvelopeSide S = blockIdx.y == 0 ? in : out;
    const int64_t l = (int64_t)blockIdx.x * kSaltThreads + threadIdx.x;
    if (l >= (int64_t)r.by * b.bx) return;
    const int ly = (int)(l / b.bx), lx = (int)(l - (int64_t)ly * b.bx);
    const int64_t at = (int64_t)ly * r.bz * b.bx + lx;
    auto f = [&](int q) {
        const int32_t c = S.k[at + (int64_t)q * b.bx];
        const double d = dx * (double)c;
        return c < 0 ? inf_d() : d * d;
    };
    envelope(r.bz, b.z0 - r.z0, b.bz, dz, f, S.v + at, b.bx, S.g + (int64_t)ly * b.bx + lx, (int64_t)r.by * b.bx);
}

__global__ void __launch_bounds__(kSaltThreads) k_fill_u32(int64_t n, unsigned val, unsigned *p)
{
    for (int64_t q = (int64_t)blockIdx.x * kSaltThreads + threadIdx.x; q < n; q += (int64_t)gridDim.x * kSaltThreads)
        p[q] = val;
}

// erode (op 0): set where the voxel and its six neighbours are all set;
// dilate (op 1): set where the voxel or any neighbour is set; a thread per
// word.  A neighbour outside the volume counts as empty.
__global__ void __launch_bounds__(kSaltThreads) k_morph(int op, int nz, int ny, int nx, const uint64_t *in, uint64_t *out)
{
    const int nw = row_words(nx);
    const int64_t q = (int64_t)blockIdx.x * kSaltThreads + threadIdx.x, plane = (int64_t)ny * nw;
    if (q >= plane * nz) return;
    const int w = (int)(q % nw);
    const int64_t row = q / nw;
    const int iy = (int)(row % ny), iz = (int)(row / ny);
    const uint64_t c = in[q];
    const uint64_t zm = iz > 0 ? in[q - plane] : 0, zp = iz < nz - 1 ? in[q + plane] : 0;
    const uint64_t ym = iy > 0 ? in[q - nw] : 0, yp = iy < ny - 1 ? in[q + nw] : 0;
    const uint64_t xm = c << 1 | (w > 0 ? in[q - 1] >> 63 : 0), xp = c >> 1 | (w < nw - 1 ? in[q + 1] << 63 : 0);
    uint64_t r = op == 0 ? (c & zm & zp & ym & yp & xm & xp) : (c | zm | zp | ym | yp | xm | xp);
    if (w == nw - 1 && (nx & 63)) r &= ~(~0ull << (nx & 63));
    out[q] = r;
}

// Labels form a forest over the salt voxels: label[x] <= x, a root has
// label[r] == r, and every label names a voxel of the same component.  Labels
// only ever decrease (atomicMin), so a chain strictly decreases and find ends;
// a stale read returns an older ancestor, which is still an ancestor.
__device__ inline int find_root(const int *label, int x)
{
    for (;;) {
        const int p = label[x];
        if (p == x) return x;
        x = p;
    }
}

// Link the roots of a and b, the larger under the smaller.  atomicMin returns
// the previous value: equal to the root means linked; otherwise that root had
// been linked meanwhile and the loop continues from its (smaller) parent.
// Every retry lowers a + b, so the loop ends; no thread waits on another.
__device__ inline void unite(int *label, int a, int b)
{
    for (;;) {
        a = find_root(label, a);
        b = find_root(label, b);
        if (a == b) return;
        if (a > b) {
            const int t = a;
            a = b;
            b = t;
        }
        const int old = atomicMin(&label[b], a);
        if (old == b) return;
        b = old;
    }
}

// Calls f(row, word index, word) for the words of `rows` rows from row0 that
// have a bit set; one wave walks them (64 words are read at a time, a lane each).
template <class F>
__device__ __forceinline__ void set_words(const uint64_t *K, int nw, int64_t row0, int rows, int64_t nrow, F f)
{
    const int lane = threadIdx.x & 63;
    const int64_t end = min(row0 + rows, nrow) * nw;
    for (int64_t q0 = row0 * nw; q0 < end; q0 += 64) {
        const uint64_t mine = q0 + lane < end ? K[q0 + lane] : 0;
        for (uint64_t any = __ballot(mine != 0); any; any &= any - 1) {
            const int l = __ffsll((unsigned long long)any) - 1;
            const uint64_t lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)mine, l);
            const uint64_t hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(mine >> 32), l);
            const int64_t q = q0 + l, row = q / nw;
            f(row, (int)(q - row * nw), hi << 32 | lo);
        }
    }
}
constexpr int kRowsPerWave = 16;

// Initial forest: a salt voxel points at the first voxel of its run along x
// within its word, with a count of 0.  Other voxels have no label.
__global__ void __launch_bounds__(kSaltThreads) k_cc_init(int64_t nrow, int nx, const uint64_t *K, int *label,
                                                          unsigned *count)
{
    const int lane = threadIdx.x & 63;
    set_words(K, row_words(nx), wave_index() * kRowsPerWave, kRowsPerWave, nrow, [&](int64_t row, int w, uint64_t bits) {
        if (!(bits >> lane & 1)) return;
        const uint64_t gaps = ~bits & (~0ull >> (63 - lane));
        const int start = gaps ? 64 - __clzll((long long)gaps) : 0;   // one past the last gap at or below the lane
        const int64_t q = row * nx + w * 64;
        label[q + lane] = (int)(q + start);
        count[q + lane] = 0;
    });
}

// Joins the runs: across a word boundary along x, and along -y and -z unless
// the voxel's left neighbour and that neighbour's own -y (-z) neighbour are
// both salt, in which case the left neighbour's join (or one further left)
// already connects the two runs.
__global__ void __launch_bounds__(kSaltThreads) k_cc_merge(int64_t nrow, int ny, int nx, const uint64_t *K, int *label)
{
    const int lane = threadIdx.x & 63, nw = row_words(nx);
    set_words(K, nw, wave_index() * kRowsPerWave, kRowsPerWave, nrow, [&](int64_t row, int w, uint64_t bits) {
        const uint64_t *kw = K + row * nw + w;
        auto joins = [&](const uint64_t *o) {   // where to join with the row of words o (the neighbour along -y or -z)
            const uint64_t both = bits & o[0];
            return both & ~(both << 1 | (w > 0 ? (kw[-1] & o[-1]) >> 63 : 0));
        };
        const uint64_t at = 1ull << lane;
        const int64_t q = row * nx + w * 64 + lane;
        if (w > 0 && lane == 0 && (bits & 1) && kw[-1] >> 63) unite(label, (int)q, (int)(q - 1));
        if (row % ny > 0 && (joins(kw - nw) & at)) unite(label, (int)q, (int)(q - nx));
        if (row >= ny && (joins(kw - (int64_t)ny * nw) & at)) unite(label, (int)q, (int)(q - (int64_t)ny * nx));
    });
}

// After the merge has finished: every label becomes its root (only the
// thread's own entry is written, and only with an ancestor of it), and the
// sizes of the components: a wave adds up the voxels of one root as long as
// it meets no other, then adds them to a small table of (label, count) in LDS
// (linear probing by atomicCAS on the label slot); the table goes to memory
// with one atomic per distinct label per workgroup, and counts that find
// the table full go straight to memory.
constexpr int kCountSlots = 32;

__global__ void __launch_bounds__(kSaltThreads) k_cc_count(int64_t nrow, int nx, const uint64_t *K, int *label,
                                                           unsigned *count)
{
    __shared__ int tl[kCountSlots];
    __shared__ unsigned tc[kCountSlots];
    if (threadIdx.x < kCountSlots) {
        tl[threadIdx.x] = -1;
        tc[threadIdx.x] = 0u;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    auto add = [&](int l, unsigned c) {
        for (int i = 0; i < kCountSlots; ++i) {
            const int slot = (l + i) & (kCountSlots - 1);
            const int old = atomicCAS(&tl[slot], -1, l);
            if (old == -1 || old == l) {
                atomicAdd(&tc[slot], c);
                return;
            }
        }
        atomicAdd(&count[l], c);
    };
    int cur = -1;        // (uniform over the wave)
    unsigned cnt = 0;
    set_words(K, row_words(nx), wave_index() * kRowsPerWave, kRowsPerWave, nrow, [&](int64_t row, int w, uint64_t bits) {
        const bool set = bits >> lane & 1;
        int root = -1;
        if (set) {
            const int64_t q = row * nx + w * 64 + lane;
            const int l = label[q];
            root = find_root(label, l);
            if (root != l) label[q] = root;
        }
        for (uint64_t left = bits; left;) {
            const int r = __builtin_amdgcn_readlane(root, __ffsll((unsigned long long)left) - 1);
            const uint64_t same = __ballot(set && root == r) & left;
            if (r != cur) {
                if (cur >= 0 && lane == 0) add(cur, cnt);
                cur = r;
                cnt = 0;
            }
            cnt += (unsigned)__popcll((unsigned long long)same);
            left &= ~same;
        }
    });
    if (cur >= 0 && lane == 0) add(cur, cnt);
    __syncthreads();
    if (threadIdx.x < kCountSlots && tl[threadIdx.x] >= 0) atomicAdd(&count[tl[threadIdx.x]], tc[threadIdx.x]);
}

// One wave per row; VEC: four voxels per lane (rows and pointers allow it), 256
// of them per step, two steps in flight; else one voxel per lane, four words
// in flight.
template <bool VEC>
__global__ void __launch_bounds__(kSaltThreads) k_salt_write(int64_t nrow, int nx, const float *__restrict__ v,
                                                             const uint64_t *__restrict__ K,
                                                             const int *__restrict__ label,
                                                             const unsigned *__restrict__ count, unsigned min_voxels,
                                                             float v_salt, float v_water, float *__restrict__ out,
                                                             uint8_t *__restrict__ mask_out)
{
    const int64_t row = wave_index();
    if (row >= nrow) return;
    const int lane = threadIdx.x & 63, nw = row_words(nx);
    constexpr int kPer = VEC ? 4 : 1, kFlight = VEC ? 2 : 4, kStep = 64 * kPer;
    typedef float Values __attribute__((ext_vector_type(VEC ? 4 : 1)));
    typedef uint8_t Bytes __attribute__((ext_vector_type(VEC ? 4 : 1)));
    for (int x0 = kPer * lane; x0 < nx; x0 += kFlight * kStep) {
        Values vq[kFlight];
        unsigned bits[kFlight];
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int x = min(x0 + u * kStep, nx - kPer);
            vq[u] = __builtin_nontemporal_load((const Values *)(v + row * nx + x));
            bits[u] = (unsigned)(K[row * nw + x / 64] >> (x & 63)) & (VEC ? 15u : 1u);
        }
#pragma unroll
        for (int u = 0; u < kFlight; ++u) {
            const int x = x0 + u * kStep;
            if (x >= nx) continue;
            const int64_t q = row * nx + x;
            Bytes m;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                const bool k = (bits[u] >> j & 1) && count[label[q + j]] >= min_voxels && vq[u][j] >= v_water;
                if (k) vq[u][j] = v_salt;
                m[j] = k;
            }
            __builtin_nontemporal_store(vq[u], (Values *)(out + q));
            if (mask_out) __builtin_nontemporal_store(m, (Bytes *)(mask_out + q));
        }
    }
}

// The pass along z searches while no search can go farther than kFarSearch
// cells (the largest |a rbar xi|, or the box's planes), and takes the envelopes
// beyond: a search's cost grows with its length, an envelope's does not.  One
// body with a smooth field, both transforms: 619 x 1000 x 1000 voxels, radii 155
// cells, search up to 85 cells 1.07 ms and envelopes 1.48, 170 2.10 and 1.65, 283
// 3.52 and 1.75, 567 11.3 and 1.93; radii 413, 227 cells 24.8 and 10.5; 300 x 400 x
// 400, radii 83, 118 cells 0.34 and 0.49, 235 0.60 and 0.48.  An envelope is one
// thread per line, so below kFewLines lines, which leave the chip idle, the
// searches may be longer in proportion: 4000 x 200 x 100 (20000 lines), 520 cells
// 2.9 and 3.0; 619 x 1 x 1000, 124 cells 0.06 and 0.80.
// (The pass along y ends at the decision, whatever the limit: 567 cells in the
// full volume 11.5 ms and 9.3 by envelopes, 378 with radii of 413 11.9 and 22.2,
// 880 in 20 x 2000 x 600 voxels 0.5 and 2.5.  Envelopes in both passes were faster
// in all on very long lines under fields of several times the radii: 200 x 10000 x
// 100 at amplitude 3 27.0 ms against 30.8, 400 x 1500 x 1000 50.3 against 50.6.)
constexpr double kFarSearch = 160.0, kFewLines = 80000.0;

// The workspace holds six arrays of 8 bytes and two of 4 bytes per voxel, and
// two of a byte.  Used: the two transforms' x distances and their distances
// over x and z (d_in, d_out, f), the sets K and its scratch (words; as many as
// voxels where rows have one voxel), the raster's words, the extremes.
struct SaltWorkspace {
    double *din, *dout, *f[2];
    uint64_t *K, *T, *raster;
    unsigned *ext;
};

inline size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

SaltWorkspace carve(void *ws, int64_t n)
{
    char *p = (char *)ws;
    SaltWorkspace W{};
    const size_t a8 = align256(8 * (size_t)n), a4 = align256(4 * (size_t)n), a1 = align256((size_t)n);
    W.din = (double *)p;
    W.dout = (double *)(p + a8);
    W.f[0] = (double *)(p + 2 * a8);
    W.f[1] = (double *)(p + 3 * a8);
    W.K = (uint64_t *)(p + 4 * a8);
    W.T = (uint64_t *)(p + 5 * a8);
    W.raster = (uint64_t *)(p + 6 * a8);   // two arrays of 4 bytes per voxel
    W.ext = (unsigned *)(p + 6 * a8 + 2 * a4 + 2 * a1);
    return W;
}

// Index range [lo, hi] along one axis of spacing h and n voxels covering
// centre +- reach (metres) plus two voxels; false if it misses the axis.
bool axis_range(double centre, double reach, double h, int n, int &lo, int &hi)
{
    if (!std::isfinite(reach)) {
        lo = 0;
        hi = n - 1;
        return true;
    }
    const double a = std::floor((centre - reach) / h) - 2.0, b = std::ceil((centre + reach) / h) + 2.0;
    if (b < 0.0 || a > n - 1.0) return false;
    lo = a < 0.0 ? 0 : (int)a;
    hi = b > n - 1.0 ? n - 1 : (int)b;
    return true;
}

}  // namespace

size_t salt_workspace_bytes(int64_t n)
{
    return 6 * align256(8 * (size_t)n) + 2 * align256(4 * (size_t)n) + 2 * align256((size_t)n) +
           align256(2 * sizeof(unsigned) * kSaltMaxBodies);
}

hipError_t launch_salt_sdt(const float *v, int nz, int ny, int nx, double dz, double dy, double dx, int nbodies,
                           const SaltBody *bodies, const float *grf, double amplitude, float v_salt, float v_water,
                           unsigned min_voxels, float *out, uint8_t *mask_out, void *ws, hipStream_t st)
{
    const int64_t n = (int64_t)nz * ny * nx;
    const SaltWorkspace W = carve(ws, n);
    const dim3 blk(kSaltThreads);
    const int nw = row_words(nx);
    const int64_t nrow = (int64_t)nz * ny;
    hipError_t e;
    hipLaunchKernelGGL(k_fill_u32, dim3(std::min(blocks_for(2 * nrow * nw), 65536u)), blk, 0, st, 2 * nrow * nw, 0u,
                       (unsigned *)W.K);
    std::vector<unsigned> ext(2 * (size_t)nbodies, 0u);
    if (nbodies > 0) {
        hipLaunchKernelGGL(k_fill_u32, dim3(blocks_for(2 * nbodies)), blk, 0, st, (int64_t)2 * nbodies, 0u, W.ext);
        const unsigned per_body = std::min(blocks_for(n), 1024u);
        hipLaunchKernelGGL(k_field_extremes, dim3(per_body, nbodies), blk, 0, st, n, grf, W.ext);
        if ((e = hipMemcpyAsync(ext.data(), W.ext, ext.size() * sizeof(unsigned), hipMemcpyDeviceToHost, st)) !=
            hipSuccess)
            return e;
        if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
    }
    for (int i = 0; i < nbodies; ++i) {
        const SaltBody &B = bodies[i];
        const double rbar = (B.r[0] + B.r[1] + B.r[2]) / 3.0;
        float hi, lo;
        std::memcpy(&hi, &ext[2 * i], sizeof hi);
        std::memcpy(&lo, &ext[2 * i + 1], sizeof lo);
        // largest a rbar xi over the volume: how far beyond the raster the body can reach
        const double reach = std::max(0.0, amplitude >= 0 ? amplitude * rbar * hi : -amplitude * rbar * lo);
        // half extent of the rotated ellipsoid along world axis j: |column j of R^T diag(r)|
        const double h[3] = {dz, dy, dx};
        const int nn[3] = {nz, ny, nx};
        // bo: the raster's box widened by the reach (where the body can add salt, and d_out is needed);
        // bi: the raster's box alone (d_in is needed only at inside voxels)
        int lo_o[3], hi_o[3], lo_n[3], hi_n[3];
        bool hit = true;
        for (int j = 0; j < 3 && hit; ++j) {
            double e2 = 0.0;
            for (int k = 0; k < 3; ++k) e2 += (B.R[3 * k + j] * B.r[k]) * (B.R[3 * k + j] * B.r[k]);
            const double ext = std::sqrt(e2) * (1.0 + 1e-6);
            hit = axis_range(B.c[j], ext, h[j], nn[j], lo_n[j], hi_n[j]) &&
                  axis_range(B.c[j], ext + reach, h[j], nn[j], lo_o[j], hi_o[j]);
        }
        if (!hit) continue;   // the raster misses the volume: the body adds nothing
        const Box bo{lo_o[0], lo_o[1], lo_o[2], hi_o[0] - lo_o[0] + 1, hi_o[1] - lo_o[1] + 1, hi_o[2] - lo_o[2] + 1};
        const Box bi{lo_n[0], lo_n[1], lo_n[2], hi_n[0] - lo_n[0] + 1, hi_n[1] - lo_n[1] + 1, hi_n[2] - lo_n[2] + 1};
        // the ellipsoid's projection onto (z, y): covariance R^T diag(r^2) R
        auto cov = [&](int p, int q) {
            double s = 0.0;
            for (int k = 0; k < 3; ++k) s += B.R[3 * k + p] * B.R[3 * k + q] * B.r[k] * B.r[k];
            return s;
        };
        // (margins for a rotation that is orthonormal within 1e-7 only, amplified by unequal radii)
        const double rmax = std::max(B.r[0], std::max(B.r[1], B.r[2])), tol = 1e-6 * rmax * rmax;
        const double cyy = cov(1, 1), slope = cov(0, 1) / cyy;
        const ZSpan S{B.c[0], B.c[1], slope, std::max(cov(0, 0) - slope * cov(0, 1), 0.0) + tol, cyy + tol,
                      1e-6 * rmax + tol / std::sqrt(cyy)};
        const double a_rbar = amplitude * rbar;
        const float *xi = grf + (int64_t)i * n;
        hipLaunchKernelGGL(k_raster, dim3(wave_blocks((int64_t)bi.bz * bi.by * box_words(bi))), blk, 0, st, bi, dz, dy,
                           dx, B, W.raster);
        auto dist_x = [&](const Box &b, int outside, bool by_y, void *k) {
            hipLaunchKernelGGL(k_dist_x, dim3(wave_blocks((int64_t)bi.bz * bi.by)), blk, 0, st, bi, b.x0, b.bx,
                               (const uint64_t *)W.raster, outside, by_y, (int32_t *)k);
        };
        // d_in: distance to the nearest voxel outside, on bi; d_out: to the nearest inside, on the planes and
        // columns of bo and (before the last pass) the rows y of bi, which hold the whole body
        const double reach_in = std::max(0.0, amplitude >= 0 ? amplitude * rbar * lo : -amplitude * rbar * hi);
        const double far = std::max(std::min(reach / dz, (double)bo.bz), std::min(reach_in / dz, (double)bi.bz));
        const double lines = (double)bi.by * bo.bx;
        if (far > kFarSearch * std::max(kFewLines / lines, 1.0)) {
            dist_x(bi, 1, true, W.din);
            dist_x(bo, 0, true, W.dout);
            // (the roots lie behind the x distances: 8 bytes a voxel hold both)
            const EnvelopeSide in{(const int32_t *)W.din, W.f[0], (int32_t *)W.din + n};
            const EnvelopeSide out{(const int32_t *)W.dout, W.f[1], (int32_t *)W.dout + n};
            hipLaunchKernelGGL(k_envelope_z, dim3(blocks_for((int64_t)bi.by * bo.bx), 2), blk, 0, st, bi, bo, dz, dx, in,
                               out);
        } else {
            float2 *lohi = (float2 *)W.T;
            hipLaunchKernelGGL(k_field_bounds, dim3(wave_blocks((int64_t)((bo.bx + 63) / 64) * bo.bz)), blk, 0, st, bo,
                               ny, nx, xi, lohi);
            auto transform = [&](const Box &b, int inner, int32_t *k, double *g) {
                dist_x(b, inner, false, k);
                const int64_t waves = (int64_t)((b.bx + 63) / 64) * bi.by * ((b.bz + kOutZ - 1) / kOutZ);
                hipLaunchKernelGGL(k_dist_z, dim3(wave_blocks(waves)), blk, 0, st, bi, b, dz, dy, dx, S, inner, a_rbar,
                                   bo, (const float2 *)lohi, (const int32_t *)k, g);
            };
            transform(bi, 1, (int32_t *)W.din, W.f[0]);
            transform(bo, 0, (int32_t *)W.dout, W.f[1]);
        }
        const int64_t waves = (int64_t)box_words(bo) * bo.bz * ((bo.by + kOutY - 1) / kOutY);
        hipLaunchKernelGGL(k_dist_y, dim3(wave_blocks(waves)), blk, 0, st, bi, bo, ny, nx, dy,
                           (const uint64_t *)W.raster, (const double *)W.f[0], (const double *)W.f[1], xi, a_rbar, W.K);
    }
    // opening (erode, dilate) then closing (dilate, erode), ping-ponging K and T
    const int ops[4] = {0, 1, 1, 0};
    for (int i = 0; i < 4; ++i)
        hipLaunchKernelGGL(k_morph, dim3(blocks_for(nrow * nw)), blk, 0, st, ops[i], nz, ny, nx,
                           (const uint64_t *)(i % 2 ? W.T : W.K), i % 2 ? W.K : W.T);
    // components: labels in d_in's storage, sizes in d_out's
    int *label = (int *)W.din;
    unsigned *count = (unsigned *)W.dout;
    const dim3 cc(wave_blocks((nrow + kRowsPerWave - 1) / kRowsPerWave));
    hipLaunchKernelGGL(k_cc_init, cc, blk, 0, st, nrow, nx, (const uint64_t *)W.K, label, count);
    hipLaunchKernelGGL(k_cc_merge, cc, blk, 0, st, nrow, ny, nx, (const uint64_t *)W.K, label);
    hipLaunchKernelGGL(k_cc_count, cc, blk, 0, st, nrow, nx, (const uint64_t *)W.K, label, count);
    const bool vec = nx % 4 == 0 && ((uintptr_t)v & 15) == 0 && ((uintptr_t)out & 15) == 0 &&
                     ((uintptr_t)mask_out & 3) == 0;
    auto *write = vec ? k_salt_write<true> : k_salt_write<false>;
    hipLaunchKernelGGL(write, dim3(wave_blocks(nrow)), blk, 0, st, nrow, nx, v, (const uint64_t *)W.K,
                       (const int *)label, (const unsigned *)count, min_voxels, v_salt, v_water, out, mask_out);
    return hipGetLastError();
}

}  // namespace sg
