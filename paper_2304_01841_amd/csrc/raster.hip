// Rasterization and Scatter-Add on gfx950 (arXiv:2304.01841, Sec. 2 steps 1-2).
//
// Per depo (FP64): drift to the response plane, Gaussian widths sqrt(2 D T),
// continuous bin coordinates and the inclusive window floor(mu -/+ n s) on each
// axis.  Bin weights are differences of erf at the bin edges normalised over
// the window (FP64); the patch is the outer product of the two weight vectors
// times the charge (FP32).  With fluctuation, every bin draws a normal deviate
// from a Philox4x32-10 stream keyed by (event, depo, absolute bin) and takes
// the normal approximation of a binomial draw, clamped at zero, and the patch
// is rescaled to the depo charge.
//
// Scatter-Add (Sec. 2 step 2) runs two ways:
//  * fused (simulate path): depos are binned by the grid tile holding their
//    window origin (count -> list offsets -> fill; offsets in tile order, the
//    scan of Sec. 4.3, for reproducible sums);
//    a tile's list is cut into work items of a few dozen depos, and one
//    wavefront per work item rasterizes them, one patch at a time, into its
//    own LDS copy of the tile plus a halo, then adds the non-zero LDS cells to
//    the grid with float atomics, so the grid sees one atomic per touched cell
//    per work item instead of one per patch bin;
//  * unfused (patch-set API): patches are written to a flat buffer at the
//    scanned offsets and a second kernel adds them to the grid atomically, summed
//    in LDS first where consecutive patches lie close together.
#include <math.h>

#include <limits.h>

#include <atomic>
#include <type_traits>

#include "wcsim_internal.h"

namespace wcs {
namespace {

constexpr double kSqrt2 = 1.41421356237309504880;  // sqrt(2), correctly rounded

// Philox4x32-10 round constants (Salmon et al., SC'11).
constexpr uint32_t kPhiloxM0 = 0xD2511F53u, kPhiloxM1 = 0xCD9E8D57u;
constexpr uint32_t kPhiloxW0 = 0x9E3779B9u, kPhiloxW1 = 0xBB67AE85u;

// a ^ b ^ c in one gfx950 three-input bitwise instruction (truth table 0x96:
// the result bit is set when an odd number of input bits are)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r > 0) {
            k0 += kPhiloxW0;
            k1 += kPhiloxW1;
        }
        const uint64_t a = (uint64_t)kPhiloxM0 * c.x;
        const uint64_t b = (uint64_t)kPhiloxM1 * c.z;
        c = make_uint4(xor3((uint32_t)(b >> 32), c.y, k0), (uint32_t)b,
                       xor3((uint32_t)(a >> 32), c.w, k1), (uint32_t)a);
    }
    return c;
}

// Uniform ((r >> 9) + 1/2) 2^-23 in (0, 1), exact in binary32: the float
// 1 + m 2^-23 (m = r >> 9 as its mantissa) minus (1 - 2^-24) is
// (2m + 1) 2^-24, an exact difference.
__device__ __forceinline__ float word_to_uniform(uint32_t r)
{
    return __uint_as_float((r >> 9) | 0x3f800000u) - (1.0f - 0x1p-24f);
}

// Box-Muller pair: cosine branch (even tick) and sine branch (odd tick).
// v_sin/v_cos take their argument in revolutions, so theta = 2 pi u is u;
// v_log gives log2, and -2 ln u = (-2 ln 2) log2 u.  u >= 2^-24 is never
// denormal, so the hardware instructions need no range fix-ups.
__device__ __forceinline__ void box_muller(uint32_t a, uint32_t b, float &zc, float &zs)
{
    constexpr float kMinus2Ln2 = -1.38629436111989061883f;
    const float rho =
        __builtin_amdgcn_sqrtf(kMinus2Ln2 * __builtin_amdgcn_logf(word_to_uniform(a)));
    const float u = word_to_uniform(b);
    zc = rho * __builtin_amdgcn_cosf(u);
    zs = rho * __builtin_amdgcn_sinf(u);
}

// ln u in FP64 for a uniform u in (0, 1) (a normal number): u = 2^e f with f in
// (sqrt(1/2), sqrt(2)], ln f = 2 atanh(s) with s = (f - 1) / (f + 1), |s| <
// 0.1716, by the series of atanh to s^19 (the next term is below 2^-55 of the
// sum).  f - 1 is exact, so the digits stay where ln u nears zero (u > 0.7 has
// e = 0).  The library function's special cases cannot occur.
__device__ __forceinline__ double ln_uniform(double u)
{
    const long long b = __double_as_longlong(u);
    int e = (int)(b >> 52) - 1023;
    double f = __longlong_as_double((b & 0xfffffffffffffll) | 0x3ff0000000000000ll);
    const bool up = f > kSqrt2;
    f = up ? 0.5 * f : f;
    e += up ? 1 : 0;
    const double d = f + 1.0;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    r = fma(r, fma(-d, r, 1.0), r);
    const double s = (f - 1.0) * r, w = s * s;
    double p = 1.0 / 19.0;
    p = fma(p, w, 1.0 / 17.0);
    p = fma(p, w, 1.0 / 15.0);
    p = fma(p, w, 1.0 / 13.0);
    p = fma(p, w, 1.0 / 11.0);
    p = fma(p, w, 1.0 / 9.0);
    p = fma(p, w, 1.0 / 7.0);
    p = fma(p, w, 1.0 / 5.0);
    p = fma(p, w, 1.0 / 3.0);
    const double l = 2.0 * fma(s * w, p, s);
    return fma((double)e, 0.69314718055994530942, l);
}

// sqrt(x) in FP64 for x of ordinary magnitude: the hardware's reciprocal root
// refined by two coupled Newton steps (root g and half reciprocal root h), then
// one correction by the residual x - g^2.
__device__ __forceinline__ double sqrt_pos_d(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    return fma(fma(-g, g, x), h, g);
}

// cos and sin of 2 pi u in FP64 for a uniform u of 24 bits: 4 u = k + x exactly,
// x in [-1/2, 1/2], then the Taylor series of the angle x pi / 2 (|angle| < 0.79;
// the first terms left out are below 2^-56) turned by k quarters.
__device__ __forceinline__ void cos_sin_turns(double u, double &c, double &s)
{
    const double t = 4.0 * u, k = rint(t);
    const double a = (t - k) * 1.57079632679489661923, w = a * a;
    double p = 1.0 / 355687428096000.0;           // 1 / 17!
    p = fma(p, w, -1.0 / 1307674368000.0);        // 1 / 15!
    p = fma(p, w, 1.0 / 6227020800.0);
    p = fma(p, w, -1.0 / 39916800.0);
    p = fma(p, w, 1.0 / 362880.0);
    p = fma(p, w, -1.0 / 5040.0);
    p = fma(p, w, 1.0 / 120.0);
    p = fma(p, w, -1.0 / 6.0);
    const double sn = fma(a * w, p, a);
    double q = 1.0 / 20922789888000.0;            // 1 / 16!
    q = fma(q, w, -1.0 / 87178291200.0);          // 1 / 14!
    q = fma(q, w, 1.0 / 479001600.0);
    q = fma(q, w, -1.0 / 3628800.0);
    q = fma(q, w, 1.0 / 40320.0);
    q = fma(q, w, -1.0 / 720.0);
    q = fma(q, w, 1.0 / 24.0);
    q = fma(q, w, -0.5);
    const double cs = fma(w, q, 1.0);
    const int n = (int)k;
    c = (n & 1) ? sn : cs;
    s = (n & 1) ? cs : sn;
    c = ((n + 1) & 2) ? -c : c;
    s = (n & 2) ? -s : s;
}

// FP64 Box-Muller pair of the digitisation noise: the uniforms of the two
// words, rho = sqrt(-2 ln u_a), theta = 2 pi u_b, cosine branch (even column)
// and sine branch (odd column), all in double precision.
__device__ __forceinline__ void box_muller_d(uint32_t a, uint32_t b, double &zc, double &zs)
{
    const double ua = ((double)(a >> 9) + 0.5) * 0x1p-23;
    const double ub = ((double)(b >> 9) + 0.5) * 0x1p-23;
    const double rho = sqrt_pos_d(-2.0 * ln_uniform(ua));
    double sn, cs;
    cos_sin_turns(ub, cs, sn);
    zc = rho * cs;
    zs = rho * sn;
}

struct Win {
    double T;  // drift time to the response plane
    double mu_p, s_p, mu_t, s_t, q;
    int lo_p, lo_t, n_p, n_t;
    int status;  // 0 ok, 1 invalid, 2 misses the grid, 3 window too long
};

// Drift, diffusion and window of one depo.  FP64 with no contraction, in the
// order the definitions are written, so that the integer window bounds are
// reproducible bit for bit.
__device__ __forceinline__ Win depo_window(const wcsim_depo &dep, const PlaneParams &P)
{
#pragma clang fp contract(off)
    Win w;
    w.T = 0.0;
    w.status = 0;
    w.lo_p = w.lo_t = w.n_p = w.n_t = 0;
    const double x = dep.x, y = dep.y, z = dep.z, t = dep.t, q = dep.q;
    w.q = q;
    w.mu_p = w.s_p = w.mu_t = w.s_t = 0.0;
    if (!isfinite(x) || !isfinite(y) || !isfinite(z) || !isfinite(t) || !isfinite(q) || q < 0.0 ||
        x < P.plane_x) {
        w.status = 1;
        return w;
    }
    // The drift speed changes linearly with drift time at the rate accel and
    // equals v on the response plane: the depo starts at v_s = sqrt(v^2 -
    // 2 accel L) and drifts for T = 2 L / (v + v_s) (T = L / v exactly when
    // accel = 0); a depo with v^2 - 2 accel L < 0 cannot reach the plane.
    const double L = x - P.plane_x;
    const double disc = P.v * P.v - 2.0 * P.accel * L;
    if (disc < 0.0) {
        w.status = 1;
        return w;
    }
    const double T = (2.0 * L) / (P.v + sqrt(disc));
    w.T = T;
    const double t_arr = t + T;
    const double sigma_p = sqrt(2.0 * P.DT * T);
    const double sigma_t = sqrt(2.0 * P.DL * T) / P.v;
    const double proj = y * P.dir_y + z * P.dir_z;
    w.mu_p = (proj - P.pitch_origin) / P.dp;
    w.s_p = sigma_p / P.dp;
    w.mu_t = (t_arr - P.t0) / P.tick;
    w.s_t = sigma_t / P.tick;
    const double lo_p = floor(w.mu_p - P.nsigma * w.s_p);
    const double hi_p = floor(w.mu_p + P.nsigma * w.s_p);
    const double lo_t = floor(w.mu_t - P.nsigma * w.s_t);
    const double hi_t = floor(w.mu_t + P.nsigma * w.s_t);
    if (hi_p < 0.0 || lo_p >= (double)P.Np || hi_t < 0.0 || lo_t >= (double)P.Nt) {
        w.status = 2;
        return w;
    }
    if (hi_p - lo_p + 1.0 > (double)kMaxWindow || hi_t - lo_t + 1.0 > (double)kMaxWindow) {
        w.status = 3;
        return w;
    }
    w.lo_p = (int)lo_p;
    w.lo_t = (int)lo_t;
    w.n_p = (int)hi_p - w.lo_p + 1;
    w.n_t = (int)hi_t - w.lo_t + 1;
    return w;
}

__device__ __forceinline__ double edge_erf(int lo, int k, double mu, double s)
{
    return erf(((double)(lo + k) - mu) / (kSqrt2 * s));
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int WIDTH>
__device__ __forceinline__ double seg_sum(double v)
{
#pragma unroll
    for (int m = WIDTH / 2; m > 0; m >>= 1)
        v += __shfl_xor(v, m, WIDTH);
    return v;
}

// q / S in FP64 for S > 0 of ordinary magnitude (a patch total): hardware
// reciprocal refined by two Newton steps, then the product, within a few FP64
// ulps of the quotient -- far below the float32 rounding the factor gets.
__device__ __forceinline__ double div_pos_d(double q, double S)
{
    double r = __builtin_amdgcn_rcp(S);
    r = fma(fma(-S, r, 1.0), r, r);
    r = fma(fma(-S, r, 1.0), r, r);
    return q * r;
}

// Inclusive prefix sum over the wavefront's lanes in FP64: within each row of
// 16 lanes by shifts of 1, 2, 4 and 8 lanes, then each row adds the last lane
// of the rows before it (row broadcasts of lanes 15 and 31).  Fixed order.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_shift_d(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((uint64_t)b >> 32), CTRL, ROWS,
                                               0xf, true);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ double wave_incl_scan_d(double v)
{
    v += dpp_shift_d<0x111, 0xf>(v);  // row_shr:1
    v += dpp_shift_d<0x112, 0xf>(v);  // row_shr:2
    v += dpp_shift_d<0x114, 0xf>(v);  // row_shr:4
    v += dpp_shift_d<0x118, 0xf>(v);  // row_shr:8
    v += dpp_shift_d<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v += dpp_shift_d<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_shift_i(int v, int other)
{
    return __builtin_amdgcn_update_dpp(other, v, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum of an integer, and the largest (MIN: smallest) integer of
// the wavefront's lanes (uniform), by the same shifts: no LDS round trips.
__device__ __forceinline__ int wave_incl_scan_i(int v)
{
    v += dpp_shift_i<0x111, 0xf>(v, 0);
    v += dpp_shift_i<0x112, 0xf>(v, 0);
    v += dpp_shift_i<0x114, 0xf>(v, 0);
    v += dpp_shift_i<0x118, 0xf>(v, 0);
    v += dpp_shift_i<0x142, 0xa>(v, 0);
    v += dpp_shift_i<0x143, 0xc>(v, 0);
    return v;
}

template <bool MIN>
__device__ __forceinline__ int wave_max_i(int v)
{
    auto pick = [](int a, int b) { return MIN ? min(a, b) : max(a, b); };
    v = pick(v, dpp_shift_i<0x111, 0xf>(v, v));
    v = pick(v, dpp_shift_i<0x112, 0xf>(v, v));
    v = pick(v, dpp_shift_i<0x114, 0xf>(v, v));
    v = pick(v, dpp_shift_i<0x118, 0xf>(v, v));
    v = pick(v, dpp_shift_i<0x142, 0xa>(v, v));
    v = pick(v, dpp_shift_i<0x143, 0xc>(v, v));
    return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ double readlane_d(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, lane);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)b >> 32), lane);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// Electrons of a depo that survive the drift (electron lifetime tau; an
// extension beyond the paper, which starts from the drifted charge): each
// survives the drift time T with probability p = exp(-T / tau).  The depo
// keeps q p, or with fluctuation the normal approximation of Binomial(q, p),
// clamped at zero.  Absorption precedes the readout planes, so the deviate
// belongs to the depo alone: Philox under the lifetime key (no plane in it)
// at counter (0, 0, depo index in the event, event), the cosine branch of
// Box-Muller on words 0 and 1, all in FP64 (one draw per depo).
__device__ __forceinline__ double surviving_charge(const Win &w, const PlaneParams &P, int d,
                                                   uint32_t event)
{
    if (!(P.tau > 0.0))
        return w.q;
    const double p = exp(-w.T / P.tau);
    if (!P.fluct)
        return w.q * p;
    const uint4 r = philox4x32_10(make_uint4(0u, 0u, (uint32_t)d, event), P.lkey0, P.lkey1);
    const double ua = ((double)(r.x >> 9) + 0.5) * 0x1p-23;
    const double ub = ((double)(r.y >> 9) + 0.5) * 0x1p-23;
    double c, sn;
    cos_sin_turns(ub, c, sn);
    const double z = sqrt_pos_d(-2.0 * ln_uniform(ua)) * c;
    const double F = w.q * p + z * sqrt(w.q * p * (1.0 - p));
    return (F < 0.0) ? 0.0 : F;
}

// Fluctuated bin value before rescaling: normal approximation of the binomial
// draw of q electrons with probability p, clamped at zero.
__device__ __forceinline__ float fluct_value(float q, float p, float z)
{
    const float qp = q * p;
    const float var = fmaf(-qp, p, qp);  // q p (1 - p)
    return fmaxf(0.0f, fmaf(z, __builtin_amdgcn_sqrtf(var), qp));
}

// The same value from the squared Box-Muller radius r2 = -2 ln u and the
// branch's cosine or sine c: z sqrt(var) = c sqrt(r2 var), as rho and the
// standard deviation are both non-negative (one square root instead of two
// per value pair).
__device__ __forceinline__ float fluct_value_r2(float q, float p, float r2, float c)
{
    const float qp = q * p;
    const float var = fmaf(-qp, p, qp);  // q p (1 - p)
    return fmaxf(0.0f, fmaf(c, __builtin_amdgcn_sqrtf(r2 * var), qp));
}

__device__ __forceinline__ int quad_of(int J) { return J >> 2; }  // floor(J / 4)

// ---------------------------------------------------------------------------
// Fill and Philox diagnostic kernels
// ---------------------------------------------------------------------------
__global__ void k_fill_zero16(uint4 *p, size_t n16)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

__global__ void k_fill_zero1(unsigned char *p, size_t n)
{
    size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = 0;
}

__global__ void k_philox(const uint4 *ctr, const uint2 *key, int64_t n, uint4 *out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n)
        out[i] = philox4x32_10(ctr[i], key[i].x, key[i].y);
}

// ---------------------------------------------------------------------------
// Exclusive scan (three phases: block sums, scan of block sums, add)
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256, kScanPer = 4, kScanBlock = kScanThreads * kScanPer;

template <typename T>
__device__ T block_exclusive_scan(T v, T *sh, T *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T u = __shfl_up(inc, o, 64);
        if (lane >= o)
            inc += u;
    }
    if (lane == 63)
        sh[wave] = inc;
    __syncthreads();
    T base = 0, tot = 0;
    for (int k = 0; k < kScanThreads / 64; ++k) {
        if (k < wave)
            base += sh[k];
        tot += sh[k];
    }
    __syncthreads();
    *total = tot;
    return base + inc - v;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_local(T *data, int64_t n, T *block_sums)
{
    __shared__ T sh[kScanThreads / 64];
    const int64_t base = blockIdx.x * (int64_t)kScanBlock + threadIdx.x * kScanPer;
    T v[kScanPer];
    T sum = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        v[k] = (base + k < n) ? data[base + k] : T(0);
        sum += v[k];
    }
    T total;
    T run = block_exclusive_scan<T>(sum, sh, &total);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (base + k < n)
            data[base + k] = run;
        run += v[k];
    }
    if (threadIdx.x == 0)
        block_sums[blockIdx.x] = total;
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_sums(T *sums, int64_t nb)
{
    __shared__ T sh[kScanThreads / 64];
    T carry = 0;
    for (int64_t b0 = 0; b0 < nb; b0 += kScanThreads) {
        const int64_t i = b0 + threadIdx.x;
        T v = (i < nb) ? sums[i] : T(0);
        T total;
        T ex = block_exclusive_scan<T>(v, sh, &total);
        if (i < nb)
            sums[i] = ex + carry;
        carry += total;
    }
}

template <typename T>
__global__ __launch_bounds__(kScanThreads) void k_scan_add(T *data, int64_t n, const T *sums)
{
    const int64_t base = blockIdx.x * (int64_t)kScanBlock + threadIdx.x * kScanPer;
    const T add = sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < kScanPer; ++k)
        if (base + k < n)
            data[base + k] += add;
}

template <typename T>
hipError_t exclusive_scan(T *data, int64_t n, void *scratch, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    const int64_t nb = (n + kScanBlock - 1) / kScanBlock;
    T *sums = (T *)scratch;
    hipLaunchKernelGGL(k_scan_local<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, n, sums);
    hipLaunchKernelGGL(k_scan_sums<T>, dim3(1), dim3(kScanThreads), 0, s, sums, nb);
    hipLaunchKernelGGL(k_scan_add<T>, dim3((unsigned)nb), dim3(kScanThreads), 0, s, data, n, sums);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Unfused path: patch sizes, flat patch values, flat scatter
// ---------------------------------------------------------------------------
// Patches with more than 64 window edges or kWaveItems passes of (row, tick quad)
// items are beyond k_patch_wave's wavefront; `large` lists them for k_patch_generic
// and *nlarge counts them, so that the host, which waits for the patch total anyway,
// can size that launch.
constexpr int kWaveItems = 3;

__device__ __forceinline__ uint64_t lanemask_lt(int lane) { return (1ull << lane) - 1ull; }

__device__ __forceinline__ bool beyond_wave(const Win &w)
{
    const int nq = quad_of(w.lo_t + w.n_t - 1) - quad_of(w.lo_t) + 1;
    return w.status == 0 && (w.n_p + w.n_t + 2 > 64 || w.n_p * nq > 64 * kWaveItems);
}

// Cells of a wavefront's LDS region in k_scatter_flat, and the neighbours that
// PatchSums::close looks at together.
constexpr int kScatCells = 1536, kCloseDepos = 8;

__global__ __launch_bounds__(256) void k_patch_sizes(const wcsim_depo *depos, int64_t n,
                                                     PlaneParams P, int32_t *meta, int64_t *sizes,
                                                     int32_t *large, PatchSums *sums)
{
    const int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    if (d == 0)
        sizes[n] = 0;
    Win w{};
    w.status = 2;
    bool ok = false;
    if (d < n) {
        w = depo_window(depos[d], P);
        ok = (w.status == 0);
        meta[4 * d + 0] = ok ? w.lo_p : 0;
        meta[4 * d + 1] = ok ? w.lo_t : 0;
        meta[4 * d + 2] = ok ? w.n_p : 0;
        meta[4 * d + 3] = ok ? w.n_t : 0;
        sizes[d] = ok ? (int64_t)w.n_p * w.n_t : 0;
    }
    const bool big = beyond_wave(w);
    const uint64_t m = __ballot(big);
    if (m) {
        int base = 0;
        if (lane == 0)
            base = atomicAdd(&sums->nlarge, __popcll(m));
        base = __builtin_amdgcn_readlane(base, 0);
        if (big)
            large[base + __popcll(m & lanemask_lt(lane))] = (int32_t)d;
    }
    // Groups of neighbours whose patches' bounding box fits the region, less those
    // whose does not, over every eighth workgroup (all of them on the one counter
    // cost 4 us for 100,000 depos).
    if (blockIdx.x & 7)
        return;
    int rlo = ok ? max(w.lo_p, 0) : INT_MAX, rhi = ok ? min(w.lo_p + w.n_p, P.Np) : 0;
    int clo = ok ? max(w.lo_t, 0) : INT_MAX, chi = ok ? min(w.lo_t + w.n_t, P.Nt) : 0;
#pragma unroll
    for (int k = 1; k < kCloseDepos; k <<= 1) {
        rlo = min(rlo, __shfl_xor(rlo, k, 64));
        rhi = max(rhi, __shfl_xor(rhi, k, 64));
        clo = min(clo, __shfl_xor(clo, k, 64));
        chi = max(chi, __shfl_xor(chi, k, 64));
    }
    const bool first = (lane & (kCloseDepos - 1)) == 0 && rlo < rhi && clo < chi;
    const bool fits = (int64_t)(rhi - rlo) * (chi - clo) <= kScatCells;
    const int close = __syncthreads_count(first && fits), apart = __syncthreads_count(first && !fits);
    if (threadIdx.x == 0 && close != apart)
        atomicAdd(&sums->close, close - apart);
}

template <int NT>
__device__ double block_sum_d(double v, double *red)
{
    v = seg_sum<64>(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0)
        red[wave] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k)
        s += red[k];
    return s;
}

// Window weights of one axis by a whole workgroup (any window up to
// kMaxWindow bins): erf at every edge into LDS, then differences and the sum.
template <int NT>
__device__ void block_axis_weights(int lo, int n, double mu, double s, float *W, double *E,
                                   double *red)
{
    for (int k = threadIdx.x; k <= n; k += NT)
        E[k] = (s > 0.0) ? edge_erf(lo, k, mu, s) : 0.0;
    __syncthreads();
    double part = 0.0;
    for (int i = threadIdx.x; i < n; i += NT)
        part += 0.5 * (E[i + 1] - E[i]);
    const double sum = block_sum_d<NT>(part, red);
    for (int i = threadIdx.x; i < n; i += NT)
        W[i] = (s > 0.0) ? (float)((0.5 * (E[i + 1] - E[i])) / sum) : (i == 0 ? 1.0f : 0.0f);
    __syncthreads();
}

// One workgroup per depo, any window size.  FLAT: write the patch at its
// offset in the flat value buffer.  Otherwise add it to the grid with float
// atomics (used for the few depos whose patch does not fit the LDS tiles).
// With fluctuation the rescaling needs the patch total before any value is
// final: FLAT stores the clamped draws and rescales them in place; the grid
// variant draws twice (same counters, same numbers).
template <int NT, bool FLAT, bool B>
__global__ __launch_bounds__(NT) void k_patch_generic(EventCtx e0, BatchTables bt,
                                                      const int32_t *index_list,
                                                      const int32_t *list_count, int64_t n_direct,
                                                      const int64_t *offsets, float *values)
{
    __shared__ float Wp[kMaxWindow], Wt[kMaxWindow];
    __shared__ double E[kMaxWindow + 1];
    __shared__ double red[NT / 64];
    const int64_t count = index_list ? (int64_t)*list_count : n_direct;
    for (int64_t k = blockIdx.x; k < count; k += gridDim.x) {
        const int gd = index_list ? index_list[k] : (int)k;
        const EventCtx &Ev = B ? bt.ev[find_event(bt.depo_base, bt.nev, gd)] : e0;
        const PlaneParams &P = Ev.kp;
        const uint32_t event = Ev.event;
        const gptr<float> grid = glb(Ev.grid);
        const int d = gd - (int)Ev.depo_base;  // index in the event's own depo array
        const wcsim_depo dep = glb(Ev.depos)[d];
        const Win w = depo_window(dep, P);
        if (w.status != 0)
            continue;
        block_axis_weights<NT>(w.lo_p, w.n_p, w.mu_p, w.s_p, Wp, E, red);
        block_axis_weights<NT>(w.lo_t, w.n_t, w.mu_t, w.s_t, Wt, E, red);
        const double qd = surviving_charge(w, P, d, event);
        const float qf = (float)qd;
        float *out = FLAT ? values + offsets[d] : nullptr;
        if (!P.fluct) {
            const int cnt = w.n_p * w.n_t;
            for (int it = threadIdx.x; it < cnt; it += NT) {
                const int i = it / w.n_t, j = it - i * w.n_t;
                const float v = qf * Wp[i] * Wt[j];
                if (FLAT) {
                    out[it] = v;
                } else {
                    const int I = w.lo_p + i, J = w.lo_t + j;
                    if ((unsigned)I < (unsigned)P.Np && (unsigned)J < (unsigned)P.Nt)
                        unsafeAtomicAdd(grid + (size_t)I * P.Nt + J, v);
                }
            }
        } else {
            const int qlo = quad_of(w.lo_t), nq = quad_of(w.lo_t + w.n_t - 1) - qlo + 1;
            const int items = w.n_p * nq;
            double S = 0.0;
            for (int it = threadIdx.x; it < items; it += NT) {
                const int i = it / nq, qd = qlo + (it - i * nq);
                const uint4 r = philox4x32_10(
                    make_uint4((uint32_t)qd, (uint32_t)(w.lo_p + i), (uint32_t)d, event), P.key0,
                    P.key1);
                float z[4];
                box_muller(r.x, r.y, z[0], z[1]);
                box_muller(r.z, r.w, z[2], z[3]);
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int j = 4 * qd + m - w.lo_t;
                    if (j >= 0 && j < w.n_t) {
                        const float F = fluct_value(qf, Wp[i] * Wt[j], z[m]);
                        S += (double)F;
                        if (FLAT)
                            out[i * w.n_t + j] = F;
                    }
                }
            }
            S = block_sum_d<NT>(S, red);
            const float scale = (S > 0.0) ? (float)(qd / S) : 0.0f;
            for (int it = threadIdx.x; it < items; it += NT) {
                const int i = it / nq, qd = qlo + (it - i * nq);
                float z[4];
                if (!FLAT) {
                    const uint4 r = philox4x32_10(
                        make_uint4((uint32_t)qd, (uint32_t)(w.lo_p + i), (uint32_t)d, event),
                        P.key0, P.key1);
                    box_muller(r.x, r.y, z[0], z[1]);
                    box_muller(r.z, r.w, z[2], z[3]);
                }
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const int j = 4 * qd + m - w.lo_t;
                    if (j >= 0 && j < w.n_t) {
                        const float p = Wp[i] * Wt[j];
                        if (FLAT) {
                            float &o = out[i * w.n_t + j];
                            o = (S > 0.0) ? o * scale : qf * p;
                        } else {
                            const int I = w.lo_p + i, J = w.lo_t + j;
                            if ((unsigned)I < (unsigned)P.Np && (unsigned)J < (unsigned)P.Nt) {
                                const float v =
                                    (S > 0.0) ? fluct_value(qf, p, z[m]) * scale : qf * p;
                                unsafeAtomicAdd(grid + (size_t)I * P.Nt + J, v);
                            }
                        }
                    }
                }
            }
        }
        if (gridDim.x == 1)
            __threadfence();  // one workgroup: this patch's adds complete before the next's
        __syncthreads();
    }
}

// floor(a / b) for 0 <= a < 4096 and 1 <= b <= 64 by a multiply-shift with
// m = ceil(2^20 / b): the error term a (m b - 2^20) / (b 2^20) stays below 1/b.
__device__ __forceinline__ int div_small(int a, int m) { return (int)(__umul24(a, m) >> 20); }
__device__ __forceinline__ int magic_small(int b) { return ((1 << 20) + b - 1) / b; }

// Flat patch set -> grid, bound by the rate of float atomics.  A wavefront takes `per`
// consecutive patches.  Plain: one patch, added bin by bin.  SUM: depos that follow
// one another mostly lie on one track and their patches share cells: when the bounding
// box of the wavefront's patches fits its LDS region it sums them there, one patch at a
// time (a patch's cells are distinct, and a wavefront's LDS accesses complete in
// order), and adds each touched cell to the grid once; patches that lie apart go to
// the grid bin by bin all the same.
// SUM is for sets of kScatMany depos or more most of whose neighbours lie together
// (k_patch_sizes counts that over 256 of each 2,048: PatchSums::close); `per` doubles from 4 to 16 while
// kScatFill wavefronts remain.  Plain / SUM with 4, 8, 16: tracks, 3,000 depos 9.6 / 8.1,
// 9.5, 17 us, 6,000 15 / 9.1, 11, 20, 30,000 57 / 21, 18, 28, 60,000 113 / 37, 31, 35,
// 100,000 174 / 56, 42, 41; uniform depos, 1,000 7.6 / 8.7, 13, 22, 30,000 44 / 47, 47,
// 48, 100,000 139 / 142, 143, 145; uniform with windows of 1,500 bins, 10,000 92 / 97,
// 114, 154.  (The workgroup's four wavefronts on one region by LDS atomics: 100,000
// track depos 95 us.)
constexpr int64_t kScatMany = 4096, kScatFill = 12288;
constexpr int kScatRegs = 4;
// wavefronts a workgroup
template <bool SUM>
constexpr int kScatWaves = SUM ? 1 : 4;

template <bool SUM>
__global__ __launch_bounds__(64 * kScatWaves<SUM>) void k_scatter_flat(
    int64_t n, int per, const int32_t *__restrict__ meta, const int64_t *__restrict__ offsets,
    const float *__restrict__ values, float *grid, int Np, int Nt)
{
    __shared__ float acc[SUM ? kScatCells : 1];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t d0 = (blockIdx.x * (int64_t)kScatWaves<SUM> + wave) * per;
    if (d0 >= n)
        return;
    const int K = (int)min((int64_t)per, n - d0);
    int4 win = make_int4(0, 0, 0, 0);
    int64_t off = 0;
    if (lane < K) {
        win = *(const int4 *)(meta + 4 * (d0 + lane));
        off = offsets[d0 + lane];
    }
    int rlo = 0, clo = 0, W = 1, cells = 0;  // the LDS region (cells = 0: none)
    if (SUM) {
        // bounding box of the patches' cells inside the grid
        const bool some = win.z > 0 && win.w > 0;
        rlo = wave_max_i<true>(some ? max(win.x, 0) : INT_MAX);
        clo = wave_max_i<true>(some ? max(win.y, 0) : INT_MAX);
        const int rhi = wave_max_i<false>(some ? min(win.x + win.z, Np) : INT_MIN);
        const int chi = wave_max_i<false>(some ? min(win.y + win.w, Nt) : INT_MIN);
        if (rlo >= rhi || clo >= chi)
            return;  // every patch is empty or outside the grid
        const int64_t w64 = (int64_t)chi - clo, cells64 = w64 * ((int64_t)rhi - rlo);
        W = (int)w64;
        cells = (int)(cells64 <= kScatCells ? cells64 : 0);
        for (int x = lane; x < cells; x += 64)
            acc[x] = 0.0f;
        wave_lds_sync();
    }
    for (int k = 0; k < K; ++k) {
        const int lo_p = __builtin_amdgcn_readlane(win.x, k), lo_t = __builtin_amdgcn_readlane(win.y, k);
        const int n_p = __builtin_amdgcn_readlane(win.z, k), n_t = __builtin_amdgcn_readlane(win.w, k);
        const int64_t o = ((int64_t)__builtin_amdgcn_readlane((int)(off >> 32), k) << 32) |
                          (uint32_t)__builtin_amdgcn_readlane((int)off, k);
        const float *v = values + o;
        const int cnt = n_p * n_t;
        const bool small = n_t <= 64 && cnt <= 4096;  // (what div_small takes)
        const int magic = small ? magic_small(max(n_t, 1)) : 0;
        for (int i0 = 0; i0 < cnt; i0 += 64 * kScatRegs) {
            float x[kScatRegs];
#pragma unroll
            for (int u = 0; u < kScatRegs; ++u)
                x[u] = v[min(i0 + 64 * u + lane, cnt - 1)];
#pragma unroll
            for (int u = 0; u < kScatRegs; ++u) {
                const int it = i0 + 64 * u + lane;
                if (it >= cnt)
                    break;
                const int i = small ? div_small(it, magic) : it / n_t, j = it - i * n_t;
                const int I = lo_p + i, J = lo_t + j;
                if ((unsigned)I < (unsigned)Np && (unsigned)J < (unsigned)Nt) {
                    if (SUM && cells > 0)
                        acc[(I - rlo) * W + (J - clo)] += x[u];
                    else
                        unsafeAtomicAdd(grid + (size_t)I * Nt + J, x[u]);
                }
            }
        }
        if (SUM)
            wave_lds_sync();  // the next patch may cover the same cells
    }
    for (int x = lane; SUM && x < cells; x += 64) {
        const float v = acc[x];
        const int r = x / W;
        if (v != 0.0f)
            unsafeAtomicAdd(grid + (size_t)(rlo + r) * Nt + clo + (x - r * W), v);
    }
}

// ---------------------------------------------------------------------------
// Fused path: tile binning and LDS-staged rasterization
// ---------------------------------------------------------------------------
constexpr int kHaloP = 32, kHaloT = 16;   // LDS region = tile + halo
constexpr int kRecP = kHaloP;             // longest pitch window of the tile path
constexpr int kRecT = kHaloT + 1;         // longest tick window of the tile path
constexpr int kRecQuads = (kRecT + 2) / 4 + 1;  // most tick quads such a window touches
constexpr int kRecWords = 64;             // floats per depo record (256 bytes)
constexpr int kRecWp = 8;                 // record offset of the pitch weights
constexpr int kRecWt = kRecWp + kRecP;    // record offset of the quad-aligned tick weights
static_assert(kRecWt % 4 == 0, "tick quads must be 16-byte aligned");
static_assert(kRecWt + 4 * kRecQuads <= kRecWords, "depo record overflow");
// Depos per tile work item (one wavefront).  Each work item flushes its own
// region cells with global atomics, and the regions of items sharing a track
// overlap, so longer chunks mean fewer atomics; at most 64, one window per
// lane for the bounding box.
constexpr int kChunk = 32;
static_assert(kChunk <= 64, "the chunk bounding box takes one patch window per lane");
constexpr int kFluctItems = 3;            // work items per lane held in registers
// A tile-path patch has at most kRecP * kRecQuads = 160 (row, quad) items.
static_assert(kRecP * kRecQuads <= 64 * kFluctItems, "patch items overflow");

struct TileGeom {
    int tp, tt, rp, rt, ntt;
};

__device__ __forceinline__ bool fits_tile(const Win &w, int p0, int t0, const TileGeom &g,
                                          const PlaneParams &P)
{
    if (w.n_p > kRecP || w.n_t > kRecT)
        return false;
    return min(w.lo_p + w.n_p, P.Np) <= p0 + g.rp && min(w.lo_t + w.n_t, P.Nt) <= t0 + g.rt;
}

// Mark the occupancy-map blocks that a window (status 0: it meets the grid)
// reaches.  Every writer stores the same value, so no atomics are needed.
__device__ __forceinline__ void mark_blocks(const Win &w, const PlaneParams &P, gptr<uint8_t> occ,
                                            int shift)
{
    const int p0 = max(w.lo_p, 0), p1 = min(w.lo_p + w.n_p, P.Np) - 1;
    const int t0 = max(w.lo_t, 0), t1 = min(w.lo_t + w.n_t, P.Nt) - 1;
    for (int b = p0 / kOccRows; b <= p1 / kOccRows; ++b)
        for (int c = t0 >> shift; c <= (t1 >> shift); ++c)
            occ[b * kOccCols + c] = 1;
}

// depo_tile of a depo whose patch does not fit a tile region (-1: no tile and
// no patch).
constexpr int32_t kTileLarge = -2;

// Window and tile of every depo.  Slots in a tile's list come from one atomic
// per distinct tile per wavefront (consecutive depos of a track share tiles).
// The atomics of a wavefront's tiles are issued together: a wavefront's time is
// the latency of one round trip and not of one per tile (1,000 uniform depos,
// up to 64 tiles a wavefront: 28.7 -> 7.1 us; 500,000 track depos 14.3 -> 12.0 us).
// Depos and tiles carry global indices: in a batch, depo gd belongs to the
// event whose depo_base range holds it, and tile numbers continue across
// events from each event's tile_base.
template <bool B>
__global__ __launch_bounds__(256) void k_prep_bin(EventCtx e0, BatchTables bt, int64_t ntotal,
                                                  TileGeom g, int32_t *counters,
                                                  int32_t *tile_count, int32_t *depo_tile,
                                                  int32_t *depo_slot, int32_t *large)
{
    const int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    int tile = -1;
    bool bad = false, big = false;
    if (d < ntotal) {
        const EventCtx &E = B ? bt.ev[find_event(bt.depo_base, bt.nev, (int)d)] : e0;
        const PlaneParams &P = E.kp;
        const int64_t dl = d - E.depo_base;
        // a batch reserves capacity per event; depos past its count are absent
        const Win w = (dl < E.n) ? depo_window(E.depos[dl], P) : Win{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 2};
        if (w.status == 1 || w.status == 3) {
            bad = true;
        } else if (w.status == 0) {
            mark_blocks(w, P, glb(E.occ), E.occ_shift);
            const int tp = min(max(w.lo_p, 0), P.Np - 1) / g.tp;
            const int tt = min(max(w.lo_t, 0), P.Nt - 1) / g.tt;
            if (fits_tile(w, tp * g.tp, tt * g.tt, g, P))
                tile = E.tile_base + tp * E.ntt + tt;
            else
                big = true;
        }
    }
    const uint64_t badm = __ballot(bad);
    if (lane == 0 && badm)
        atomicAdd(&counters[0], __popcll(badm));
    const uint64_t bigm = __ballot(big);
    if (bigm) {
        int base = 0;
        const int leader = __ffsll((unsigned long long)bigm) - 1;
        if (lane == leader)
            base = atomicAdd(&counters[1], __popcll(bigm));
        base = __shfl(base, leader);
        if (big)
            large[base + __popcll(bigm & lanemask_lt(lane))] = (int32_t)d;
    }
    // the lanes that share this lane's tile, one distinct tile at a time
    uint64_t mine = 0, active = __ballot(tile >= 0);
    while (active) {
        const int lt = __builtin_amdgcn_readlane(tile, __ffsll((unsigned long long)active) - 1);
        const uint64_t same = __ballot(tile == lt);
        if (tile == lt)
            mine = same;
        active &= ~same;
    }
    int slot = 0;
    if (tile >= 0 && (mine & lanemask_lt(lane)) == 0)
        slot = atomicAdd(&tile_count[tile], __popcll(mine));
    slot = __shfl(slot, mine ? __ffsll((unsigned long long)mine) - 1 : lane) +
           __popcll(mine & lanemask_lt(lane));
    if (d < ntotal) {
        depo_tile[d] = big ? kTileLarge : tile;
        depo_slot[d] = slot;
    }
}

// Tile schedule over blocks of kSchedTiles tiles: per-tile depo counts -> list
// offsets (in place) and the list of work items {tile, first record, end
// record, 0} of at most kChunk depos each.  counters[2] = number of work items.
// With float atomics (k_tile_schedule<false>) a block takes its place in both lists by
// one atomic, so the lists hold the blocks in the order they came; one launch.
// Reproducible sums need the lists in tile order (the scan of Sec. 4.3, ntiles +
// 1 exclusive offsets): block totals, their scan, then the same pass; three
// launches.  On the collection plane (225,000 tiles) 5.9 us against 16.8 us.
constexpr int kSchedThreads = 256, kSchedPer = 16, kSchedTiles = kSchedThreads * kSchedPer;
// Tiles a thread of the unordered lists, read four at a time: with 16 a plane's few
// blocks leave most CUs idle, with 4 the blocks of a batch queue at the one
// atomic.  4 / 8 / 16 tiles, 1000 x 1000 plane 3.3 / 3.6 / 4.4 us, 9600 x 6000 6.1 /
// 5.9 / 6.8, twelve such planes 25 / 18 / 17 (one word a load: 5.9, 8.1, 19).
constexpr int kListPer = 8;

__device__ __forceinline__ int chunks_of(int count) { return (count + kChunk - 1) / kChunk; }

// Block totals of depos and of work items.
__global__ __launch_bounds__(kSchedThreads) void k_tile_sums(const int32_t *tile_count, int ntiles,
                                                            int2 *block_tot)
{
    __shared__ int sh[kSchedThreads / 64];
    const int first = blockIdx.x * kSchedTiles + threadIdx.x * kSchedPer;
    int st = 0, sc = 0;
#pragma unroll
    for (int k = 0; k < kSchedPer; ++k) {
        const int idx = first + k;
        const int c = (idx < ntiles) ? tile_count[idx] : 0;
        st += c;
        sc += chunks_of(c);
    }
    int tot_t, tot_c;
    block_exclusive_scan<int>(st, sh, &tot_t);
    block_exclusive_scan<int>(sc, sh, &tot_c);
    if (threadIdx.x == 0)
        block_tot[blockIdx.x] = make_int2(tot_t, tot_c);
}

// Exclusive scan of the block totals in place (one workgroup), so that each
// schedule block reads its two bases with one load.
__global__ __launch_bounds__(kSchedThreads) void k_scan_block_tot(int2 *block_tot, int nb)
{
    __shared__ int sh[kSchedThreads / 64];
    int carry_t = 0, carry_c = 0;
    for (int b0 = 0; b0 < nb; b0 += kSchedThreads) {
        const int i = b0 + threadIdx.x;
        const int2 v = (i < nb) ? block_tot[i] : make_int2(0, 0);
        int tot_t, tot_c;
        const int ex_t = block_exclusive_scan<int>(v.x, sh, &tot_t);
        const int ex_c = block_exclusive_scan<int>(v.y, sh, &tot_c);
        if (i < nb)
            block_tot[i] = make_int2(ex_t + carry_t, ex_c + carry_c);
        carry_t += tot_t;
        carry_c += tot_c;
    }
}

// One block of tiles.  ORDERED: the block's bases come from the scanned totals;
// otherwise from one 64-bit atomic on counters[2] (low word: work items) and
// counters[3] (high word: depos), both below 2^31.
template <bool ORDERED>
__global__ __launch_bounds__(kSchedThreads) void k_tile_schedule(int32_t *tile_count, int ntiles,
                                                                const int2 *block_base,
                                                                int4 *items, int32_t *counters)
{
    __shared__ int sh[kSchedThreads / 64];
    __shared__ unsigned long long place;
    constexpr int PER = ORDERED ? kSchedPer : kListPer;
    const int first = (blockIdx.x * kSchedThreads + threadIdx.x) * PER;
    int cnt[PER];
    int st = 0, sc = 0;
#pragma unroll
    for (int k = 0; k < PER; k += 4) {
        int4 c = make_int4(0, 0, 0, 0);
        if (first + k + 3 < ntiles) {
            c = *(const int4 *)(tile_count + first + k);
        } else {
            c.x = (first + k < ntiles) ? tile_count[first + k] : 0;
            c.y = (first + k + 1 < ntiles) ? tile_count[first + k + 1] : 0;
            c.z = (first + k + 2 < ntiles) ? tile_count[first + k + 2] : 0;
        }
        cnt[k] = c.x;
        cnt[k + 1] = c.y;
        cnt[k + 2] = c.z;
        cnt[k + 3] = c.w;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        st += cnt[k];
        sc += chunks_of(cnt[k]);
    }
    int tot_t, tot_c;
    int off_t = block_exclusive_scan<int>(st, sh, &tot_t);
    int off_c = block_exclusive_scan<int>(sc, sh, &tot_c);
    if (ORDERED) {
        off_t += block_base[blockIdx.x].x;
        off_c += block_base[blockIdx.x].y;
    } else {
        if (tot_t == 0)
            return;  // no depo in the block: its offsets are never read
        if (threadIdx.x == 0)
            place = atomicAdd((unsigned long long *)(counters + 2),
                              ((unsigned long long)(uint32_t)tot_t << 32) | (uint32_t)tot_c);
        __syncthreads();
        off_t += (int)(place >> 32);
        off_c += (int)(uint32_t)place;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int idx = first + k;
        if (ORDERED ? idx <= ntiles : cnt[k] > 0)
            tile_count[idx] = off_t;
        const int nch = chunks_of(cnt[k]);
        for (int j = 0; j < nch; ++j) {
            const int b = off_t + j * kChunk;
            items[off_c + j] = make_int4(idx, b, min(b + kChunk, off_t + cnt[k]), 0);
        }
        off_t += cnt[k];
        off_c += nch;
    }
    if (ORDERED && blockIdx.x == gridDim.x - 1 && threadIdx.x == kSchedThreads - 1)
        counters[2] = off_c;
}

// ---------------------------------------------------------------------------
// Tile lists in depo order (reproducible sums).  The slots that binning takes
// by atomics order a tile's depos as the wavefronts happened to run; a stable
// least-significant-digit radix sort of the keys (tile; kTileLarge depos after
// the last tile; depos without a patch last) over the depo indices gives every
// depo its rank in its tile's list by index, and the large-patch list in index
// order.  Blocks of kSortBlock keys; one count / offsets / scatter triple per digit
// of 8 or 9 bits.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 256, kSortPer = 16, kSortBlock = kSortThreads * kSortPer;
static_assert(kSortThreads == kScanThreads, "the sort uses the block scan");

__global__ __launch_bounds__(256) void k_sort_keys(const int32_t *depo_tile, int64_t n,
                                                   uint32_t ntiles, uint32_t *keys,
                                                   int32_t *vals)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const int t = depo_tile[i];
    keys[i] = (t >= 0) ? (uint32_t)t : (t == kTileLarge ? ntiles : ntiles + 1u);
    vals[i] = (int32_t)i;
}

// counts[b][d]: keys of block b with digit d of BITS bits.
template <int BITS>
__global__ __launch_bounds__(kSortThreads) void k_sort_count(const uint32_t *keys, int64_t n,
                                                            int shift, int32_t *counts)
{
    constexpr int ND = 1 << BITS;
    __shared__ int hist[ND];
    const int tid = threadIdx.x;
#pragma unroll
    for (int d = tid; d < ND; d += kSortThreads)
        hist[d] = 0;
    __syncthreads();
    const int64_t b0 = blockIdx.x * (int64_t)kSortBlock;
#pragma unroll 4
    for (int k = 0; k < kSortPer; ++k) {
        const int64_t i = b0 + k * kSortThreads + tid;
        if (i < n)
            atomicAdd(&hist[(keys[i] >> shift) & (ND - 1)], 1);
    }
    __syncthreads();
#pragma unroll
    for (int d = tid; d < ND; d += kSortThreads)
        counts[(int64_t)blockIdx.x * ND + d] = hist[d];
}

// One workgroup, each thread PER neighbouring digits: the first output position
// of digit d in each block (the keys of smaller digits plus those of digit d in
// earlier blocks), in place.
template <int BITS>
__global__ __launch_bounds__(kSortThreads) void k_sort_offsets(int32_t *counts, int nblk)
{
    constexpr int ND = 1 << BITS, PER = ND / kSortThreads, U = 8;
    __shared__ int sh[kSortThreads / 64];
    int32_t *c0 = counts + PER * threadIdx.x;
    int tot[PER] = {}, all = 0;
    for (int b = 0; b < nblk; b += U) {
        int c[U][PER];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < PER; ++m)
                c[u][m] = (b + u < nblk) ? c0[(int64_t)(b + u) * ND + m] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < PER; ++m)
                tot[m] += c[u][m];
    }
#pragma unroll
    for (int m = 0; m < PER; ++m)
        all += tot[m];
    int total;
    int run[PER];
    run[0] = block_exclusive_scan<int>(all, sh, &total);
#pragma unroll
    for (int m = 1; m < PER; ++m)
        run[m] = run[m - 1] + tot[m - 1];
    for (int b = 0; b < nblk; b += U) {
        int c[U][PER];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < PER; ++m)
                c[u][m] = (b + u < nblk) ? c0[(int64_t)(b + u) * ND + m] : 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int m = 0; m < PER; ++m)
                if (b + u < nblk) {
                    c0[(int64_t)(b + u) * ND + m] = run[m];
                    run[m] += c[u][m];
                }
    }
}

// Stable scatter of one block: its keys are taken in rounds of kSortThreads
// consecutive keys; a key's position is its digit's next free slot plus the
// keys of the same digit before it in the round (earlier wavefronts, then
// lower lanes of its own).
template <int BITS>
__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const uint32_t *kin,
                                                              const int32_t *vin, int64_t n,
                                                              int shift, const int32_t *offsets,
                                                              uint32_t *kout, int32_t *vout)
{
    constexpr int NW = kSortThreads / 64, ND = 1 << BITS;
    __shared__ int next[ND];
    __shared__ int wcnt[NW][ND];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
    for (int d = tid; d < ND; d += kSortThreads) {
        next[d] = offsets[(int64_t)blockIdx.x * ND + d];
#pragma unroll
        for (int u = 0; u < NW; ++u)
            wcnt[u][d] = 0;
    }
    __syncthreads();
    const int64_t b0 = blockIdx.x * (int64_t)kSortBlock;
    for (int k = 0; k < kSortPer; ++k) {
        const int64_t i = b0 + k * kSortThreads + tid;
        const bool valid = i < n;
        const uint32_t key = valid ? kin[i] : 0u;
        const int32_t val = valid ? vin[i] : 0;
        const int dg = (int)((key >> shift) & (uint32_t)(ND - 1));
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int bit = 0; bit < BITS; ++bit) {
            const uint64_t m = __ballot((dg >> bit) & 1);
            same &= ((dg >> bit) & 1) ? m : ~m;
        }
        const int rank = __popcll(same & lanemask_lt(lane));
        if (valid && rank == 0)
            wcnt[w][dg] = __popcll(same);
        __syncthreads();
        if (valid) {
            int pos = next[dg] + rank;
            for (int u = 0; u < w; ++u)
                pos += wcnt[u][dg];
            kout[pos] = key;
            vout[pos] = val;
        }
        __syncthreads();  // every position is formed before the counts move on
#pragma unroll
        for (int d = tid; d < ND; d += kSortThreads) {
            int add = 0;
#pragma unroll
            for (int u = 0; u < NW; ++u) {
                add += wcnt[u][d];
                wcnt[u][d] = 0;
            }
            next[d] += add;
        }
        __syncthreads();
    }
}

// From the sorted keys: each tile-listed depo's slot (its rank in the tile's
// list) and the large-patch list in depo order.  tile_off: the tiles'
// exclusive list offsets, ntiles + 1 entries.
__global__ __launch_bounds__(256) void k_sort_slots(const uint32_t *keys, const int32_t *vals,
                                                    int64_t n, uint32_t ntiles,
                                                    const int32_t *tile_off, int32_t *depo_slot,
                                                    int32_t *large)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= n)
        return;
    const uint32_t key = keys[i];
    if (key < ntiles)
        depo_slot[vals[i]] = (int32_t)(i - tile_off[key]);
    else if (key == ntiles)
        large[i - tile_off[ntiles]] = vals[i];
}

// Weights of one axis computed by one thread into a record, in FP64: the
// Gaussian's integral over each bin, normalised by the window total, rounded
// once to float32.  The edge arguments are x_k = (lo + k - mu) / (sqrt(2) s);
// the integrals come from the complementary error function of |x_k|,
// c_k = erfc(|x_k|), with erf(x) = sign(x) (1 - c): a bin on one side of the
// centre is the difference c_a - c_b of two tail values (no cancellation of
// values near 1, so tail bins keep their full relative precision), a bin
// holding the centre is 2 - c_a - c_b.  The window total is the same
// difference taken between the window's outer edges.
// erfc(x) for x >= 0 in FP64 without branches: exp(-x^2) erfcx(x), with
// erfcx(x) = exp(x^2) erfc(x) a polynomial of degree 18 in
// u = 9 / (3 + x) - 2 (the interval [0, 6] of x mapped onto [-1, 1]).  The
// polynomial is a Chebyshev expansion fitted by weighted least squares at 300
// Chebyshev nodes in 40-digit arithmetic, turned into powers of u in 50-digit
// arithmetic; the magnitudes of its coefficients sum to 1.0003, so Horner's
// rule loses nothing to cancellation: at most 2e-15 relative to the library
// erfc on [0, 6].  Beyond x = 6 erfcx is held at its value at 6 (erfc(6) =
// 2.2e-17: the absolute error stays below 1e-17).  The library erfc branches
// over three ranges of x here, and the lanes of a wavefront take all three.
__constant__ const double kErfcxPoly[19] = {
    0.32158541645431749, 0.36815156489826012, 0.2014388568192258,
    0.081626845134045015, 0.023308261232626117, 0.003956151636291854,
    7.0125313652629907e-05, -0.00012716419781459492, -1.5153801949992285e-05,
    4.532602482660329e-06, 8.1181436388616683e-07, -2.2753363747095745e-07,
    -3.482226636786867e-08, 1.44452931474044e-08, 8.4853769242305189e-10,
    -9.2921436560768322e-10, 4.7966663774361644e-11, 4.402449211974955e-11,
    -6.2047195508566893e-12};

// 1 / d for d in [3, 9] (no scaling or special cases needed): the hardware
// reciprocal refined by two Newton steps, each squaring the relative error.
__device__ __forceinline__ double recip_3_9(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    return fma(r, fma(-d, r, 1.0), r);
}

__device__ __forceinline__ double erfc_tail(double x)
{
    const double u = fma(9.0, recip_3_9(3.0 + fmin(x, 6.0)), -2.0);
    double p = kErfcxPoly[18];
#pragma unroll
    for (int k = 17; k >= 0; --k)
        p = fma(p, u, kErfcxPoly[k]);
    return exp(-x * x) * p;
}

__device__ __forceinline__ double edge_tail(int lo, int k, double mu, double inv, bool &neg)
{
    const double x = ((double)(lo + k) - mu) * inv;
    neg = x < 0.0;
    return erfc_tail(fabs(x));
}

__device__ __forceinline__ double bin_integral(double ca, bool na, double cb, bool nb)
{
    // erf(b) - erf(a) for edges a < b
    if (!na)
        return ca - cb;
    if (nb)
        return cb - ca;
    return (2.0 - ca) - cb;
}

// `part` of `parts`: only the bins n part / parts .. n (part + 1) / parts - 1
// (the outer edges are evaluated by every part).
__device__ __forceinline__ void thread_axis_weights(int lo, int n, double mu, double s, float *W,
                                                    int part = 0, int parts = 1)
{
    if (s == 0.0) {
        if (part == 0)
            W[0] = 1.0f;
        return;
    }
    const double inv = 1.0 / (kSqrt2 * s);
    bool n0, nn;
    double c_lo = edge_tail(lo, 0, mu, inv, n0);
    const double c_n = edge_tail(lo, n, mu, inv, nn);
    const double rtot = 1.0 / bin_integral(c_lo, n0, c_n, nn);
    bool n_lo = n0;
    const int i0 = n * part / parts, i1 = n * (part + 1) / parts;
    if (i0 > 0 && i0 < i1)
        c_lo = edge_tail(lo, i0, mu, inv, n_lo);
    for (int i = i0; i < min(i1, n - 1); ++i) {
        bool n_hi;
        const double c_hi = edge_tail(lo, i + 1, mu, inv, n_hi);
        W[i] = (float)(bin_integral(c_lo, n_lo, c_hi, n_hi) * rtot);
        c_lo = c_hi;
        n_lo = n_hi;
    }
    if (i1 == n)
        W[n - 1] = (float)(bin_integral(c_lo, n_lo, c_n, nn) * rtot);  // the last edge is c_n
}

// Patch values of a patch set (flat, at the scanned offsets).  A wavefront takes
// `per` consecutive depos: lane k forms the window and charge of depo k,
// then the patches are drawn one after another.  Every lane evaluates one window
// edge (the pitch edges first, then the tick edges: erfc tails as in
// thread_axis_weights), the weights go through LDS, and the (row, tick quad)
// items of the patch are held in registers until its total is known.  Patches
// with more edges or items than that (beyond_wave) are left to
// k_patch_generic.  One workgroup per depo with its barriers, 16 KB of LDS and
// library erf took 283 us for 100,000 track depos, this 92 us (16 depos a
// wavefront 106 us, too few wavefronts; held to 80 registers 143 us).
// A patch is a chain of about 2 us, so a wavefront takes several only once the set
// has kWaveFill wavefronts of half as many (window and charge are then formed side by
// side).  Whole rasterize call with one / two / four / eight: 1,000 uniform depos 54 / 56
// / 59 / 65 us, 8,000 64 / 62 / 62 / 67, 16,000 75 / 71 / 69 / 72, 100,000 185 / 154 /
// 141 / 139.
constexpr int kWavePatches = 8;
constexpr int64_t kWaveFill = 4096;
constexpr int kWaveWt = 64, kWaveWords = kWaveWt + 72;  // pitch weights, quad-aligned tick weights

template <bool FLUCT>
__global__ __launch_bounds__(256) void k_patch_wave(const wcsim_depo *__restrict__ depos, int64_t n,
                                                    PlaneParams P, uint32_t event, int per,
                                                    const int64_t *__restrict__ offsets,
                                                    float *__restrict__ values)
{
    __shared__ float4 weights[4][kWaveWords / 4];
    const int lane = threadIdx.x & 63;
    float *wl = (float *)weights[threadIdx.x >> 6];
    const int64_t d0 = (blockIdx.x * 4LL + (threadIdx.x >> 6)) * per;
    if (d0 >= n)
        return;
    const int K = (int)min((int64_t)per, n - d0);
    Win w{};
    w.status = 2;
    double qs = 0.0;
    int64_t off = 0;
    if (lane < K) {
        w = depo_window(depos[d0 + lane], P);
        if (w.status == 0) {
            qs = surviving_charge(w, P, (int)(d0 + lane), event);
            off = offsets[d0 + lane];
        }
    }
    // edge scale 1 / (sqrt(2) s), 0 for a zero width (one bin of weight 1)
    const double inv_p = (w.s_p > 0.0) ? 1.0 / (kSqrt2 * w.s_p) : 0.0;
    const double inv_t = (w.s_t > 0.0) ? 1.0 / (kSqrt2 * w.s_t) : 0.0;
    uint64_t todo = __ballot(w.status == 0 && !beyond_wave(w));
    while (todo) {
        const int k = __ffsll((unsigned long long)todo) - 1;
        todo &= todo - 1;
        const int lo_p = __builtin_amdgcn_readlane(w.lo_p, k);
        const int lo_t = __builtin_amdgcn_readlane(w.lo_t, k);
        const int n_p = __builtin_amdgcn_readlane(w.n_p, k);
        const int n_t = __builtin_amdgcn_readlane(w.n_t, k);
        const double q = readlane_d(qs, k);
        const int qlo = quad_of(lo_t), nq = quad_of(lo_t + n_t - 1) - qlo + 1;
        // weights: lane e <= n_p holds pitch edge e, the lanes behind it the ticks'
        const double mu_p = readlane_d(w.mu_p, k), mu_t = readlane_d(w.mu_t, k);
        const double ip = readlane_d(inv_p, k), it = readlane_d(inv_t, k);
        const bool tick = lane > n_p;
        const int e = tick ? lane - n_p - 1 : lane, ne = tick ? n_t : n_p;
        const double inv = tick ? it : ip;
        bool neg;
        const double c = edge_tail(tick ? lo_t : lo_p, min(e, ne), tick ? mu_t : mu_p, inv, neg);
        const double c_hi = dpp_shift_d<0x130, 0xf>(c);  // wave_shl:1
        const uint64_t negm = __ballot(neg);
        const int t0 = n_p + 1, t1 = t0 + n_t;  // lanes of the first and last tick edge
        const double tot =
            tick ? bin_integral(readlane_d(c, t0), (negm >> t0) & 1, readlane_d(c, t1),
                                (negm >> t1) & 1)
                 : bin_integral(readlane_d(c, 0), negm & 1, readlane_d(c, n_p), (negm >> n_p) & 1);
        const float wgt = (inv > 0.0) ? (float)div_pos_d(bin_integral(c, neg, c_hi,
                                                                      (negm >> lane >> 1) & 1),
                                                         tot)
                                      : 1.0f;
        wave_lds_sync();  // the previous patch's weights have been read
        for (int x = lane; x < 4 * nq; x += 64)
            wl[kWaveWt + x] = 0.0f;
        wave_lds_sync();
        if (e < ne)
            wl[tick ? kWaveWt + (lo_t & 3) + e : e] = wgt;
        wave_lds_sync();
        const float qf = (float)q;
        const int items = n_p * nq, magic = magic_small(nq);
        float *out = values + ((int64_t)__builtin_amdgcn_readlane((int)(off >> 32), k) << 32 |
                               (uint32_t)__builtin_amdgcn_readlane((int)off, k));
        float F[kWaveItems][4];
        double S = 0.0;
#pragma unroll
        for (int b = 0; b < kWaveItems; ++b) {
            if (64 * b >= items)
                break;
            const int x = min(64 * b + lane, items - 1);
            const int i = div_small(x, magic), qq = x - i * nq;
            const float wp = wl[i];
            const float4 wt = *(const float4 *)(wl + kWaveWt + 4 * qq);
            const float w4[4] = {wt.x, wt.y, wt.z, wt.w};
            if constexpr (FLUCT) {
                const uint4 r = philox4x32_10(
                    make_uint4((uint32_t)(qlo + qq), (uint32_t)(lo_p + i), (uint32_t)(d0 + k),
                               event),
                    P.key0, P.key1);
                constexpr float kMinus2Ln2 = -1.38629436111989061883f;
                const float ra = kMinus2Ln2 * __builtin_amdgcn_logf(word_to_uniform(r.x));
                const float rb = kMinus2Ln2 * __builtin_amdgcn_logf(word_to_uniform(r.z));
                const float ua = word_to_uniform(r.y), ub = word_to_uniform(r.w);
                const float r2[4] = {ra, ra, rb, rb};
                const float cs[4] = {__builtin_amdgcn_cosf(ua), __builtin_amdgcn_sinf(ua),
                                     __builtin_amdgcn_cosf(ub), __builtin_amdgcn_sinf(ub)};
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    F[b][m] = fluct_value_r2(qf, wp * w4[m], r2[m], cs[m]);
                if (64 * b + lane < items)
                    S += ((double)F[b][0] + (double)F[b][1]) + ((double)F[b][2] + (double)F[b][3]);
            } else {
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    F[b][m] = qf * (wp * w4[m]);
            }
        }
        float scale = 1.0f;
        if constexpr (FLUCT) {
            S = readlane_d(wave_incl_scan_d(S), 63);
            scale = (S > 0.0) ? (float)div_pos_d(q, S) : -1.0f;
        }
#pragma unroll
        for (int b = 0; b < kWaveItems; ++b) {
            const int x = 64 * b + lane;
            if (x >= items)
                break;
            const int i = div_small(x, magic), qq = x - i * nq;
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const int j = 4 * (qlo + qq) + m - lo_t;
                // (rare: a patch whose draws are all zero keeps its mean)
                const float v = (scale >= 0.0f) ? F[b][m] * scale
                                                : qf * (wl[i] * wl[kWaveWt + 4 * qq + m]);
                if (j >= 0 && j < n_t)
                    out[i * n_t + j] = v;
            }
        }
    }
}

// Depo records in tile-list order.  Header words: lo_p, lo_t, n_p, n_t, depo
// index, charge (FP64, two words) and the division magic of the tick quad
// count; then
// the pitch weights, and the tick weights placed by tick quad: entry
// 4 (floor(J / 4) - floor(lo_t / 4)) + J mod 4 holds the weight of tick J, and
// the entries of the first and last quad outside the window hold zero.
enum { kHLoP, kHLoT, kHNp, kHNt, kHDepo, kHQlo, kHQhi, kHMq, kHeaderWords };
static_assert(kHeaderWords <= kRecWp, "record header overflow");
constexpr int kStageStride = kRecWords + 1;  // odd: one LDS bank per lane

// Zero the blocks of one band of kOccRows grid rows whose bits are set in
// `m` (bit c: ticks c 2^shift .. (c + 1) 2^shift - 1), by one wavefront.  A
// block's row is a power of two of words long, so a lane's row and column are
// shifts of its index (a division per store cost a fifth of this loop).
__device__ __forceinline__ void clear_blocks(gptr<float> grid, int Np, int Nt, int band,
                                             uint64_t m, int shift, int lane)
{
    const int r0 = band * kOccRows, nr = min(kOccRows, Np - r0);
    const gptr<float> base = grid + (int64_t)r0 * Nt;
    while (m) {
        const int c0 = (__ffsll((unsigned long long)m) - 1) << shift;
        m &= m - 1;
        if ((Nt & 3) == 0) {  // rows of whole float4 words
            for (int i = lane; i < nr << (shift - 2); i += 64) {
                const int r = i >> (shift - 2), c = c0 + 4 * (i & ((1 << (shift - 2)) - 1));
                if (c < Nt)
                    *(gptr<float4>)(base + (int64_t)r * Nt + c) =
                        make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        } else {
            for (int i = lane; i < nr << shift; i += 64) {
                const int r = i >> shift, c = c0 + (i & ((1 << shift) - 1));
                if (c < Nt)
                    base[(int64_t)r * Nt + c] = 0.0f;
            }
        }
    }
}

// NW wavefronts per block of 64 depos: lane l of the last computes depo l's
// header, charge and tick weights into LDS, lane l of the others its pitch
// weights in NW - 1 parts (several FP64 chains per depo in flight for the same
// LDS), then the block writes the records out one 256-byte row at a time.  The
// first `nclr` blocks instead clear the occupied blocks of the grids, one part of
// a band of kOccRows rows per wavefront at a time (nbands bands over all events):
// the clear is bound by HBM writes and the records by FP64 arithmetic, so one
// launch runs both side by side.
template <bool B, int NW>
__global__ __launch_bounds__(64 * NW) void k_fill_records(EventCtx e0, BatchTables bt, int64_t ntotal,
                                                     const int32_t *depo_tile,
                                                     const int32_t *depo_slot,
                                                     const int32_t *tile_off, float *records,
                                                     int nbands, int nclr, int parts_shift)
{
    __shared__ float stage[64 * kStageStride];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if ((int)blockIdx.x < nclr) {
        for (int u = NW * blockIdx.x + wv; u < nbands << parts_shift; u += NW * nclr) {
            const int gb = u >> parts_shift, part = u & ((1 << parts_shift) - 1);
            const int e = B ? find_event(bt.band_base, bt.nev, gb) : 0;
            const EventCtx &E = B ? bt.ev[e] : e0;
            const int band = B ? gb - bt.band_base[e] : gb;
            const bool mine = (lane >> (6 - parts_shift)) == part;
            const uint64_t m = __ballot(mine && glb(E.occ)[band * kOccCols + lane] != 0);
            clear_blocks(glb(E.grid), E.kp.Np, E.kp.Nt, band, m, E.occ_shift, lane);
        }
        return;
    }
    const int64_t gd = (blockIdx.x - nclr) * (int64_t)64 + lane;
    int pos = -1;
    const int t = (gd < ntotal) ? depo_tile[gd] : -1;
    if (t >= 0) {
        const EventCtx &E = B ? bt.ev[find_event(bt.depo_base, bt.nev, (int)gd)] : e0;
        const int64_t d = gd - E.depo_base;  // index in the event's own depo array
        pos = tile_off[t] + depo_slot[gd];
        const Win w = depo_window(E.depos[d], E.kp);
        float *rec = stage + lane * kStageStride;
        int *h = (int *)rec;
        const int off = w.lo_t & 3;
        const int nq = quad_of(w.lo_t + w.n_t - 1) - quad_of(w.lo_t) + 1;
        if (wv < NW - 1) {
            thread_axis_weights(w.lo_p, w.n_p, w.mu_p, w.s_p, rec + kRecWp, wv, NW - 1);
        } else {
            h[kHLoP] = w.lo_p;
            h[kHLoT] = w.lo_t;
            h[kHNp] = w.n_p;
            h[kHNt] = w.n_t;
            h[kHDepo] = (int)d;
            const double qs = surviving_charge(w, E.kp, (int)d, E.event);
            h[kHQlo] = (int)(uint32_t)__double_as_longlong(qs);
            h[kHQhi] = (int)(uint32_t)((uint64_t)__double_as_longlong(qs) >> 32);
            h[kHMq] = magic_small(nq);
            float *Wt = rec + kRecWt;
            for (int k = 0; k < off; ++k)
                Wt[k] = 0.0f;
            for (int k = off + w.n_t; k < 4 * nq; ++k)
                Wt[k] = 0.0f;
            thread_axis_weights(w.lo_t, w.n_t, w.mu_t, w.s_t, Wt + off);
        }
    }
    __syncthreads();
    for (int r = wv; r < 64; r += NW) {
        const int pr = __builtin_amdgcn_readlane(pos, r);
        if (pr >= 0)
            records[(int64_t)pr * kRecWords + lane] = stage[r * kStageStride + lane];
    }
}

// Region columns start at the tile's first tick (a multiple of four) and rows
// are a multiple of four floats, so that a tick quad (four ticks 4k .. 4k + 3,
// the unit one Philox block covers) is one aligned 16-byte LDS access.  A
// window starts inside its tile and spans at most kHaloT + 1 ticks, so its
// last quad ends before column TT + kHaloT.  A quad's ticks outside the window
// carry weight zero, hence deposit zero; quads before tick 0 (windows of the
// first tile that start before the grid) are dropped, and cells outside the
// grid are never flushed.
template <int TT>
constexpr int region_cols()
{
    return TT + kHaloT;
}

// Patches per batch of items: consecutive patches of a work item whose (row,
// tick quad) items number at most kBatchItems are drawn together, their
// items laid out flat over kBatchItems / 64 passes of the wavefront, so that
// the lanes of a pass serve several small patches instead of one.
constexpr int kBatchItems = 64 * kFluctItems;

// One wavefront per work item (tile, chunk of <= kChunk depos), rasterizing
// its patches into its own LDS copy of the tile region (tile + halo).  The
// patches are taken in batches of consecutive patches whose (row, tick quad)
// items fit kFluctItems passes of 64 lanes; the items of a batch are laid out
// flat (patch after patch), each lane finds its item's patch from the
// patches' item offsets, reads the patch's header from the lane that holds it
// (lane k holds patch k) and its weights from the depo record.  With
// fluctuation every item's four values are added, in FP64, to its patch's
// total in LDS; once the batch is drawn, each patch's factor q / S is formed
// in FP64 by the lane holding it, and every value is rescaled and deposited.
// The bins of one patch are distinct, so depositing the batch one patch at a
// time makes every deposit a plain read-add-write LDS access (two patches of
// a batch may cover the same cell).  No other wavefront touches the region.
// The region's non-zero cells are then added to the grid with float atomics.
// OWN: the caller clears the whole region before the tile's first item and
// flushes it after the last (the owner flush); the item neither clears nor
// flushes.
template <int TP, int TT, bool B, bool FLUCT, bool OWN = false>
__device__ __forceinline__ void raster_item(float4 *acc4, double *xsum, const int4 item,
                                            const float *__restrict__ records,
                                            const EventCtx &e0, const BatchTables &bt)
{
    constexpr int RT = region_cols<TT>();
    constexpr int RP = TP + kHaloP;
    const int tile = item.x, beg = item.y, end = item.z;
    const int K = end - beg;  // patches of the work item (<= kChunk)
    const int lane = threadIdx.x & 63;  // the item's wavefront (one of OWN's workgroup)
    // lane k < K holds the header of patch k: window, depo index, charge
    int4 win = make_int4(INT_MAX, INT_MAX, 0, 0), hdr = make_int4(0, 0, 0, 0);
    if (lane < K) {
        const int4 *rec = (const int4 *)(records + (int64_t)(beg + lane) * kRecWords);
        win = rec[0];  // lo_p lo_t n_p n_t
        hdr = rec[1];  // depo, q low word, q high word, quad-count magic
    }
    const EventCtx &E = B ? bt.ev[find_event(bt.tile_base, bt.nev, tile)] : e0;
    const PlaneParams P = E.kp;
    const int local = tile - E.tile_base;
    const int p0 = (local / E.ntt) * TP, t0 = (local % E.ntt) * TT;
    const int c0 = t0;  // grid tick of region column 0
    // Only the bounding box of the chunk's patches (in region rows and tick
    // quads, within the grid) is cleared and flushed; deposits outside the
    // grid land outside it and are never read.
    const int rlo = wave_max_i<true>(win.x);
    const int rhi = wave_max_i<false>((win.z > 0) ? win.x + win.z : INT_MIN);
    const int qlo = wave_max_i<true>(quad_of(win.y));
    const int qhi = wave_max_i<false>((win.z > 0) ? quad_of(win.y + win.w - 1) + 1 : INT_MIN);
    const int br0 = max(rlo, p0) - p0;
    const int br1 = min(min(rhi, (int)P.Np), p0 + RP) - p0;
    const int bq0 = max(4 * max(qlo, 0) - c0, 0) >> 2;
    const int bq1 = min(4 * min(qhi, quad_of((int)P.Nt - 1) + 1) - c0, RT) >> 2;
    const int bnq = max(bq1 - bq0, 0), bcells = max(br1 - br0, 0) * bnq;
    const int bmagic = magic_small(max(bnq, 1));
    for (int x = lane; x < (OWN ? 0 : bcells); x += 64) {
        const int r = div_small(x, bmagic);
        acc4[r * (RT / 4) + bq0 + br0 * (RT / 4) + (x - r * bnq)] =
            make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    // per-patch item counts and their inclusive prefix over the lanes
    const int pqlo = quad_of(win.y);
    const int pnq = (lane < K) ? quad_of(win.y + win.w - 1) - pqlo + 1 : 0;
    const int pitems = (lane < K) ? win.z * pnq : 0;
    const int incl = wave_incl_scan_i(pitems);
    // records of the item: 32-bit offsets from here
    const gptr<const float> item_rec = glb(records) + (int64_t)beg * kRecWords;
    const double pq = __longlong_as_double(
        (long long)(((uint64_t)(uint32_t)hdr.z << 32) | (uint32_t)hdr.y));  // patch charge, FP64
    const float pqf = (float)pq;

    wave_lds_sync();  // the cleared region is visible to every lane

    int kb = 0;  // first patch of the batch (uniform)
    while (kb < K) {
        const int base = __builtin_amdgcn_readlane(incl - pitems, kb);
        // the batch: patches kb .. ke, the longest run whose items fit
        const uint64_t fits = __ballot(lane >= kb && lane < K && incl - base <= kBatchItems);
        const int ke = 63 - __builtin_clzll(fits);
        const int nitems = __builtin_amdgcn_readlane(incl, ke) - base;
        const int npass = (nitems + 63) >> 6;
        float F[kFluctItems][4];
        int cell[kFluctItems], kk[kFluctItems];
        double carry = 0.0;  // total of the batch's earlier passes (uniform)
        // each item's patch: kb plus the patch ends at or below its flat index
        // (one pass over the batch's patch ends serves the lane's items)
#pragma unroll
        for (int b = 0; b < kFluctItems; ++b)
            kk[b] = kb;
        for (int j = kb; j < ke; ++j) {
            const int e = __builtin_amdgcn_readlane(incl, j) - base;
#pragma unroll
            for (int b = 0; b < kFluctItems; ++b)
                kk[b] += (64 * b + lane >= e) ? 1 : 0;
        }
#pragma unroll
        for (int b = 0; b < kFluctItems; ++b) {
            cell[b] = -1;
            if (b < npass) {
                const int g = 64 * b + lane;  // flat item index within the batch
                const bool valid = g < nitems;
                const int k = kk[b];
                // the patch's header, from the lane holding it
                const int lo_p = __shfl(win.x, k, 64), lo_t = __shfl(win.y, k, 64);
                const int d = __shfl(hdr.x, k, 64), m = __shfl(hdr.w, k, 64);
                const int nq = __shfl(pnq, k, 64);
                const int first = __shfl(incl - pitems, k, 64) - base;
                const float q = __shfl(pqf, k, 64);
                const int it = valid ? g - first : 0;
                const int i = div_small(it, m);
                const int qq = it - (int)__umul24(i, nq);
                const int qd = quad_of(lo_t) + qq;
                const int r = lo_p + i - p0, c = 4 * qd - c0;
                cell[b] = (valid && (unsigned)r < (unsigned)RP && (unsigned)c <= (unsigned)(RT - 4))
                              ? (r * RT + c) >> 2
                              : -1;
                // loaded by every lane (a surplus one reads its batch's last
                // patch): a branch around the loads would make each pass wait
                // for them before its Philox rounds
                const float wpl = item_rec[(uint32_t)(k * kRecWords + kRecWp + i)];
                const float4 wt =
                    *(gptr<const float4>)(item_rec + (uint32_t)(k * kRecWords + kRecWt + 4 * qq));
                const float w4[4] = {wt.x, wt.y, wt.z, wt.w};
                if constexpr (FLUCT) {
                    const uint4 rr = philox4x32_10(
                        make_uint4((uint32_t)qd, (uint32_t)(lo_p + i), (uint32_t)d, E.event),
                        P.key0, P.key1);
                    const float wp = valid ? wpl : 0.0f;
                    constexpr float kMinus2Ln2 = -1.38629436111989061883f;
                    const float r2a = kMinus2Ln2 * __builtin_amdgcn_logf(word_to_uniform(rr.x));
                    const float r2b = kMinus2Ln2 * __builtin_amdgcn_logf(word_to_uniform(rr.z));
                    const float ua = word_to_uniform(rr.y), ub = word_to_uniform(rr.w);
                    const float r2[4] = {r2a, r2a, r2b, r2b};
                    const float c[4] = {__builtin_amdgcn_cosf(ua), __builtin_amdgcn_sinf(ua),
                                        __builtin_amdgcn_cosf(ub), __builtin_amdgcn_sinf(ub)};
#pragma unroll
                    for (int mm = 0; mm < 4; ++mm)
                        F[b][mm] = fluct_value_r2(q, wp * w4[mm], r2[mm], c[mm]);
                    // the item's total in FP64, and its prefix over the batch
                    const double t = valid ? ((double)F[b][0] + (double)F[b][1]) +
                                                 ((double)F[b][2] + (double)F[b][3])
                                           : 0.0;
                    const double x = wave_incl_scan_d(t) + carry;
                    xsum[g] = x;
                    carry = readlane_d(x, 63);
                } else {
                    const float wp = valid ? wpl : 0.0f;
#pragma unroll
                    for (int mm = 0; mm < 4; ++mm)
                        F[b][mm] = q * (wp * w4[mm]);
                }
            }
        }
        if constexpr (FLUCT) {
            // the lane of each patch of the batch forms its total S as the
            // difference of the prefix sums at its last item and before its
            // first, and its factor q / S, in FP64 (negative when the clamped
            // total is zero: the patch keeps its mean)
            wave_lds_sync();
            float scale = 0.0f;
            if (lane >= kb && lane <= ke) {
                const int s0 = incl - pitems - base, s1 = incl - base;
                const double S = xsum[s1 - 1] - (s0 > 0 ? xsum[s0 - 1] : 0.0);
                scale = (S > 0.0) ? (float)div_pos_d(pq, S) : -1.0f;
            }
            wave_lds_sync();  // the next batch may overwrite the prefix sums
            // Rare: every fluctuated bin of a patch is zero.  The wavefront
            // takes this branch together: the lane holding a patch's header may
            // have no item of its own (a shuffle's source lane has to be active).
            const bool mean = __any(scale < 0.0f);
#pragma unroll
            for (int b = 0; b < kFluctItems; ++b) {
                const float sc = __shfl(scale, kk[b], 64);
                if (mean) {
                    const int k = kk[b];
                    const int first = __shfl(incl - pitems, k, 64) - base;
                    const int m = __shfl(hdr.w, k, 64), nq = __shfl(pnq, k, 64);
                    const float q = __shfl(pqf, k, 64);
                    if (b < npass && cell[b] >= 0 && sc < 0.0f) {
                        const int it = 64 * b + lane - first;
                        const int i = div_small(it, m);
                        const int qq = it - (int)__umul24(i, nq);
                        const float *rec = records + (int64_t)(beg + k) * kRecWords;
                        const float wp = rec[kRecWp + i];
                        const float4 wt = *(const float4 *)(rec + kRecWt + 4 * qq);
                        F[b][0] = -(q * (wp * wt.x));
                        F[b][1] = -(q * (wp * wt.y));
                        F[b][2] = -(q * (wp * wt.z));
                        F[b][3] = -(q * (wp * wt.w));
                    }
                }
                // (a scale of -1 turns the negated mean back)
#pragma unroll
                for (int mm = 0; mm < 4; ++mm)
                    F[b][mm] *= sc;
            }
        }
        // Deposit, one patch of the batch at a time: the bins of one patch are
        // distinct, but two patches of a batch may share cells.  A wavefront's
        // LDS accesses complete in program order, so each round reads what the
        // previous one wrote.
        for (int k = kb; k <= ke; ++k) {
#pragma unroll
            for (int b = 0; b < kFluctItems; ++b) {
                if (b < npass && cell[b] >= 0 && kk[b] == k) {
                    float4 a4 = acc4[cell[b]];
                    a4.x += F[b][0];
                    a4.y += F[b][1];
                    a4.z += F[b][2];
                    a4.w += F[b][3];
                    acc4[cell[b]] = a4;
                }
            }
        }
        kb = ke + 1;
    }
    wave_lds_sync();  // every deposit lands before the flush reads the region
    if constexpr (OWN)
        return;
    // Flush: consecutive lanes take consecutive ticks of a row, so that one
    // atomic instruction covers 256 contiguous bytes (few L2 lines) rather
    // than 16-byte pieces of many lines.
    const gptr<float> grid = glb(E.grid);
    const float *acc = (const float *)acc4;
    const int W = 4 * bnq;  // floats per bounding-box row
    const int nrows = max(br1 - br0, 0);
    auto flush_one = [&](int r, int col) {
        const float v = acc[(br0 + r) * RT + 4 * bq0 + col];
        const int J = c0 + 4 * bq0 + col;
        if (v != 0.0f && (unsigned)J < (unsigned)P.Nt)
            unsafeAtomicAdd(grid + (size_t)(p0 + br0 + r) * P.Nt + J, v);
    };
    if (W > 0 && W <= 64) {
        const int per = 64 / W, r_l = lane / W, col = lane - r_l * W;
        if (r_l < per)
            for (int r = r_l; r < nrows; r += per)
                flush_one(r, col);
    } else if (W > 64) {
        for (int r = 0; r < nrows; ++r)
            for (int col = lane; col < W; col += 64)
                flush_one(r, col);
    }
}

// FLUCT: the planes fluctuate (a template argument, so that no branch on it
// separates a pass's weight loads from the Philox rounds that need no weight).
template <int TP, int TT, bool B, bool FLUCT>
__global__ __launch_bounds__(64) void k_raster_tiles(const float *__restrict__ records,
                                                     const int4 *__restrict__ items,
                                                     const int32_t *__restrict__ counters,
                                                     EventCtx e0, BatchTables bt)
{
    constexpr int RP = TP + kHaloP, RT = region_cols<TT>();
    static_assert(RT % 4 == 0, "region rows must hold whole quads");
    __shared__ float4 acc4[RP * RT / 4];
    __shared__ double xsum[kBatchItems];  // prefix sums of a batch's fluctuated item totals
    // The launch has at most as many wavefronts as a typical work list has
    // items (the count is known only on the device); a wavefront takes items
    // blockIdx.x, + gridDim.x, ... so that every item is drawn.
    const int nitems_all = counters[2];
    for (int itm = blockIdx.x; itm < nitems_all; itm += gridDim.x)
        raster_item<TP, TT, B, FLUCT>(acc4, xsum, items[itm], records, e0, bt);
}

// Owner flush (reproducible sums).  Tiles are coloured by (tile row mod CP,
// tile column mod CT), with CP TP >= RP and CT TT >= RT, so that the LDS
// regions of two tiles of one colour never share a grid cell; one launch per
// colour, in a fixed order.  In a launch each tile of the colour is owned by one
// workgroup or one wavefront.  Light tiles (at most kLightItems work items) go to
// a wavefront each, which draws their items one after another into its region and
// adds the region to the grid with plain read-add-writes.  Heavy tiles -- a track
// nearly along the wires leaves most of its 2,500 depos, 78 work items, in a few
// tiles, and set the time of a phase -- go to a workgroup of kOwnerWaves
// wavefronts: wavefront w draws items w, w + kOwnerWaves, ... into its own copy of
// the region, and the workgroup adds the sum of the copies.  Every cell receives
// its sums in the same order on every run.  The launch is persistent over the
// colour's lists (the items that open the tiles), heavy tiles first.
// Whole events, four sets of 150,000 track depos on 480 wires: 660-1490 us with
// two wavefronts for every tile, 570-740 us so; 500,000 depos on 960 wires
// 1310-2180 and 1100-1240 us.  (Two items a light tile: 670-890 us; eight
// wavefronts a heavy one 570-680 and 1160-1250 us, four 570-900 and 1040-1340.)
constexpr int kOwnerWaves = 6, kLightItems = 1;
// counters: tiles per list, places handed out; lists: colour c's heavy tiles at
// 2 c, its light tiles at 2 c + 1
constexpr int kMaxColours = 9;
constexpr int kColourCount = 4, kColourNext = kColourCount + 2 * kMaxColours;

template <int TP, int TT>
constexpr int owner_colours_p()
{
    return (TP + kHaloP + TP - 1) / TP;
}
template <int TT>
constexpr int owner_colours_t()
{
    return (region_cols<TT>() + TT - 1) / TT;
}

// Add a complete region to the grid (NT threads, exclusive owners of the region's
// cells): quads wholly inside the grid as 16-byte
// read-add-writes when rows are whole float4 words, the others cell by cell.
// The region is the sum of the NW wavefronts' copies, taken in wavefront
// order.  Each thread's grid values are all loaded before any is stored, so
// that the loads are in flight together.
template <int RP, int RT, int NW, int NT>
__device__ __forceinline__ void owner_flush(const float4 *acc4, gptr<float> grid, int Np, int Nt,
                                            int p0, int c0, int tid)
{
    constexpr int RQ = RT / 4, NQ = (RP * RQ + NT - 1) / NT;
    const bool vec = (Nt & 3) == 0;
    float4 a[NQ], g[NQ];
    int64_t off[NQ];
    bool whole[NQ], any[NQ];
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int x = tid + NT * u;
        const int r = x / RQ, q = x - r * RQ;
        const int I = p0 + r, J = c0 + 4 * q;
        const bool in = x < RP * RQ && I < Np && J < Nt;
        a[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (in) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const float4 v = acc4[w * RP * RQ + x];
                a[u] = make_float4(a[u].x + v.x, a[u].y + v.y, a[u].z + v.z, a[u].w + v.w);
            }
        }
        any[u] = in && (a[u].x != 0.0f || a[u].y != 0.0f || a[u].z != 0.0f || a[u].w != 0.0f);
        whole[u] = vec && J + 3 < Nt;
        off[u] = (int64_t)I * Nt + J;
        g[u] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if (any[u] && whole[u])
            g[u] = *(const gptr<float4>)(grid + off[u]);
    }
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        if (!any[u])
            continue;
        if (whole[u]) {
            *(gptr<float4>)(grid + off[u]) =
                make_float4(g[u].x + a[u].x, g[u].y + a[u].y, g[u].z + a[u].z, g[u].w + a[u].w);
        } else {
            const int J = (int)(off[u] % Nt);
            const float v[4] = {a[u].x, a[u].y, a[u].z, a[u].w};
#pragma unroll
            for (int m = 0; m < 4; ++m)
                if (v[m] != 0.0f && J + m < Nt)
                    grid[off[u] + m] = grid[off[u] + m] + v[m];
        }
    }
}

// Lists of the items that open a tile, by colour: counts (counters[kColourCount
// + c]), then each item's place behind the counts of the smaller colours
// (counters[kColourNext + c] hands out places; the order within a colour does
// not matter: its tiles are independent).
template <int TP, int TT, bool B, bool SCATTER>
__global__ __launch_bounds__(256) void k_owner_lists(const int4 *__restrict__ items,
                                                     int32_t *counters,
                                                     const int32_t *__restrict__ tile_off,
                                                     EventCtx e0, BatchTables bt,
                                                     int32_t *colour_list)
{
    constexpr int CP = owner_colours_p<TP, TT>(), CT = owner_colours_t<TT>();
    static_assert(CP * CT <= kMaxColours, "counters of the colour lists");
    const int nitems_all = counters[2];
    const int lane = threadIdx.x & 63;
    const int stride = gridDim.x * blockDim.x;
    // whole wavefronts iterate together: one atomic per list per wavefront
    for (int i0 = blockIdx.x * blockDim.x + (threadIdx.x & ~63); i0 < nitems_all; i0 += stride) {
        const int itm = i0 + lane;
        int c = -1;
        if (itm < nitems_all) {
            const int4 it = items[itm];
            if (it.y == tile_off[it.x]) {  // the tile's first item
                const EventCtx &E = B ? bt.ev[find_event(bt.tile_base, bt.nev, it.x)] : e0;
                const int local = it.x - E.tile_base;
                const int tp = local / E.ntt, tt = local - tp * E.ntt;
                const int ndepos = tile_off[it.x + 1] - it.y;
                c = 2 * ((tp % CP) * CT + tt % CT) + (chunks_of(ndepos) <= kLightItems ? 1 : 0);
            }
        }
        int base = 0;
        if (SCATTER)
            for (int u = 0; u < 2 * CP * CT; ++u)
                base += (u < c) ? counters[kColourCount + u] : 0;
        for (int u = 0; u < 2 * CP * CT; ++u) {
            const uint64_t m = __ballot(c == u);
            if (!m)
                continue;
            const int leader = __ffsll((unsigned long long)m) - 1;
            int first = 0;
            if (lane == leader)
                first = atomicAdd(&counters[(SCATTER ? kColourNext : kColourCount) + u],
                                  __popcll(m));
            first = __shfl(first, leader);
            if (SCATTER && c == u)
                colour_list[base + first + __popcll(m & lanemask_lt(lane))] = itm;
        }
    }
}

template <int TP, int TT, bool B, bool FLUCT>
__global__ __launch_bounds__(64 * kOwnerWaves) void k_raster_owner(
    const float *__restrict__ records, const int4 *__restrict__ items,
    const int32_t *__restrict__ counters, const int32_t *__restrict__ colour_list, EventCtx e0,
    BatchTables bt, int colour_p, int colour_t)
{
    constexpr int RP = TP + kHaloP, RT = region_cols<TT>(), NW = kOwnerWaves;
    constexpr int CP = owner_colours_p<TP, TT>(), CT = owner_colours_t<TT>();
    static_assert(CP * TP >= RP && CT * TT >= RT, "regions of one colour must be disjoint");
    constexpr int RQ4 = RP * RT / 4;
    __shared__ float4 acc4[NW * RQ4];
    __shared__ double xsum[NW * kBatchItems];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int nitems_all = counters[2];
    const int list = 2 * (colour_p * CT + colour_t);
    int base = 0;
    for (int c = 0; c < list; ++c)
        base += counters[kColourCount + c];
    const int nheavy = counters[kColourCount + list], nlight = counters[kColourCount + list + 1];
    float4 *mine = acc4 + w * RQ4;
    double *xs = xsum + w * kBatchItems;
    // draws items first, first + step, ... of the tile that item `itm` opens
    auto draw = [&](int itm, int tile, int first, int step) {
        for (int x = lane; x < RQ4; x += 64)
            mine[x] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        wave_lds_sync();
        for (int j = itm + first; j < nitems_all; j += step) {
            const int4 it = items[j];
            if (it.x != tile)
                break;
            raster_item<TP, TT, B, FLUCT, true>(mine, xs, it, records, e0, bt);
        }
        wave_lds_sync();
    };
    const int nlg = (nlight + NW - 1) / NW;  // light tiles: one per wavefront
    for (int k = blockIdx.x; k < nheavy + nlg; k += gridDim.x) {
        const bool heavy = k < nheavy;
        const int at = heavy ? k : nheavy + (k - nheavy) * NW + w;
        if (!heavy && at >= nheavy + nlight)
            continue;
        const int itm = __builtin_amdgcn_readfirstlane(colour_list[base + at]);
        const int tile = __builtin_amdgcn_readfirstlane(items[itm].x);
        const EventCtx &E = B ? bt.ev[find_event(bt.tile_base, bt.nev, tile)] : e0;
        const int local = tile - E.tile_base;
        const int tp = local / E.ntt, tt = local - tp * E.ntt;
        if (heavy) {
            draw(itm, tile, w, NW);
            __syncthreads();  // every copy of the region is complete
            owner_flush<RP, RT, NW, 64 * NW>(acc4, glb(E.grid), E.kp.Np, E.kp.Nt, tp * TP, tt * TT,
                                             threadIdx.x);
            __syncthreads();  // the copies are read before the next tile clears them
        } else {
            draw(itm, tile, 0, 1);
            owner_flush<RP, RT, 1, 64>(mine, glb(E.grid), E.kp.Np, E.kp.Nt, tp * TP, tt * TT,
                                       lane);
            wave_lds_sync();
        }
    }
}

// Descriptor of a single event (kernel argument; no table lookups).
EventCtx single_event(const wcsim_plane *pl, const wcsim_depo *depos, int64_t n,
                      uint64_t event_id, float *grid, uint8_t *occ = nullptr)
{
    EventCtx e{};
    e.kp = pl->kp;
    e.depos = depos;
    e.grid = grid;
    e.occ = occ;
    e.occ_shift = occ_shift_of(pl->Nt);
    e.depo_base = 0;
    e.n = (int32_t)n;
    e.event = (uint32_t)event_id;
    e.tile_base = 0;
    e.ntt = pl->ntt;
    return e;
}

unsigned blocks_for(int64_t n, int threads)
{
    return (unsigned)((n + threads - 1) / threads);
}

}  // namespace

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
TileShape tile_shape(int id)
{
    switch (id) {
    case 1:
        return {32, 32, kHaloP, kHaloT};
    case 2:
        return {64, 8, kHaloP, kHaloT};
    default:
        return {32, 8, kHaloP, kHaloT};
    }
}

// Compute units of the current device (cached per device).
int device_cus()
{
    static std::atomic<int> cus[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
        return 256;
    int v = cus[dev].load(std::memory_order_relaxed);
    if (v <= 0) {
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            v <= 0)
            v = 256;
        cus[dev].store(v, std::memory_order_relaxed);
    }
    return v;
}

hipError_t launch_fill_zero(void *ptr, size_t bytes, hipStream_t s)
{
    if (bytes == 0)
        return hipSuccess;
    const size_t n16 = bytes / 16;
    if (n16) {
        const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 8192);
        hipLaunchKernelGGL(k_fill_zero16, dim3(blocks), dim3(256), 0, s, (uint4 *)ptr, n16);
    }
    const size_t rem = bytes - n16 * 16;
    if (rem)
        hipLaunchKernelGGL(k_fill_zero1, dim3(1), dim3(16), 0, s, (unsigned char *)ptr + n16 * 16,
                           rem);
    return hipGetLastError();
}

// The code of one sample: float32 in the order the definition states.
__device__ __forceinline__ uint16_t adc_code(float w, float gain, float pedestal, float sigma,
                                             float noise, float top)
{
#pragma clang fp contract(off)
    float v = w * gain;
    v = v + pedestal;
    v = v + sigma * noise;
    return (uint16_t)fminf(fmaxf(rintf(v), 0.0f), top);
}

// One thread per four consecutive samples of a row (one Philox call).  The
// deviates are evaluated in FP64 and rounded once to float32.  Bound by vector
// issue (Philox and two FP64 Box-Muller pairs per thread).  VEC: rows of whole
// quads and aligned pointers, one 16-byte load and one 8-byte store a thread.
// 5.76 M samples: 20.5 us with the library's logarithm, root and sine and scalar
// accesses, 13.7 us so (2.5 TB/s).
template <bool VEC>
__global__ __launch_bounds__(256) void k_digitize(const float *__restrict__ wave, int64_t total,
                                                  int64_t ncols, uint32_t nq, float gain,
                                                  float pedestal, float sigma, float top,
                                                  uint32_t k0, uint32_t k1, uint32_t event,
                                                  uint16_t *__restrict__ adc)
{
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (g >= total)
        return;
    // (32-bit division where the indices allow it: a 64-bit one is as long as
    // the Philox rounds)
    const int64_t row = (total >> 32) ? g / nq : (int64_t)((uint32_t)g / nq), q = g - row * nq;
    const int64_t i0 = row * ncols + 4 * q;
    float w[4] = {0.0f, 0.0f, 0.0f, 0.0f}, z[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (VEC) {
        const float4 v = *(const float4 *)(wave + i0);
        w[0] = v.x;
        w[1] = v.y;
        w[2] = v.z;
        w[3] = v.w;
    } else {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (4 * q + m < ncols)
                w[m] = wave[i0 + m];
    }
    if (sigma > 0.0f) {
        const uint4 r = philox4x32_10(make_uint4((uint32_t)q, (uint32_t)row, 0u, event), k0, k1);
        double zd[4];
        box_muller_d(r.x, r.y, zd[0], zd[1]);
        box_muller_d(r.z, r.w, zd[2], zd[3]);
#pragma unroll
        for (int m = 0; m < 4; ++m)
            z[m] = (float)zd[m];
    }
    uint16_t c[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
        c[m] = adc_code(w[m], gain, pedestal, sigma, z[m], top);
    if (VEC) {
        *(ushort4 *)(adc + i0) = make_ushort4(c[0], c[1], c[2], c[3]);
    } else {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            if (4 * q + m < ncols)
                adc[i0 + m] = c[m];
    }
}

hipError_t launch_digitize(const float *wave, int64_t nrows, int64_t ncols, float gain,
                           float pedestal, float sigma, int bits, uint64_t seed, uint32_t event,
                           uint16_t *adc, hipStream_t s)
{
    const int64_t nq = (ncols + 3) / 4, n = nrows * nq;
    if (n <= 0)
        return hipSuccess;
    const bool vec = ncols % 4 == 0 && ((uintptr_t)wave & 15) == 0 && ((uintptr_t)adc & 7) == 0;
    auto *kernel = vec ? k_digitize<true> : k_digitize<false>;
    hipLaunchKernelGGL(kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, wave, n, ncols,
                       (uint32_t)nq, gain, pedestal, sigma, (float)((1 << bits) - 1),
                       (uint32_t)seed ^ 0x6e6f6973u, (uint32_t)(seed >> 32), event, adc);
    return hipGetLastError();
}

// Coloured noise.  A workgroup of T / 8 threads (or more) takes T columns of one row: it
// draws the white deviates of those columns and of the 8 ceil(nfir / 8) before
// them into LDS in FP64 (one Philox call per quad, as k_digitize), then each
// thread filters eight consecutive columns (FP64 sums in order of the tap),
// rounds the filtered noise once to float32 and digitises.
// Eight columns of a thread share their deviates: a block of eight taps needs
// eight new ones and gives 64 products, where one column at a time read LDS for
// every product and was bound by that.  Column c's deviate lies at
// z[c mod 8][c / 8], so that neighbouring threads read neighbouring words.
// Taps come by scalar loads; zeros stand for the noise before column 0 and the
// taps past the last (exact while the taps are finite).  5.76 M samples, 64 taps:
// 67.7 -> 33.8 us; the deviates alone take 13 us, the FP64 products 12 us.
// Launches of at most kFirShared workgroups a CU take rows that are not whole groups of
// eight by kRowsShared, where the single accesses show (960 rows of 1001 columns, one
// tap 8.6 -> 7.4 us, 400 x 6001 14.3 -> 13.2); in larger ones other workgroups hide them and
// the exchange's barriers cost more (960 x 3001 15.8 -> 16.9).
constexpr int kFirPer = 8;
constexpr int kFirShared = 5;  // workgroups a CU
constexpr int kFirPad = 4;  // rows of z are 8 k + 4 long: quads are written to all banks

__device__ __forceinline__ int fir_stride(int nz) { return nz / kFirPer / 8 * 8 + 8 + kFirPad; }

// ROWS: how samples and codes are read and written.  kRowsWhole: rows of whole groups
// of eight, two 16-byte loads and a 16-byte store a thread.  kRowsShared: any row, the
// noise exchanged through LDS, neighbouring threads on neighbouring columns.
// kRowsSingle: any row, eight single accesses a thread and no exchange.
// MORE: two threads for every eight columns; those past the filter's only draw.
enum { kRowsWhole, kRowsShared, kRowsSingle };
template <int ROWS, bool MORE>
__global__ __launch_bounds__(256) void k_digitize_fir(const float *__restrict__ wave, int64_t nrows,
                                                      int64_t ncols, int64_t tiles, float gain,
                                                      float pedestal, float sigma,
                                                      const float *__restrict__ fir, int nfir,
                                                      float top, uint32_t k0, uint32_t k1,
                                                      uint32_t event, uint16_t *__restrict__ adc)
{
    extern __shared__ double fir_lds[];
    const int T = kFirPer / (MORE ? 2 : 1) * blockDim.x, tid = threadIdx.x;
    const bool filters = !MORE || tid < T / kFirPer;
    const int nkb = (nfir + kFirPer - 1) / kFirPer;  // blocks of taps
    const int nz = T + kFirPer * nkb, stride = fir_stride(nz);
    double *z = fir_lds;
    const int64_t row = blockIdx.x / tiles;
    const int64_t t0 = (blockIdx.x - row * tiles) * T, base = t0 - kFirPer * nkb;
    const int64_t c0 = t0 + kFirPer * tid;  // this thread's first column
    const int64_t i0 = row * ncols + c0;
    // The samples and the first taps are under way before the draws.
    float w[kFirPer];
    if (ROWS == kRowsWhole) {
        const int64_t i = (filters && c0 < ncols) ? i0 : row * ncols;
#pragma unroll
        for (int m = 0; m < kFirPer; m += 4) {
            const float4 v = *(const float4 *)(wave + i + m);
            w[m] = v.x;
            w[m + 1] = v.y;
            w[m + 2] = v.z;
            w[m + 3] = v.w;
        }
    } else if (ROWS == kRowsShared) {
#pragma unroll
        for (int m = 0; m < kFirPer; ++m) {
            const int c = tid + m * (int)blockDim.x;
            w[m] = ((!MORE || c < T) && t0 + c < ncols) ? wave[row * ncols + t0 + c] : 0.0f;
        }
    }
    const float tap = fir[min(tid, nfir - 1)];
    for (int qi = tid; 4 * qi < nz; qi += blockDim.x) {
        const int64_t c = base + 4 * qi;  // first column of the quad
        double zz[4] = {0.0, 0.0, 0.0, 0.0};
        if (c >= 0 && c < ncols && sigma > 0.0f) {
            const uint4 r =
                philox4x32_10(make_uint4((uint32_t)(c >> 2), (uint32_t)row, 0u, event), k0, k1);
            box_muller_d(r.x, r.y, zz[0], zz[1]);
            box_muller_d(r.z, r.w, zz[2], zz[3]);
        }
#pragma unroll
        for (int m = 0; m < 4; ++m)
            z[((4 * qi + m) & (kFirPer - 1)) * stride + (4 * qi + m) / kFirPer] = zz[m];
    }
    bool bad = !isfinite(tap);
    for (int k = tid + (int)blockDim.x; k < nfir; k += blockDim.x)
        bad = bad || !isfinite(fir[k]);
    const bool general = __syncthreads_or(bad);
    double n[kFirPer];
#pragma unroll
    for (int m = 0; m < kFirPer; ++m)
        n[m] = 0.0;
    const int pos = nkb + tid;
    if (!filters) {
    } else if (!general) {
        // one block of taps t[r]: columns of x (this octet) and y (the one before)
        auto block = [&](const double *t, const double *x, const double *y) {
#pragma unroll
            for (int r = 0; r < kFirPer; ++r)
#pragma unroll
                for (int m = 0; m < kFirPer; ++m)
                    n[m] = fma(t[r], (m >= r) ? x[m - r] : y[kFirPer + m - r], n[m]);
        };
        auto octet = [&](int at, double *x) {
#pragma unroll
            for (int m = 0; m < kFirPer; ++m)
                x[m] = z[m * stride + at];
        };
        double x[kFirPer], y[kFirPer], t[kFirPer];
        octet(pos, x);
        int kb = 0;
        for (; (kb + 2) * kFirPer <= nfir; kb += 2) {
            const float *f = fir + kFirPer * kb;  // (the same for every lane: scalar loads)
            octet(pos - kb - 1, y);
#pragma unroll
            for (int r = 0; r < kFirPer; ++r)
                t[r] = (double)f[r];
            block(t, x, y);
            octet(pos - kb - 2, x);
#pragma unroll
            for (int r = 0; r < kFirPer; ++r)
                t[r] = (double)f[kFirPer + r];
            block(t, y, x);
        }
        for (; kb < nkb; ++kb) {  // at most two more, the last one filled up with zero taps
            octet(pos - kb - 1, y);
#pragma unroll
            for (int r = 0; r < kFirPer; ++r) {
                const int k = kFirPer * kb + r;
                const float v = fir[min(k, nfir - 1)];
                t[r] = (k < nfir) ? (double)v : 0.0;
            }
            block(t, x, y);
#pragma unroll
            for (int m = 0; m < kFirPer; ++m)
                x[m] = y[m];
        }
    } else {
        // a tap that is not finite must not meet the zeros before column 0
        for (int k = 0; k < nfir; ++k) {
            const double t = (double)fir[k];
#pragma unroll
            for (int m = 0; m < kFirPer; ++m) {
                const int c = kFirPer * pos + m - k;
                if (k <= c0 + m)
                    n[m] = fma(t, z[(c & (kFirPer - 1)) * stride + c / kFirPer], n[m]);
            }
        }
    }
    if (ROWS == kRowsWhole) {
        if (!filters || c0 >= ncols)
            return;
        uint32_t c[kFirPer];
#pragma unroll
        for (int m = 0; m < kFirPer; ++m)
            c[m] = adc_code(w[m], gain, pedestal, sigma, (float)n[m], top);
        *(uint4 *)(adc + i0) = make_uint4(c[0] | c[1] << 16, c[2] | c[3] << 16, c[4] | c[5] << 16,
                                          c[6] | c[7] << 16);
    } else if (ROWS == kRowsSingle) {
#pragma unroll
        for (int m = 0; m < kFirPer; ++m)
            w[m] = (filters && c0 + m < ncols) ? wave[i0 + m] : 0.0f;
#pragma unroll
        for (int m = 0; m < kFirPer; ++m)
            if (filters && c0 + m < ncols)
                adc[i0 + m] = adc_code(w[m], gain, pedestal, sigma, (float)n[m], top);
    } else {
        // the filtered noise through LDS (in place of the deviates) to the threads
        // that hold the samples
        float *nf = (float *)fir_lds;
        __syncthreads();
        if (filters) {
#pragma unroll
            for (int m = 0; m < kFirPer; ++m)
                nf[m * stride + tid] = (float)n[m];
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < kFirPer; ++m) {
            const int c = tid + m * (int)blockDim.x;
            if ((!MORE || c < T) && t0 + c < ncols)
                adc[row * ncols + t0 + c] =
                    adc_code(w[m], gain, pedestal, sigma,
                             nf[(c & (kFirPer - 1)) * stride + c / kFirPer], top);
        }
    }
}

hipError_t launch_digitize_fir(const float *wave, int64_t nrows, int64_t ncols, float gain,
                               float pedestal, float sigma, const float *fir, int nfir, int bits,
                               uint64_t seed, uint32_t event, uint16_t *adc, hipStream_t s)
{
    if (nrows <= 0 || ncols <= 0)
        return hipSuccess;
    // A tap past the row's length meets no sample (960 rows of 64 columns, 1,000 taps:
    // 34.5 -> 10 us).
    nfir = (int)std::min<int64_t>(nfir, ncols);
    // Columns per workgroup: the fewest columns drawn for the row, history
    // included; at least 1024 for rows longer than one workgroup takes (the
    // limit on the waveform's size counts blocks of 1024).
    const int hist = (nfir + kFirPer - 1) / kFirPer * kFirPer;
    int T = 0;
    int64_t best = 0;
    for (int t : {2048, 1536, 1024, 512}) {
        if (t == 512 && ncols > 512)
            break;
        const int64_t cost = (ncols + t - 1) / t * (t + hist);
        if (!T || cost < best) {
            T = t;
            best = cost;
        }
    }
    // A launch that leaves most of the chip idle lasts as long as one workgroup: twice the
    // threads then share its draws and samples (the filter keeps eight columns a
    // thread), and short filters, whose workgroups are all draws, take 1024 columns
    // unless that alone makes it more than one workgroup a CU.  400 rows of 1001
    // columns, one tap: 7.5 -> 6.3 us, 64 taps 10.3 -> 9.0; 200 x 3001, one tap 8.1 -> 7.2 (256
    // taps 18.1 -> 19.0, so not there); 200 x 2000, one tap 5.0 -> 5.6, so not there; 960 x
    // 1001, 64 taps 10.3 -> 11.4.
    const int64_t cus = device_cus(), few = nfir <= 32 ? 3 * cus : 2 * cus;
    auto launch_blocks = [&](int t) { return nrows * ((ncols + t - 1) / t); };
    if (nfir <= 32 && T > 1024 && launch_blocks(1024) <= few &&
        (launch_blocks(1024) <= cus || launch_blocks(T) > cus))
        T = 1024;
    const int64_t tiles = (ncols + T - 1) / T, blocks = nrows * tiles;
    const bool more = T <= 1024 && blocks <= few;
    const int nz = T + hist;
    const size_t lds =
        sizeof(double) * kFirPer * (size_t)(nz / kFirPer / 8 * 8 + 8 + kFirPad);
    const bool vec = ncols % kFirPer == 0 && ((uintptr_t)wave & 15) == 0 &&
                     ((uintptr_t)adc & 15) == 0;
    auto *kernel = vec ? (more ? k_digitize_fir<kRowsWhole, true> : k_digitize_fir<kRowsWhole, false>)
                   : blocks > kFirShared * cus ? k_digitize_fir<kRowsSingle, false>
                   : more ? k_digitize_fir<kRowsShared, true> : k_digitize_fir<kRowsShared, false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(T / kFirPer * (more ? 2 : 1)), lds, s,
                       wave, nrows, ncols, tiles, gain, pedestal, sigma, fir, nfir, (float)((1 << bits) - 1),
                       (uint32_t)seed ^ 0x6e6f6973u, (uint32_t)(seed >> 32), event, adc);
    return hipGetLastError();
}

hipError_t launch_philox(const uint32_t *ctr, const uint32_t *key, int64_t n, uint32_t *out,
                         hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_philox, dim3(blocks_for(n, 256)), dim3(256), 0, s, (const uint4 *)ctr,
                       (const uint2 *)key, n, (uint4 *)out);
    return hipGetLastError();
}

size_t scan_scratch_bytes(int64_t n)
{
    return align_up(sizeof(int64_t) * (size_t)((n + kScanBlock - 1) / kScanBlock + 1));
}

hipError_t launch_exclusive_scan_i64(int64_t *data, int64_t n, void *scratch, hipStream_t s)
{
    return exclusive_scan<int64_t>(data, n, scratch, s);
}

hipError_t launch_patch_sizes(const wcsim_plane *pl, const wcsim_depo *depos, int64_t n,
                              int32_t *meta, int64_t *sizes, int32_t *large, hipStream_t s)
{
    PatchSums *sums = (PatchSums *)(sizes + n + 1);
    static_assert(sizeof(PatchSums) <= 16, "cleared by one small workgroup");
    hipLaunchKernelGGL(k_fill_zero1, dim3(1), dim3(16), 0, s, (unsigned char *)sums, sizeof(PatchSums));
    hipLaunchKernelGGL(k_patch_sizes, dim3(blocks_for(std::max<int64_t>(n, 1), 256)), dim3(256), 0,
                       s, depos, n, pl->kp, meta, sizes, large, sums);
    return hipGetLastError();
}

// The patches beyond a wavefront get a workgroup each: of four wavefronts while they are
// few, of one when they fill the chip with those (at long drift, at nsigma = 5 or
// with twice the diffusion most of a set is among them).  Whole call, one wavefront /
// four: 300 windows of 13,000 bins 209 / 103 us, 789 of 1,500 bins 81 / 74, 3,159 103
// / 104, 79,920 1026 / 1235 (on 256 workgroups of four for any number: 2684).
constexpr int64_t kFewLarge = 1024;

hipError_t launch_patch_values(const wcsim_plane *pl, const wcsim_depo *depos, int64_t n,
                               uint64_t event_id, const int64_t *offsets, float *values,
                               const int32_t *large, const int32_t *nlarge, int64_t count,
                               hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    if (count < n) {
        int per = 1;
        while (per < kWavePatches && n >= 2 * per * kWaveFill)
            per *= 2;
        auto *kernel = pl->kp.fluct ? k_patch_wave<true> : k_patch_wave<false>;
        hipLaunchKernelGGL(kernel, dim3(blocks_for(n, 4 * per)), dim3(256), 0, s, depos, n, pl->kp,
                           (uint32_t)event_id, per, offsets, values);
    }
    if (count > 0) {
        const EventCtx e0 = single_event(pl, depos, n, event_id, nullptr);
        const bool few = count <= kFewLarge;
        auto *kernel = few ? k_patch_generic<256, true, false> : k_patch_generic<64, true, false>;
        hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<int64_t>(count, 1 << 20)),
                           dim3(few ? 256 : 64), 0, s, e0, BatchTables{}, large, nlarge,
                           (int64_t)0, offsets, values);
    }
    return hipGetLastError();
}

hipError_t launch_scatter_flat(const wcsim_plane *pl, int64_t n, bool close, const int32_t *meta,
                               const int64_t *offsets, const float *values, float *grid,
                               hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    const bool sum = close && n >= kScatMany;
    int per = sum ? 4 : 1;
    while (sum && per < 16 && n >= per * kScatFill)
        per *= 2;
    const int waves = sum ? kScatWaves<true> : kScatWaves<false>;
    auto *kernel = sum ? k_scatter_flat<true> : k_scatter_flat<false>;
    hipLaunchKernelGGL(kernel, dim3(blocks_for(n, waves * per)), dim3(64 * waves), 0, s, n, per, meta,
                       offsets, values, grid, (int)pl->Np, (int)pl->Nt);
    return hipGetLastError();
}

// Blocks of the record kernel that clear the occupied blocks of the grids: one
// wavefront per part of a band of grid rows, at most kMaxClearBlocks blocks.
// Bands are cut into 2^shift parts of map columns until kClearWaves wavefronts
// share the clear: one wavefront took 110 us over a whole band of a long odd
// readout (dword stores) and set the kernel's time.  333 wires x 4097 ticks: 120
// us with whole bands, 53 with 256 wavefronts, 41 with 512 or 1024; 960 wires x
// 6000 ticks: 72 us before, 68 with 256 or 512, 71 with 1024 (the clearing blocks
// hold the LDS of record blocks).
constexpr int kMaxClearBlocks = 4096;
constexpr int kClearWaves = 512;

// Up to this many depos a record block has four wavefronts instead of two: the
// pitch edges of a depo in three parts, each a chain of FP64 erfc, where the
// launch cannot fill the chip anyway (the window and the outer edges are then
// evaluated by each part).  Record kernel with two / four: 1,000 uniform depos 13.3 /
// 9.0 us, 20,000 track depos 12.3 / 9.1, 50,000 14.9 / 14.4, 100,000 23.6 / 25.0,
// 500,000 67 / 77.
constexpr int64_t kWideRecords = 32768;

static size_t sched_blocks_of(int64_t ntiles)
{
    return (size_t)((ntiles + 1 + kSchedTiles - 1) / kSchedTiles);
}

static size_t items_cap(int64_t ntiles, int64_t n)
{
    return (size_t)ntiles + (size_t)(std::max<int64_t>(n, 1) / kChunk) + 1;
}

// Wavefronts of the raster launch: enough for the work lists of track-like
// and uniform depo sets (a work item holds up to kChunk depos of one tile;
// the collection plane's 500,000 depos make 29,129 items), never more than
// the worst case; any further items are taken by a second round.
static unsigned raster_grid(int64_t ntiles, int64_t n)
{
    return (unsigned)std::min<size_t>(items_cap(ntiles, n), (size_t)(n / 8) + 4096);
}

// Counters: [0..3] as RasterWork states, then the colour lists' (the words past
// them are kept free: workspace sizes stay what they were).
constexpr int kCounterWords = 64;
constexpr size_t kCounterBytes = sizeof(int32_t) * (kCounterWords + 256);

// The tile-list sort works in the record area before the records are written:
// keys and depo indices twice (ping-pong) and the per-block digit counts.
static size_t sort_blocks_of(size_t n) { return (n + kSortBlock - 1) / kSortBlock; }
static size_t sort_bytes(size_t n)  // (with 9-bit digits, n >= kSortBlock: records are larger)
{
    return 4 * align_up(sizeof(int32_t) * n) + align_up(sizeof(int32_t) * 256 * sort_blocks_of(n));
}

size_t raster_work_bytes_batch(const wcsim_plane *pl, int64_t n, int64_t ntiles, int64_t nbands)
{
    (void)pl;
    const size_t nn = (size_t)std::max<int64_t>(n, 1);
    return align_up(kCounterBytes) + align_up(sizeof(int32_t) * (size_t)(ntiles + 1)) +
           align_up((size_t)kOccCols * (size_t)nbands) +
           align_up(sizeof(int2) * sched_blocks_of(ntiles)) +
           align_up(sizeof(int4) * items_cap(ntiles, n)) + 3 * align_up(sizeof(int32_t) * nn) +
           align_up(std::max(sizeof(float) * kRecWords * nn, sort_bytes(nn)));
}

RasterWork raster_work_carve_batch(const wcsim_plane *pl, int64_t n, int64_t ntiles,
                                   int64_t nbands, void *base)
{
    (void)pl;
    const size_t nn = (size_t)std::max<int64_t>(n, 1);
    char *p = (char *)base;
    RasterWork w;
    w.counters = (int32_t *)p;
    p += align_up(kCounterBytes);
    w.tile_count = (int32_t *)p;
    p += align_up(sizeof(int32_t) * (size_t)(ntiles + 1));
    w.occ = (uint8_t *)p;  // adjacent to the counters: cleared together
    p += align_up((size_t)kOccCols * (size_t)nbands);
    w.block_tot = (int2 *)p;
    p += align_up(sizeof(int2) * sched_blocks_of(ntiles));
    w.items = (int4 *)p;
    p += align_up(sizeof(int4) * items_cap(ntiles, n));
    w.depo_tile = (int32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    w.depo_slot = (int32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    w.large = (int32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    w.records = (float *)p;
    return w;
}

size_t raster_work_bytes(const wcsim_plane *pl, int64_t n)
{
    return raster_work_bytes_batch(pl, n, pl->ntiles, occ_bands(pl->Np));
}

RasterWork raster_work_carve(const wcsim_plane *pl, int64_t n, void *base)
{
    return raster_work_carve_batch(pl, n, pl->ntiles, occ_bands(pl->Np), base);
}

// The colour lists (in depo_tile, free once the records are written: a tile
// list has at most n items), then one launch per colour of the owner flush,
// colours in row-major order, each with as many workgroups as the device
// holds at once (LDS-bound).
template <int TP, int TT, bool B, bool FLUCT>
static void launch_owner_phases(unsigned items_grid, const RasterWork &w, const EventCtx &e0,
                                const BatchTables &bt, hipStream_t s)
{
    const unsigned lg = std::max(1u, std::min(items_grid / 4, 2048u));
    hipLaunchKernelGGL((k_owner_lists<TP, TT, B, false>), dim3(lg), dim3(256), 0, s, w.items,
                       w.counters, w.tile_count, e0, bt, w.depo_tile);
    hipLaunchKernelGGL((k_owner_lists<TP, TT, B, true>), dim3(lg), dim3(256), 0, s, w.items,
                       w.counters, w.tile_count, e0, bt, w.depo_tile);
    constexpr size_t lds = sizeof(float4) * kOwnerWaves * (TP + kHaloP) * region_cols<TT>() / 4 +
                           sizeof(double) * kOwnerWaves * kBatchItems;
    const unsigned per_cu = (unsigned)std::max<size_t>(1, (160 * 1024) / lds);
    const unsigned grid = (unsigned)device_cus() * per_cu;
    for (int cp = 0; cp < owner_colours_p<TP, TT>(); ++cp)
        for (int ct = 0; ct < owner_colours_t<TT>(); ++ct)
            hipLaunchKernelGGL((k_raster_owner<TP, TT, B, FLUCT>), dim3(grid),
                               dim3(64 * kOwnerWaves), 0, s, w.records, w.items, w.counters,
                               w.depo_tile, e0, bt, cp, ct);
}

template <bool B, bool FLUCT>
static void launch_raster_owner(int tile, unsigned grid, const RasterWork &w, const EventCtx &e0,
                                const BatchTables &bt, hipStream_t s)
{
    switch (tile) {
    case 1:
        launch_owner_phases<32, 32, B, FLUCT>(grid, w, e0, bt, s);
        break;
    case 2:
        launch_owner_phases<64, 8, B, FLUCT>(grid, w, e0, bt, s);
        break;
    default:
        launch_owner_phases<32, 8, B, FLUCT>(grid, w, e0, bt, s);
        break;
    }
}

// Tile lists in depo order: sort, then slots and the ordered large-patch list.
static void launch_tile_list_sort(int64_t n, int64_t ntiles, const RasterWork &w, hipStream_t s)
{
    const size_t nn = (size_t)n;
    char *p = (char *)w.records;
    uint32_t *kA = (uint32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    uint32_t *kB = (uint32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    int32_t *vA = (int32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    int32_t *vB = (int32_t *)p;
    p += align_up(sizeof(int32_t) * nn);
    int32_t *counts = (int32_t *)p;
    const unsigned nblk = (unsigned)sort_blocks_of(nn);
    const uint32_t nt = (uint32_t)ntiles;
    int bits = 1;
    while (bits < 32 && ((uint64_t)nt + 1) >> bits)
        ++bits;
    hipLaunchKernelGGL(k_sort_keys, dim3(blocks_for(n, 256)), dim3(256), 0, s, w.depo_tile, n, nt,
                       kA, vA);
    auto digits = [&](auto width) {
        constexpr int BITS = decltype(width)::value;
        for (int shift = 0; shift < bits; shift += BITS) {
            hipLaunchKernelGGL(k_sort_count<BITS>, dim3(nblk), dim3(kSortThreads), 0, s, kA, n,
                               shift, counts);
            hipLaunchKernelGGL(k_sort_offsets<BITS>, dim3(1), dim3(kSortThreads), 0, s, counts,
                               (int)nblk);
            hipLaunchKernelGGL(k_sort_scatter<BITS>, dim3(nblk), dim3(kSortThreads), 0, s, kA, vA,
                               n, shift, counts, kB, vB);
            std::swap(kA, kB);
            std::swap(vA, vB);
        }
    };
    // Nine-bit digits where they save one (planes of 65,535 to 262,142 tiles: two
    // digits instead of three, 63 us instead of 76 for 150,000 depos) and the record
    // area holds their counts.
    if ((bits + 8) / 9 < (bits + 7) / 8 && n >= kSortBlock)
        digits(std::integral_constant<int, 9>{});
    else
        digits(std::integral_constant<int, 8>{});
    hipLaunchKernelGGL(k_sort_slots, dim3(blocks_for(n, 256)), dim3(256), 0, s, kA, vA, n, nt,
                       w.tile_count, w.depo_slot, w.large);
}

template <bool B, bool FLUCT>
static void launch_raster_tiles(int tile, unsigned grid, const RasterWork &w, const EventCtx &e0,
                                const BatchTables &bt, hipStream_t s)
{
    switch (tile) {
    case 1:
        hipLaunchKernelGGL((k_raster_tiles<32, 32, B, FLUCT>), dim3(grid), dim3(64), 0, s,
                           w.records, w.items, w.counters, e0, bt);
        break;
    case 2:
        hipLaunchKernelGGL((k_raster_tiles<64, 8, B, FLUCT>), dim3(grid), dim3(64), 0, s,
                           w.records, w.items, w.counters, e0, bt);
        break;
    default:
        hipLaunchKernelGGL((k_raster_tiles<32, 8, B, FLUCT>), dim3(grid), dim3(64), 0, s,
                           w.records, w.items, w.counters, e0, bt);
        break;
    }
}

// The launch sequence shared by single events and batches: clear counters,
// window + tile per depo, tile schedule, depo records, LDS-tiled raster,
// large-patch raster.  `ev` (single events only) receives three stage marks.
template <bool B>
static hipError_t raster_sequence(const wcsim_plane *pl, const EventCtx &e0,
                                  const BatchTables &bt, int64_t n, int64_t ntiles,
                                  int64_t nbands, const RasterWork &w, hipStream_t s,
                                  const hipEvent_t *ev)
{
    hipError_t e;
    auto mark = [&](int i) { return ev ? hipEventRecord(ev[i], s) : hipSuccess; };
    // counters, tile counts and occupancy maps are adjacent: one clear
    const size_t clear = (size_t)((char *)w.occ - (char *)w.counters) +
                         (size_t)kOccCols * (size_t)nbands;
    if ((e = launch_fill_zero(w.counters, align_up(clear, 16), s)) != hipSuccess)
        return e;
    if (n <= 0) {  // an empty map: nothing of the grid is read
        for (int i = 0; i < 3; ++i)
            if ((e = mark(i)) != hipSuccess)
                return e;
        return hipSuccess;
    }
    TileGeom g;
    g.tp = pl->ts.tp;
    g.tt = pl->ts.tt;
    g.rp = pl->ts.tp + kHaloP;
    g.rt = pl->ts.tt + kHaloT;
    g.ntt = pl->ntt;
    hipLaunchKernelGGL(k_prep_bin<B>, dim3(blocks_for(n, 256)), dim3(256), 0, s, e0, bt, n, g,
                       w.counters, w.tile_count, w.depo_tile, w.depo_slot, w.large);
    const unsigned sched_blocks = (unsigned)sched_blocks_of(ntiles);
    if (pl->det) {
        hipLaunchKernelGGL(k_tile_sums, dim3(sched_blocks), dim3(kSchedThreads), 0, s,
                           w.tile_count, (int)ntiles, w.block_tot);
        hipLaunchKernelGGL(k_scan_block_tot, dim3(1), dim3(kSchedThreads), 0, s, w.block_tot,
                           (int)sched_blocks);
        hipLaunchKernelGGL(k_tile_schedule<true>, dim3(sched_blocks), dim3(kSchedThreads), 0, s,
                           w.tile_count, (int)ntiles, w.block_tot, w.items, w.counters);
        launch_tile_list_sort(n, ntiles, w, s);
    } else {
        hipLaunchKernelGGL(k_tile_schedule<false>,
                           dim3(blocks_for(ntiles, kSchedThreads * kListPer)),
                           dim3(kSchedThreads), 0, s, w.tile_count, (int)ntiles, w.block_tot, w.items, w.counters);
    }
    int parts_shift = 0;
    while (parts_shift < 3 && (nbands << parts_shift) < kClearWaves)
        ++parts_shift;
    const int nw = n <= kWideRecords ? 4 : 2;
    const int nclr =
        (int)std::min<int64_t>(kMaxClearBlocks, ((nbands << parts_shift) + nw - 1) / nw);
    auto *records = nw == 4 ? k_fill_records<B, 4> : k_fill_records<B, 2>;
    hipLaunchKernelGGL(records, dim3(blocks_for(n, 64) + nclr), dim3(64 * nw), 0, s, e0, bt, n,
                       w.depo_tile, w.depo_slot, w.tile_count, w.records, (int)nbands, nclr,
                       parts_shift);
    if ((e = hipGetLastError()) != hipSuccess || (e = mark(0)) != hipSuccess)
        return e;
    const unsigned grid_items = raster_grid(ntiles, n);
    if (pl->det && pl->kp.fluct)
        launch_raster_owner<B, true>(pl->tile, grid_items, w, e0, bt, s);
    else if (pl->det)
        launch_raster_owner<B, false>(pl->tile, grid_items, w, e0, bt, s);
    else if (pl->kp.fluct)
        launch_raster_tiles<B, true>(pl->tile, grid_items, w, e0, bt, s);
    else
        launch_raster_tiles<B, false>(pl->tile, grid_items, w, e0, bt, s);
    if ((e = hipGetLastError()) != hipSuccess || (e = mark(1)) != hipSuccess)
        return e;
    // Depos whose patch does not fit a tile region: one workgroup each, direct
    // atomics.  The grid is persistent over the device-side count, one
    // workgroup per CU (most workloads have no such depo, and each workgroup
    // holds 17 KB of LDS while it looks).  With reproducible sums one
    // workgroup adds the patches one after another in depo order (a patch's
    // bins are distinct; its atomics complete before the next patch's).
    const unsigned lg = pl->det ? 1u : (unsigned)std::min<int64_t>(n, 256);
    hipLaunchKernelGGL((k_patch_generic<256, false, B>), dim3(lg), dim3(256), 0, s, e0, bt,
                       w.large, w.counters + 1, (int64_t)0, nullptr, nullptr);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    return mark(2);
}

hipError_t launch_raster_fused(const wcsim_plane *pl, const wcsim_depo *depos, int64_t n,
                               uint64_t event_id, const RasterWork &w, float *grid, hipStream_t s,
                               const hipEvent_t *ev)
{
    const EventCtx e0 = single_event(pl, depos, n, event_id, grid, w.occ);
    return raster_sequence<false>(pl, e0, BatchTables{}, n, pl->ntiles, occ_bands(pl->Np), w, s,
                                  ev);
}

hipError_t launch_raster_batch(const wcsim_plane *pl, const BatchTables &bt, int64_t n_total,
                               int64_t ntiles_total, int64_t nbands_total, const RasterWork &w,
                               hipStream_t s, const hipEvent_t *ev)
{
    return raster_sequence<true>(pl, EventCtx{}, bt, n_total, ntiles_total, nbands_total, w, s,
                                 ev);
}

// Zero the blocks that the occupancy map leaves unmarked (one wavefront per
// band of rows), so that the whole grid holds the event.
__global__ __launch_bounds__(64) void k_clear_unoccupied(float *grid, int Np, int Nt,
                                                         const uint8_t *occ, int shift)
{
    const int band = blockIdx.x, lane = threadIdx.x;
    const int nb = (Nt + (1 << shift) - 1) >> shift;
    const uint64_t valid = (nb >= 64) ? ~0ull : ((1ull << nb) - 1ull);
    const uint64_t m = __ballot(occ[band * kOccCols + lane] != 0);
    clear_blocks(glb(grid), Np, Nt, band, ~m & valid, shift, lane);
}

hipError_t launch_clear_unoccupied(float *grid, int Np, int Nt, const uint8_t *occ, int shift,
                                   hipStream_t s)
{
    if (Np <= 0 || Nt <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_clear_unoccupied, dim3((unsigned)occ_bands(Np)), dim3(64), 0, s, grid,
                       Np, Nt, occ, shift);
    return hipGetLastError();
}

}  // namespace wcs
