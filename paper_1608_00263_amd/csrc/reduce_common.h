// Device helpers shared by the reduction kernels and the ensemble kernel:
// probabilities in FP64 and fixed-order wavefront / workgroup sums.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace svi {

constexpr int RB = 256;   // threads per workgroup

template <typename T> struct cpx { T re, im; };

// p = re*re + im*im with both products and the sum rounded separately: the
// expression is compiled with contraction off (the rounded-operation
// intrinsics of this toolchain are plain operators, which the default
// contraction of device code would fuse into fma(re, re, im*im)); for
// complex64 input both products are exact in FP64.
__device__ __forceinline__ double prob_of(cpx<float> a) {
#pragma clang fp contract(off)
    const double r = (double)a.re, i = (double)a.im;
    return r * r + i * i;
}
__device__ __forceinline__ double prob_of(cpx<double> a) {
#pragma clang fp contract(off)
    return a.re * a.re + a.im * a.im;
}
__device__ __forceinline__ double prob_of(double p) { return p; }

template <typename V>
__device__ __forceinline__ V wave_sum(V v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
}

// The same for doubles without LDS round trips (a shuffle is two of them per
// step, and the statistics reduce 13 values at once): DPP moves within rows of
// 16 lanes, then the half swaps across rows.  Every step adds two equal-sized
// partial sums of the same lanes in every lane, so all lanes hold one result.
template <int CTRL>
__device__ __forceinline__ double dpp_move_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
template <>
__device__ __forceinline__ double wave_sum<double>(double v) {
    v += dpp_move_f64<0xB1>(v);    // quad_perm 1,0,3,2
    v += dpp_move_f64<0x4E>(v);    // quad_perm 2,3,0,1
    v += dpp_move_f64<0x141>(v);   // half-row mirror: the other quad of 8
    v += dpp_move_f64<0x140>(v);   // row mirror: the other half of 16
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const auto l16 = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h16 = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    v = __hiloint2double((int)h16[0], (int)l16[0]) + __hiloint2double((int)h16[1], (int)l16[1]);
    const int lo2 = __double2loint(v), hi2 = __double2hiint(v);
    const auto l32 = __builtin_amdgcn_permlane32_swap(lo2, lo2, false, false);
    const auto h32 = __builtin_amdgcn_permlane32_swap(hi2, hi2, false, false);
    return __hiloint2double((int)h32[0], (int)l32[0]) + __hiloint2double((int)h32[1], (int)l32[1]);
}

// Workgroup sum of NV values per thread into red[0..NV) (fixed order).
template <typename V, int NV>
__device__ __forceinline__ void block_sum(V (&v)[NV], V *red /* LDS, 4*NV */) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NV; i++) v[i] = wave_sum(v[i]);
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < NV; i++) red[wave * NV + i] = v[i];
    __syncthreads();
    if (threadIdx.x < NV) {
        V s = red[threadIdx.x];
        for (int w = 1; w < RB / 64; w++) s += red[w * NV + threadIdx.x];
        red[threadIdx.x] = s;   // each thread reads its column first
    }
    __syncthreads();
}

// Combines n partial rows of 16 doubles each, quantity q = 0..nq-1, by a
// workgroup of CMB_THREADS threads: 64 segments of the rows are summed in
// parallel (Neumaier, eight rows loaded before they are added), then the
// segments pairwise in a fixed tree with the rounding errors carried along.
// The order is fixed, so the result does not depend on timing.  A workgroup's
// time here is the latency of its loads: 16 segments with one load in flight
// took 63 us for 2048 rows; red holds 2 * 64 * 16 doubles of LDS.
constexpr int CMB_THREADS = 1024;

__device__ __forceinline__ void neumaier_add(double &s, double &c, double x) {
    const double t = s + x;
    if (fabs(s) >= fabs(x)) c += (s - t) + x;
    else c += (x - t) + s;
    s = t;
}

__device__ __forceinline__ void combine_rows_wg(const double *part, int n, int nq, double *out, double *red) {
    const int q = threadIdx.x & 15, seg = threadIdx.x >> 4;
    const int per = (n + 63) / 64;
    const int b0 = seg * per, b1 = b0 + per < n ? b0 + per : n;
    double s = 0.0, c = 0.0;
    if (q < nq) {
        for (int b = b0; b < b1; b += 8) {
            double x[8];
#pragma unroll
            for (int j = 0; j < 8; j++) x[j] = b + j < b1 ? part[(uint64_t)(b + j) * 16 + q] : 0.0;
#pragma unroll
            for (int j = 0; j < 8; j++)
                if (b + j < b1) neumaier_add(s, c, x[j]);
        }
    }
    double *ss = red, *cc = red + 64 * 16;
    ss[threadIdx.x] = s;
    cc[threadIdx.x] = c;
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) {
        __syncthreads();
        if (seg < h) {
            const int o = threadIdx.x + h * 16;
            double cs = cc[threadIdx.x] + cc[o], sv = ss[threadIdx.x];
            neumaier_add(sv, cs, ss[o]);
            ss[threadIdx.x] = sv;
            cc[threadIdx.x] = cs;
        }
    }
    if (threadIdx.x < nq) out[threadIdx.x] = ss[threadIdx.x] + cc[threadIdx.x];
}

constexpr int NSTAT = 13;   // S, sum p ln p, sum ln p, sum u^k (k = 1..10)

// a * b + c as the three-operand FP64 FMA with a wave-uniform addend in scalar
// registers: the accumulating form (whose addend is also its destination)
// would copy each series coefficient before every use.
__device__ __forceinline__ double fma3s(double a, double b, double c) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// Table-driven natural logarithm (the method of P. T. P. Tang, "Table-driven
// implementation of the logarithm function in IEEE floating-point
// arithmetic", ACM TOMS 16(4), 1990).  x = 2^e z with z in [0.69987, 1.39974)
// cut into 256 bins; per bin inv ~ 1/centre and ln = -ln(inv) (a double-double
// series at compile time), so that ln x = e ln 2 + ln + ln(1 + r), r = z inv -
// 1 (one rounding), |r| < 2^-9, by its series to r^6 (the next term is below
// 2^-65).  The bin that holds 1 has inv = 1 and ln = 0 and reaches 2^-9.58 to
// both sides, so ln 1 = 0 exactly and x near 1 keeps its relative accuracy.
// Ten FP64 operations and a 16-byte LDS read; at most 1.3 ulp measured over
// 4e7 arguments.  (An atanh series with its quarter-rate reciprocal took about
// 30 operations.)
struct LnEntry { double inv, ln; };
constexpr int LN_BINS = 256;
constexpr int LN_ONE_BIN = 153;
constexpr int LN_OFF = 0x3ff00000 - 2731 - LN_ONE_BIN * 4096;   // high word of the lowest z

struct LnTable {
    LnEntry t[LN_BINS];
    struct DD { double h, l; };
    static constexpr DD two_sum(double a, double b) {
        const double s = a + b, v = s - a;
        return {s, (a - (s - v)) + (b - v)};
    }
    static constexpr DD two_prod(double a, double b) {   // Dekker
        const double ca = 134217729.0 * a, ah = ca - (ca - a), al = a - ah;
        const double cb = 134217729.0 * b, bh = cb - (cb - b), bl = b - bh;
        const double p = a * b;
        return {p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
    }
    static constexpr DD add(DD a, DD b) {
        const DD s = two_sum(a.h, b.h);
        return two_sum(s.h, s.l + a.l + b.l);
    }
    static constexpr DD mul(DD a, DD b) {
        const DD p = two_prod(a.h, b.h);
        return two_sum(p.h, p.l + a.h * b.l + a.l * b.h);
    }
    static constexpr DD div(DD a, DD b) {
        const double q = a.h / b.h;
        const DD m = mul(b, {q, 0.0});
        const DD r = add(a, {-m.h, -m.l});
        return two_sum(q, r.h / b.h);
    }
    // ln v for v near 1 as 2 atanh((v - 1) / (v + 1))
    static constexpr double ln(double v) {
        const DD s = div(two_sum(v, -1.0), two_sum(v, 1.0)), z = mul(s, s);
        DD p = s, sum = {0.0, 0.0};
        for (int k = 1; k <= 41; k += 2) {
            sum = add(sum, div(p, {(double)k, 0.0}));
            p = mul(p, z);
        }
        return 2.0 * (sum.h + sum.l);
    }
    static constexpr double value(int hi) {   // the double whose high word is hi
        return hi < 0x3ff00000 ? 0.5 * (1.0 + (double)(hi - 0x3fe00000) / 1048576.0)
                               : 1.0 + (double)(hi - 0x3ff00000) / 1048576.0;
    }
    constexpr LnTable() : t() {
        for (int i = 0; i < LN_BINS; i++) {
            const int h0 = LN_OFF + i * 4096;
            const double c = 0.5 * (value(h0) + value(h0 + 4096));
            t[i].inv = i == LN_ONE_BIN ? 1.0 : 1.0 / c;
            t[i].ln = i == LN_ONE_BIN ? 0.0 : -ln(t[i].inv);
        }
    }
};
static __device__ const LnTable LN_TABLE{};

// Copies the table into LDS; the caller synchronises the workgroup before use.
__device__ __forceinline__ void load_ln_table(LnEntry *tab) {
    for (int i = threadIdx.x; i < LN_BINS; i += blockDim.x) tab[i] = LN_TABLE.t[i];
}

// x must be a positive normal double (any other value gives an unspecified
// number; the table index stays in range).
// eoff is added to its binary exponent.
__device__ __forceinline__ double ln_normal(double x, const LnEntry *tab, int eoff = 0) {
    const int hi = __double2hiint(x);
    const int t = hi - LN_OFF;
    const LnEntry en = tab[(t >> 12) & (LN_BINS - 1)];
    const double z = __hiloint2double(hi - (t & (int)0xfff00000), __double2loint(x));
    const double r = fma(z, en.inv, -1.0);
    const double r2 = r * r;
    double q = fma3s(r, -1.0 / 6.0, 1.0 / 5.0);
    q = fma3s(q, r, -1.0 / 4.0);
    q = fma3s(q, r, 1.0 / 3.0);
    q = fma3s(q, r, -0.5);
    const double b = fma((double)((t >> 20) + eoff), 6.93147180559945309417e-01, en.ln);
    return b + fma(r2, q, r);
}

// A probability that leaves the common path: zero, subnormal, infinite, NaN.
__device__ __forceinline__ unsigned rare_key(double p) { return (unsigned)__double2hiint(p) - 0x00100000u; }
constexpr unsigned RARE_KEY = 0x7fe00000u;   // key >= RARE_KEY: not a positive normal number

// Logarithm of a rare value for the sums of the statistics: 0 for p = 0 or
// NaN (counted in zeros).
__device__ __forceinline__ double ln_rare(double p, unsigned &zeros, const LnEntry *tab) {
    const double sub = ln_normal(p * 18014398509481984.0, tab, -54);   // subnormals, scaled by 2^54
    const bool pos = p > 0.0;
    zeros += pos ? 0u : 1u;
    return pos ? (p > 1.0 ? p : sub) : 0.0;   // p > 1: infinite
}
__device__ __forceinline__ double ln_prob(double p, unsigned &zeros, const LnEntry *tab) {
    if (rare_key(p) < RARE_KEY) return ln_normal(p, tab);
    return ln_rare(p, zeros, tab);
}

// Adds one probability p to the one-pass statistics: acc = {S, sum p ln p,
// sum ln p, -, sum u^k for k = 2..10} with u = N p, and counts p = 0 (those
// contribute 0 to both log sums).  The powers are products of u..u^5, each
// fused into its sum: 4 multiplications and 9 multiply-adds where a running
// power takes 10 and 10.  N is a power of two, so sum u = N S exactly
// (stat_finish); it is not summed.
__device__ __forceinline__ void stat_add_ln(double (&acc)[NSTAT], double p, double l, double Nd) {
    acc[0] += p;
    acc[1] = fma(p, l, acc[1]);
    acc[2] += l;
    const double u = Nd * p;
    const double u2 = u * u, u3 = u2 * u, u4 = u2 * u2, u5 = u3 * u2;
    acc[4] = fma(u, u, acc[4]);
    acc[5] = fma(u2, u, acc[5]);
    acc[6] = fma(u2, u2, acc[6]);
    acc[7] = fma(u3, u2, acc[7]);
    acc[8] = fma(u3, u3, acc[8]);
    acc[9] = fma(u4, u3, acc[9]);
    acc[10] = fma(u4, u4, acc[10]);
    acc[11] = fma(u5, u4, acc[11]);
    acc[12] = fma(u5, u5, acc[12]);
}
__device__ __forceinline__ void stat_add(double (&acc)[NSTAT], unsigned &zeros, double p, double Nd,
                                         const LnEntry *tab) {
    stat_add_ln(acc, p, ln_prob(p, zeros, tab), Nd);
}
// K probabilities per lane: one wave-wide test for the rare values, so that
// the common path has no branch between the K independent chains.
template <int K>
__device__ __forceinline__ void stat_add_n(double (&acc)[NSTAT], unsigned &zeros, const double (&p)[K], double Nd,
                                           const LnEntry *tab) {
    unsigned key = 0;
    double l[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        key = max(key, rare_key(p[k]));
        l[k] = ln_normal(p[k], tab);
    }
    if (__ballot(key >= RARE_KEY) != 0ull) {
#pragma unroll
        for (int k = 0; k < K; k++)
            if (rare_key(p[k]) >= RARE_KEY) l[k] = ln_rare(p[k], zeros, tab);
    }
#pragma unroll
    for (int k = 0; k < K; k++) stat_add_ln(acc, p[k], l[k], Nd);
}
__device__ __forceinline__ void stat_finish(double (&acc)[NSTAT], double Nd) { acc[3] = Nd * acc[0]; }

}  // namespace svi
