// Reductions over the output distribution p(x) = |<x|psi>|^2 (Sec. II):
// probabilities, the one-pass statistics (entropy, uniform cross entropy,
// normalised moments), the integer-CDF sampler and the sample cross entropy.
//
// Everything here is HBM-streaming: one read of the state per statistic
// pass, at most two for the sampler.  Floating-point sums are formed in
// FP64 per thread, reduced by fixed shuffle trees inside a workgroup and
// combined across workgroups in workgroup order with Neumaier's
// compensated summation, so results are deterministic for a given size.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "internal.h"
#include "reduce_common.h"

namespace svi {

// ---------------------------------------------------------------------------
// probabilities
// ---------------------------------------------------------------------------
template <typename T, typename O>
__global__ __launch_bounds__(RB) void k_probs(const cpx<T> *__restrict__ psi, uint64_t begin,
                                              uint64_t count, O *__restrict__ out) {
    uint64_t stride = (uint64_t)gridDim.x * RB;
    for (uint64_t i = (uint64_t)blockIdx.x * RB + threadIdx.x; i < count; i += stride)
        out[i] = (O)prob_of(psi[begin + i]);
}

// ---------------------------------------------------------------------------
// statistics: per workgroup S, sum p ln p, sum ln p, sum u^k (k = 1..10),
// zero count; u = N p
// ---------------------------------------------------------------------------

// Bound by HBM once an amplitude takes about 45 VALU issues (the table
// logarithm and the shared powers of stat_add; it was FP64-bound at about 75).
// The next UNR amplitudes of a thread are loaded before the current ones are
// used.  chunk is a multiple of RB * UNR or, for the smallest states, less.
template <typename T, bool FULL>
__global__ __launch_bounds__(RB) void k_stats(const cpx<T> *__restrict__ psi, uint64_t chunk,
                                              double Nd, double *__restrict__ part) {
    __shared__ double red[4 * NSTAT];
    __shared__ unsigned zred[4];
    __shared__ LnEntry tab[FULL ? LN_BINS : 1];
    constexpr int UNR = 4;
    const uint64_t start = (uint64_t)blockIdx.x * chunk;
    const uint64_t end = start + chunk, main_end = end - chunk % (RB * UNR);
    uint64_t j0 = start + threadIdx.x;
    cpx<T> buf[UNR], nxt[UNR];
    if (j0 < main_end) {
#pragma unroll
        for (int u = 0; u < UNR; u++) buf[u] = psi[j0 + (uint64_t)u * RB];
    }
    if (FULL) {
        load_ln_table(tab);
        __syncthreads();
    }
    double acc[NSTAT];
#pragma unroll
    for (int i = 0; i < NSTAT; i++) acc[i] = 0.0;
    unsigned zeros = 0;
    for (; j0 < main_end; j0 += RB * UNR) {
        const uint64_t jn = j0 + RB * UNR < main_end ? j0 + RB * UNR : j0;
#pragma unroll
        for (int u = 0; u < UNR; u++) nxt[u] = psi[jn + (uint64_t)u * RB];
        double p[UNR];
#pragma unroll
        for (int u = 0; u < UNR; u++) p[u] = prob_of(buf[u]);
        if constexpr (FULL) {
            stat_add_n<UNR>(acc, zeros, p, Nd, tab);
        } else {
#pragma unroll
            for (int u = 0; u < UNR; u++) acc[0] += p[u];
        }
#pragma unroll
        for (int u = 0; u < UNR; u++) buf[u] = nxt[u];
    }
    for (uint64_t j = main_end + threadIdx.x; j < end; j += RB) {
        const double p = prob_of(psi[j]);
        if (FULL) stat_add(acc, zeros, p, Nd, tab);
        else acc[0] += p;
    }
    stat_finish(acc, Nd);
    if constexpr (FULL) {
        block_sum<double, NSTAT>(acc, red);
    } else {
        double s1[1] = {acc[0]};
        block_sum<double, 1>(s1, red);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    zeros = wave_sum(zeros);
    if (lane == 0) zred[wave] = zeros;
    __syncthreads();
    if (threadIdx.x < (FULL ? NSTAT : 1)) part[(uint64_t)blockIdx.x * 16 + threadIdx.x] = red[threadIdx.x];
    if (threadIdx.x == NSTAT) {
        const unsigned long long z = (unsigned long long)zred[0] + zred[1] + zred[2] + zred[3];
        part[(uint64_t)blockIdx.x * 16 + NSTAT] = (double)z;
    }
}

// Combine per-workgroup partial rows (16 doubles each), quantity q =
// 0..nq-1, in a fixed order.
__global__ __launch_bounds__(CMB_THREADS) void k_combine(const double *__restrict__ part, int nblocks, int nq,
                                                         double *__restrict__ out) {
    __shared__ double red[2 * 64 * 16];
    combine_rows_wg(part, nblocks, nq, out, red);
}

static void stats_grid(int n, int *nblocks, uint64_t *chunk) {
    const uint64_t N = 1ull << n;
    // four amplitudes per thread at least; 2^21 amplitudes fill the chip's
    // 2048 workgroup slots
    uint64_t nb = N >> 10;
    if (nb < 1) nb = 1;
    if (nb > STATS_BLOCKS) nb = STATS_BLOCKS;
    *nblocks = (int)nb;
    *chunk = N / nb;
}

// Waits for the stream; the result block res (the slot's, or device memory) is
// then in dst.
static sv_status fetch_result(ResultSlot &slot, void *dst, const void *res, size_t bytes, hipStream_t s) {
    if (!slot.ptr) SV_HIP(hipMemcpyAsync(dst, res, bytes, hipMemcpyDeviceToHost, s));
    SV_HIP(hipStreamSynchronize(s));
    if (slot.ptr) {
        std::memcpy(dst, slot.ptr, bytes);
        slot.release();
    }
    return SV_OK;
}

template <typename T, bool FULL>
static sv_status stats_typed(sv_state *st, const void *psi, double *host16) {
    int nb;
    uint64_t chunk;
    stats_grid(st->n, &nb, &chunk);
    SV_TRY(st->ws.reserve((size_t)(nb + 1) * 16 * sizeof(double)));
    double *part = (double *)st->ws.ptr;
    ResultSlot slot(16 * sizeof(double), st->stream);
    double *res = slot.ptr ? (double *)slot.ptr : part + (size_t)nb * 16;
    hipLaunchKernelGGL((k_stats<T, FULL>), dim3(nb), dim3(RB), 0, st->stream, (const cpx<T> *)psi,
                       chunk, std::ldexp(1.0, st->n), part);
    SV_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_combine, dim3(1), dim3(CMB_THREADS), 0, st->stream, part, nb, FULL ? NSTAT + 1 : 1, res);
    SV_HIP(hipGetLastError());
    SV_TRY(fetch_result(slot, host16, res, 16 * sizeof(double), st->stream));
    return SV_OK;
}

// The normalised statistics from the combined sums r (S, sum p ln p,
// sum ln p, sum u^k, zero count) of a 2^n-amplitude state.
static void finish_stats(int n, const double *r, sv_stats *out) {
    const double N = std::ldexp(1.0, n);
    const double S = r[0];
    const double lnS = std::log(S);
    out->norm = S;
    out->entropy = lnS - r[1] / S;
    out->zero_count = (int64_t)r[NSTAT];
    out->unif_ce = out->zero_count ? INFINITY : lnS - r[2] / N;
    double Sk = 1.0;
    for (int k = 0; k < 10; k++) {
        Sk *= S;
        out->moments[k] = r[3 + k] / N / Sk;
    }
}

void finish_stats_row(int n, const double *r, sv_stats *out) { finish_stats(n, r, out); }

sv_status run_stats(sv_state *st, const void *psi, sv_stats *out) {
    double r[16] = {0};
    if (st->dt == SV_C64) SV_TRY((stats_typed<float, true>(st, psi, r)));
    else SV_TRY((stats_typed<double, true>(st, psi, r)));
    finish_stats(st->n, r, out);
    return SV_OK;
}

// Enqueue the statistics pass of st into res[0..14) without synchronising
// (used inside captured graphs); part holds up to 2048 partial rows.
sv_status stats_rows_enqueue(sv_state *st, double *part, int *nrows) {
    uint64_t chunk;
    stats_grid(st->n, nrows, &chunk);
    if (st->dt == SV_C64)
        hipLaunchKernelGGL((k_stats<float, true>), dim3(*nrows), dim3(RB), 0, st->stream,
                           (const cpx<float> *)st->data, chunk, std::ldexp(1.0, st->n), part);
    else
        hipLaunchKernelGGL((k_stats<double, true>), dim3(*nrows), dim3(RB), 0, st->stream,
                           (const cpx<double> *)st->data, chunk, std::ldexp(1.0, st->n), part);
    SV_HIP(hipGetLastError());
    return SV_OK;
}

sv_status batch_stats_enqueue(sv_state *st, double *part, double *res) {
    int nb;
    SV_TRY(stats_rows_enqueue(st, part, &nb));
    hipLaunchKernelGGL(k_combine, dim3(1), dim3(CMB_THREADS), 0, st->stream, part, nb, NSTAT + 1, res);
    SV_HIP(hipGetLastError());
    return SV_OK;
}

__global__ __launch_bounds__(CMB_THREADS) void k_combine_lists(const double *__restrict__ part, size_t stride,
                                                               const int *__restrict__ rows,
                                                               double *__restrict__ res) {
    __shared__ double red[2 * 64 * 16];
    combine_rows_wg(part + stride * blockIdx.x, rows[blockIdx.x], NSTAT + 1, res + 16 * (uint64_t)blockIdx.x, red);
}

sv_status combine_lists_enqueue(sv_state *st, const double *part, size_t stride, const int *dev_rows, int64_t count,
                                double *res) {
    if (count == 0) return SV_OK;
    hipLaunchKernelGGL(k_combine_lists, dim3((unsigned)count), dim3(CMB_THREADS), 0, st->stream, part, stride,
                       dev_rows, res);
    SV_HIP(hipGetLastError());
    return SV_OK;
}

sv_status run_norm(sv_state *st, const void *psi, double *S) {
    double r[16] = {0};
    if (st->dt == SV_C64) SV_TRY((stats_typed<float, false>(st, psi, r)));
    else SV_TRY((stats_typed<double, false>(st, psi, r)));
    *S = r[0];
    return SV_OK;
}

sv_status run_probs(sv_state *st, uint64_t begin, uint64_t count, int f64, void *out) {
    if (!count) return SV_OK;
    uint64_t g = (count + RB - 1) / RB;
    unsigned grid = (unsigned)(g < 16384 ? g : 16384);
    if (st->dt == SV_C64) {
        if (f64) hipLaunchKernelGGL((k_probs<float, double>), dim3(grid), dim3(RB), 0, st->stream,
                                    (const cpx<float> *)st->data, begin, count, (double *)out);
        else hipLaunchKernelGGL((k_probs<float, float>), dim3(grid), dim3(RB), 0, st->stream,
                                (const cpx<float> *)st->data, begin, count, (float *)out);
    } else {
        if (f64) hipLaunchKernelGGL((k_probs<double, double>), dim3(grid), dim3(RB), 0, st->stream,
                                    (const cpx<double> *)st->data, begin, count, (double *)out);
        else hipLaunchKernelGGL((k_probs<double, float>), dim3(grid), dim3(RB), 0, st->stream,
                                (const cpx<double> *)st->data, begin, count, (float *)out);
    }
    SV_HIP(hipGetLastError());
    return SV_OK;
}

// w = floor(p 2^62): the scaling by a power of two is exact and the
// conversion truncates toward zero.
__device__ __forceinline__ uint64_t weight_of(double p) {
    return (uint64_t)(p * 4611686018427387904.0);
}

// floor(p 2^62) of 0 <= p < 2 by one 64-bit shift of the mantissa (zeros and
// subnormals give 0); any p through weight_of where a wave holds a larger one.
// The conversion instructions of weight_of take twice the issues.
__device__ __forceinline__ uint64_t weight_below2(double p) {
    const unsigned hi = (unsigned)__double2hiint(p), lo = (unsigned)__double2loint(p);
    const uint64_t m = ((uint64_t)((hi & 0xfffffu) | 0x100000u) << 32 | lo) << 10;   // p = m 2^(e - 1085)
    const unsigned sh = 1023u - (hi >> 20);
    return m >> (sh < 63u ? sh : 63u);
}
__device__ __forceinline__ bool weight_is_large(double p) { return (unsigned)__double2hiint(p) >= 0x40000000u; }

// ---------------------------------------------------------------------------
// pair statistics of an ideal output a and another output b
// ---------------------------------------------------------------------------
// Per workgroup, in FP64: S_a, S_b, Re and Im of sum conj(a) b, sum p_a^2,
// sum p_b^2, sum p_a p_b, sum over p_a > 0 of p_b ln p_a and of ln p_a, sum
// over p_a = 0 of p_b; and the number of p_a = 0.  With nbins > 0, the
// histogram of z = ln(N p_a): the slot of x is decided by comparing p_a with
// the thresholds thr[0..nbins] (bin j: thr[j] <= p_a < thr[j+1]; nbins:
// below thr[0] or p_a = 0; nbins + 1: at or above thr[nbins]), starting from
// the bin that ln p_a falls into, and the slot gets the count and the integer
// masses floor(p 2^62) of both outputs (64-bit integer sums: exact, in any
// order) in LDS; the workgroup writes them as one row of hcols words.
// The slots of one wavefront's outcomes collide (most of a Porter-Thomas
// output lies in a few bins), so each slot has `copies` LDS words, one per
// lane modulo copies.  Small states are bound by latency: four outcomes per
// thread at least (2^20 amplitudes run on 1024 workgroups; 4096 outcomes per
// workgroup took 24 us).
constexpr int NPAIR = 10;
constexpr int PAIR_INLINE = 256;      // thresholds that travel as kernel arguments
struct PairThr { double t[PAIR_INLINE]; };

template <typename T, bool HIST>
__global__ __launch_bounds__(RB) void k_pair_stats(const cpx<T> *__restrict__ a, const cpx<T> *__restrict__ b,
                                                   uint64_t chunk, const double *__restrict__ thr, PairThr inl,
                                                   int nbins, int copies, double l0, double inv_dz,
                                                   double *__restrict__ part, unsigned long long *__restrict__ hrows,
                                                   int hcols) {
    __shared__ double red[4 * NPAIR];
    __shared__ unsigned zred[4];
    __shared__ LnEntry tab[LN_BINS];
    extern __shared__ unsigned long long dyn[];   // nbins + 1 thresholds, 3 nslot copies words
    const int nslot = nbins + 2, nw = 3 * nslot * copies;
    double *const sthr = (double *)dyn;
    unsigned long long *const sh = dyn + nbins + 1;
    constexpr int UNR = 4;
    const uint64_t start = (uint64_t)blockIdx.x * chunk;
    const uint64_t end = start + chunk;
    cpx<T> av[UNR], bv[UNR];
    // entries past the end of a small state's chunk read its last entry and
    // are left out below
    auto load4 = [&](uint64_t j0) {
#pragma unroll
        for (int u = 0; u < UNR; u++) {
            const uint64_t j = j0 + (uint64_t)u * RB;
            av[u] = a[j < end ? j : end - 1];
            bv[u] = b[j < end ? j : end - 1];
        }
    };
    uint64_t j0 = start + threadIdx.x;
    load4(j0);
    load_ln_table(tab);
    if constexpr (HIST) {
        for (int i = threadIdx.x; i <= nbins; i += RB) sthr[i] = thr ? thr[i] : inl.t[i];
        for (int i = threadIdx.x; i < nw; i += RB) sh[i] = 0ull;
    }
    __syncthreads();
    double acc[NPAIR];
#pragma unroll
    for (int i = 0; i < NPAIR; i++) acc[i] = 0.0;
    unsigned zeros = 0;
    const int cp = threadIdx.x & (copies - 1);
    for (uint64_t base = start; base < end; base += RB * UNR, j0 += RB * UNR) {
        cpx<T> ca[UNR], cb[UNR];
#pragma unroll
        for (int u = 0; u < UNR; u++) { ca[u] = av[u]; cb[u] = bv[u]; }
        load4(base + RB * UNR < end ? j0 + RB * UNR : j0);
#pragma unroll
        for (int u = 0; u < UNR; u++) {
            if (j0 + (uint64_t)u * RB >= end) continue;
            const double ar = ca[u].re, ai = ca[u].im, br = cb[u].re, bi = cb[u].im;
            const double pa = prob_of(ca[u]), pb = prob_of(cb[u]);
            acc[0] += pa;
            acc[1] += pb;
            acc[2] += fma(ar, br, ai * bi);
            acc[3] += fma(ar, bi, -ai * br);
            acc[4] = fma(pa, pa, acc[4]);
            acc[5] = fma(pb, pb, acc[5]);
            acc[6] = fma(pa, pb, acc[6]);
            const double l = ln_prob(pa, zeros, tab);
            acc[7] = fma(pb, l, acc[7]);
            acc[8] += l;
            acc[9] += pa > 0.0 ? 0.0 : pb;
            if constexpr (HIST) {
                int slot;
                if (!(pa >= sthr[0])) {
                    slot = nbins;
                } else if (pa >= sthr[nbins]) {
                    slot = nbins + 1;
                } else {   // thr[0] <= p_a < thr[nbins]: both walks end inside
                    const double z = (l - l0) * inv_dz;
                    slot = z > 0.0 ? (z < (double)nbins ? (int)z : nbins - 1) : 0;
                    slot = slot < nbins ? slot : nbins - 1;
                    while (pa < sthr[slot]) slot--;
                    while (pa >= sthr[slot + 1]) slot++;
                }
                // the host rejects the histogram when a norm reaches 4, so a
                // weight that would not fit is never reported
                unsigned long long wa = weight_below2(pa), wb = weight_below2(pb);
                if (weight_is_large(pa)) wa = pa < 4.0 ? weight_of(pa) : 0ull;
                if (weight_is_large(pb)) wb = pb < 4.0 ? weight_of(pb) : 0ull;
                atomicAdd(&sh[slot * copies + cp], 1ull);
                atomicAdd(&sh[(nslot + slot) * copies + cp], wa);
                atomicAdd(&sh[(2 * nslot + slot) * copies + cp], wb);
            }
        }
    }
    block_sum<double, NPAIR>(acc, red);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    zeros = wave_sum(zeros);
    if (lane == 0) zred[wave] = zeros;
    __syncthreads();
    if (threadIdx.x < NPAIR) part[(uint64_t)blockIdx.x * 16 + threadIdx.x] = red[threadIdx.x];
    if (threadIdx.x == NPAIR) {
        const unsigned long long z = (unsigned long long)zred[0] + zred[1] + zred[2] + zred[3];
        part[(uint64_t)blockIdx.x * 16 + NPAIR] = (double)z;
    }
    if constexpr (HIST) {
        for (int i = threadIdx.x; i < 3 * nslot; i += RB) {
            unsigned long long s = 0;
            for (int k = 0; k < copies; k++) s += sh[i * copies + k];
            hrows[(uint64_t)blockIdx.x * hcols + i] = s;
        }
    }
}

// The combined sums (workgroup 0) and the histogram (workgroups 1 up, 16
// columns of the rows each) into one block: 16 doubles, then the words.
__global__ __launch_bounds__(CMB_THREADS) void k_pair_finish(const double *__restrict__ part,
                                                             const unsigned long long *__restrict__ hrows, int hcols,
                                                             int nwords, int nblocks, double *__restrict__ out) {
    __shared__ unsigned long long red[2 * 64 * 16];
    if (blockIdx.x == 0) {
        combine_rows_wg(part, nblocks, NPAIR + 1, out, (double *)red);
        return;
    }
    const int q = threadIdx.x & 15, seg = threadIdx.x >> 4;
    const int col = (blockIdx.x - 1) * 16 + q;   // below hcols, a multiple of 16
    unsigned long long s = 0;
    if (col < nwords) {
#pragma unroll 8
        for (int r = seg; r < nblocks; r += 64) s += hrows[(uint64_t)r * hcols + col];
    }
    red[threadIdx.x] = s;
#pragma unroll
    for (int h = 32; h >= 1; h >>= 1) {
        __syncthreads();
        if (seg < h) red[threadIdx.x] += red[threadIdx.x + h * 16];
    }
    if (seg == 0 && col < nwords) ((unsigned long long *)(out + 16))[col] = red[q];
}

sv_status run_pair_stats(sv_state *a, sv_state *b, int nbins, double zmin, double zmax, const double *host_thr,
                         double *sums16, uint64_t *host_hist) {
    int nb;
    uint64_t chunk;
    stats_grid(a->n, &nb, &chunk);
    const int nwords = nbins > 0 ? 3 * (nbins + 2) : 0, hcols = (nwords + 15) & ~15;
    // histogram rows of at most 16 MiB in all
    while (nb > 256 && (int64_t)nb * hcols > ((int64_t)1 << 21)) { nb >>= 1; chunk <<= 1; }
    int copies = 16;   // at most 16 KiB of histogram words per workgroup, or one copy
    while (copies > 1 && nwords * copies > 2048) copies >>= 1;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t o_part = 0, o_res = al((size_t)nb * 16 * 8), o_thr = o_res + al(16 * 8 + (size_t)nwords * 8),
                 o_rows = o_thr + al((size_t)(nbins + 1) * 8), need = o_rows + al((size_t)nb * hcols * 8);
    SV_TRY(a->ws.reserve(need));
    uint8_t *w = (uint8_t *)a->ws.ptr;
    double *part = (double *)(w + o_part), *res = (double *)(w + o_res), *thr = nullptr;
    auto *rows = (unsigned long long *)(w + o_rows);
    hipStream_t s = a->stream;
    PairThr inl{};
    if (nbins >= PAIR_INLINE) {
        thr = (double *)(w + o_thr);
        SV_HIP(hipMemcpyAsync(thr, host_thr, (size_t)(nbins + 1) * 8, hipMemcpyHostToDevice, s));
    } else {
        for (int i = 0; i <= nbins && nbins > 0; i++) inl.t[i] = host_thr[i];
    }
    const double l0 = zmin - a->n * 0.69314718055994530942, inv_dz = nbins > 0 ? nbins / (zmax - zmin) : 0.0;
    const size_t lds = nbins > 0 ? ((size_t)nbins + 1 + (size_t)nwords * copies) * 8 : 0;
#define PAIR_LAUNCH(T, HIST)                                                                                        \
    hipLaunchKernelGGL((k_pair_stats<T, HIST>), dim3(nb), dim3(RB), lds, s, (const cpx<T> *)a->data,                \
                       (const cpx<T> *)b->data, chunk, thr, inl, nbins, copies, l0, inv_dz, part, rows, hcols)
    if (a->dt == SV_C64) {
        if (nbins > 0) PAIR_LAUNCH(float, true);
        else PAIR_LAUNCH(float, false);
    } else {
        if (nbins > 0) PAIR_LAUNCH(double, true);
        else PAIR_LAUNCH(double, false);
    }
#undef PAIR_LAUNCH
    SV_HIP(hipGetLastError());
    std::vector<uint64_t> host((size_t)16 + nwords);
    ResultSlot slot(host.size() * 8, s);
    if (slot.ptr) res = (decltype(res))slot.ptr;
    hipLaunchKernelGGL(k_pair_finish, dim3(1 + hcols / 16), dim3(CMB_THREADS), 0, s, part, rows, hcols, nwords, nb, res);
    SV_HIP(hipGetLastError());
    SV_TRY(fetch_result(slot, host.data(), res, host.size() * 8, s));
    std::memcpy(sums16, host.data(), (NPAIR + 1) * sizeof(double));
    if (nwords) std::memcpy(host_hist, host.data() + 16, (size_t)nwords * 8);
    return SV_OK;
}

// ---------------------------------------------------------------------------
// sampler (integer CDF)
// ---------------------------------------------------------------------------

__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// The sampler's weight sums form four levels: groups of chunks (at most 8192,
// with their exclusive prefix), chunks of 2^bs entries, at most 64 sub-buckets
// of 2^sb entries per chunk, entries.  Sums are exact 64-bit integers, so a
// sample does not depend on how the levels are cut.
//
// One wavefront sums whole chunks (no barrier) in units of UNIT entries: a row
// of 16 lanes takes the 256 entries of one smallest sub-bucket, 16 at a time
// (a 128-byte line of complex64 amplitudes per row and load), so a
// sub-bucket's sum is a row sum.  Chunks are small enough that a state of 2^23 entries still gives 8192
// wavefronts work: with 2^16-entry buckets, one workgroup each, the 16-qubit
// pass ran on one workgroup (62 us) and the 20-qubit one on 16.
constexpr int UNIT_BITS = 10, UNIT = 1 << UNIT_BITS;
constexpr int PASS_BLOCKS = 2048;      // workgroups of a pass at most
constexpr int MAX_GROUPS = 8192;
constexpr int64_t RESOLVE_SLICE = (int64_t)1 << 25;   // samples per launch

template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_u64(unsigned long long v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROWS, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xF, false);
    return ((unsigned long long)hi << 32) | lo;
}
// Inclusive prefix sum over the 64 lanes (lane order): shifts within rows of
// 16 lanes, then the row totals broadcast to the following rows.
__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v) {
    v += dpp_u64<0x111, 0xF>(v);   // row_shr 1, 2, 4, 8
    v += dpp_u64<0x112, 0xF>(v);
    v += dpp_u64<0x114, 0xF>(v);
    v += dpp_u64<0x118, 0xF>(v);
    v += dpp_u64<0x142, 0xA>(v);   // lane 15 of rows 0 and 2 to rows 1 and 3
    v += dpp_u64<0x143, 0xC>(v);   // lane 31 to rows 2 and 3
    return v;
}
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int lane) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), lane);
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v) {
    return lane_u64(wave_incl_scan_u64(v), 63);
}
// Sum over the 16 lanes of a row, in every lane of the row.
__device__ __forceinline__ unsigned long long row_sum_u64(unsigned long long v) {
    v += dpp_u64<0xB1, 0xF>(v);    // quad_perm 1,0,3,2
    v += dpp_u64<0x4E, 0xF>(v);    // quad_perm 2,3,0,1
    v += dpp_u64<0x141, 0xF>(v);   // half-row mirror
    v += dpp_u64<0x140, 0xF>(v);   // row mirror
    return v;
}
// Sum of rows 0, 1 and of rows 2, 3; then of all four.
__device__ __forceinline__ unsigned long long row_pair_sum_u64(unsigned long long v) {
    const unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return (((unsigned long long)h[0] << 32) | l[0]) + (((unsigned long long)h[1] << 32) | l[1]);
}
__device__ __forceinline__ unsigned long long half_sum_u64(unsigned long long v) {
    const unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
    const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return (((unsigned long long)h[0] << 32) | l[0]) + (((unsigned long long)h[1] << 32) | l[1]);
}

// What a pass over 2^n entries leaves besides the sums: the 14 statistic sums
// and the total weight with a status.
enum { PASS_OK = 0, PASS_BAD = 1, PASS_OVERFLOW = 2, PASS_ZERO = 3 };
struct PassResult {
    double stats[16];
    unsigned long long W;
    unsigned long long status;
    unsigned long long pad[6];
};

// The pass.  STATS: every amplitude also enters this workgroup's row of
// statistic sums.  CHECK (explicit distributions): entries outside [0, 4) are
// flagged and the weights summed exactly in halves (high and low 32 bits; a
// workgroup holds at most 2^24 of them), row = {high, low, flag, 0}.  Entries
// at index >= N (a length that is not a power of two) have weight 0 and are
// not read.  Without STATS the pass is bound by HBM.
template <typename S, bool STATS, bool CHECK>
__global__ __launch_bounds__(RB) void k_pass(const S *__restrict__ src, uint64_t N, int bs, int sb, uint64_t nb,
                                             double Nd, double *__restrict__ part,
                                             unsigned long long *__restrict__ csum,
                                             unsigned long long *__restrict__ subsum) {
    __shared__ double red[STATS ? 4 * NSTAT : 1];
    __shared__ unsigned zred[4];
    __shared__ unsigned long long chk[4 * 3];
    __shared__ LnEntry tab[STATS ? LN_BINS : 1];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr (STATS) {
        load_ln_table(tab);
        __syncthreads();
    }
    double acc[NSTAT];
#pragma unroll
    for (int i = 0; i < NSTAT; i++) acc[i] = 0.0;
    unsigned zeros = 0;
    unsigned long long chigh = 0, clow = 0;
    unsigned bad = 0;
    const int steps = 1 << (bs - UNIT_BITS + 2);   // of 256 entries, four to a unit
    const int row = lane >> 4;
    const int first = 256 * row + (lane & 15);   // this lane's first entry of a unit, then every 16th
    // one chunk; FULL: none of its entries lies beyond N (two copies, since a
    // branch around the loads makes the loop wait for them at once)
    auto chunk = [&](uint64_t c, auto full) {
        constexpr bool FULL = decltype(full)::value;
        const uint64_t start = c << bs;
        auto entry = [&](int st, int j) { return start + ((uint64_t)(st >> 2) << UNIT_BITS) + first + 64 * (st & 3) + 16 * j; };
        auto load4 = [&](int st, S (&e)[4]) {
#pragma unroll
            for (int j = 0; j < 4; j++)
                if (FULL || entry(st, j) < N) e[j] = src[entry(st, j)];
                else e[j] = S{};
        };
        unsigned long long cs = 0;   // this row's share of the chunk
        unsigned long long w = 0;
        S buf[4], nxt[4];
        load4(0, buf);
#pragma unroll 1
        for (int st = 0; st < steps; st++) {
            load4(st + 1 < steps ? st + 1 : st, nxt);
            double p[4];
            bool large = false;
#pragma unroll
            for (int j = 0; j < 4; j++) {
                p[j] = prob_of(buf[j]);
                if constexpr (CHECK) {
                    const bool ok = (p[j] >= 0.0) & (p[j] < 4.0);
                    bad |= ok ? 0u : 1u;
                    p[j] = ok ? p[j] : 0.0;
                }
                large |= weight_is_large(p[j]);
            }
            unsigned long long x[4];
#pragma unroll
            for (int j = 0; j < 4; j++) x[j] = weight_below2(p[j]);
            if (__ballot(large) != 0ull) {
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (weight_is_large(p[j])) x[j] = weight_of(p[j]);
            }
#pragma unroll
            for (int j = 0; j < 4; j++) {
                w += x[j];
                if constexpr (CHECK) { chigh += x[j] >> 32; clow += x[j] & 0xffffffffull; }
            }
            if constexpr (STATS) {
                stat_add_n<4>(acc, zeros, p, Nd, tab);
                if constexpr (!FULL) {   // entries beyond the state added exact zeros
#pragma unroll
                    for (int j = 0; j < 4; j++) zeros -= entry(st, j) >= N ? 1u : 0u;
                }
            }
#pragma unroll
            for (int j = 0; j < 4; j++) buf[j] = nxt[j];
            if ((st & 3) == 3) {
                // every lane of a row: the sum of its 256 entries, merged up
                // to 2^sb entries
                unsigned long long v = row_sum_u64(w);
                w = 0;
                cs += v;
                if (sb >= 9) v = row_pair_sum_u64(v);
                if (sb >= 10) v = half_sum_u64(v);
                const int rows = 1 << (sb - 8);   // rows per sub-bucket
                if ((lane & (16 * rows - 1)) == 0) subsum[(entry(st - 3, 0) - (lane & 15)) >> sb] = v;
            }
        }
        cs = half_sum_u64(row_pair_sum_u64(cs));
        if (lane == 0) csum[c] = cs;
    };
    for (uint64_t c = (uint64_t)blockIdx.x * (RB / 64) + wave; c < nb; c += (uint64_t)gridDim.x * (RB / 64)) {
        if ((c + 1) << bs <= N) chunk(c, std::true_type{});
        else chunk(c, std::false_type{});
    }
    if constexpr (STATS) {
        stat_finish(acc, Nd);
        block_sum<double, NSTAT>(acc, red);
        zeros = wave_sum(zeros);
        if (lane == 0) zred[wave] = zeros;
        __syncthreads();
        if (threadIdx.x < NSTAT) part[(uint64_t)blockIdx.x * 16 + threadIdx.x] = red[threadIdx.x];
        if (threadIdx.x == NSTAT) {
            const unsigned long long z = (unsigned long long)zred[0] + zred[1] + zred[2] + zred[3];
            part[(uint64_t)blockIdx.x * 16 + NSTAT] = (double)z;
        }
    }
    if constexpr (CHECK) {
        chigh = wave_sum_u64(chigh);
        clow = wave_sum_u64(clow);
        const unsigned long long any = __ballot(bad != 0u) ? 1ull : 0ull;
        if (lane == 0) { chk[wave * 3] = chigh; chk[wave * 3 + 1] = clow; chk[wave * 3 + 2] = any; }
        __syncthreads();
        if (threadIdx.x < 3) {
            auto *row = (unsigned long long *)(part + (uint64_t)blockIdx.x * 16);
            row[threadIdx.x] = chk[threadIdx.x] + chk[3 + threadIdx.x] + chk[6 + threadIdx.x] + chk[9 + threadIdx.x];
        }
    }
}

// Two workgroups: the second combines the statistic rows (nrows > 0); the
// first sums the chunks of each group (cg = 2^k <= 64 chunks) and forms the
// exclusive prefix off[0..ng] of the ng = nb / cg groups, the total W and its
// status (check: from the exact sums of the check rows).  The loads of the
// chunk sums are coalesced rows, four in flight per wavefront.  The status and
// the statistics go to copy (host memory, or res itself).
__global__ __launch_bounds__(CMB_THREADS) void k_finish_pass(const unsigned long long *__restrict__ csum, uint64_t nb,
                                                             int cg, const double *__restrict__ part, int nrows,
                                                             int check, unsigned long long *__restrict__ off,
                                                             PassResult *__restrict__ res,
                                                             PassResult *__restrict__ copy) {
    __shared__ unsigned long long lds[MAX_GROUPS];
    __shared__ unsigned long long wtot[16];
    __shared__ unsigned long long chk[16 * 5];
    if (blockIdx.x == 1) {
        combine_rows_wg(part, nrows, NSTAT + 1, copy->stats, (double *)lds);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ng = (int)(nb / (uint64_t)cg);
    for (uint64_t i0 = (uint64_t)wave * 64; i0 < nb; i0 += 4 * 1024) {
        unsigned long long v[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint64_t i = i0 + (uint64_t)j * 1024 + lane;
            v[j] = i < nb ? csum[i] : 0ull;
        }
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const uint64_t i = i0 + (uint64_t)j * 1024 + lane;
            for (int m = 1; m < cg; m <<= 1) v[j] += __shfl_xor(v[j], m, 64);
            if (i < nb && (lane & (cg - 1)) == 0) lds[i / (uint64_t)cg] = v[j];
        }
    }
    __syncthreads();
    const int per = (ng + 1023) / 1024;
    const int b = tid * per, e = b + per < ng ? b + per : ng;
    unsigned long long s = 0;
    for (int i = b; i < e; i++) s += lds[i];
    const unsigned long long incl = wave_incl_scan_u64(s);
    if (lane == 63) wtot[wave] = incl;
    __syncthreads();
    unsigned long long run = incl - s, W = 0;
    for (int w = 0; w < 16; w++) {
        if (w < wave) run += wtot[w];
        W += wtot[w];
    }
    for (int i = b; i < e; i++) {
        off[i] = run;
        run += lds[i];
    }
    unsigned long long status = PASS_OK;
    if (check) {
        // exact total: sums of the 32-bit halves of the rows' halves
        unsigned long long h1 = 0, h0 = 0, l1 = 0, l0 = 0, bad = 0;
        for (int r = tid; r < check; r += CMB_THREADS) {
            const auto *row = (const unsigned long long *)(part + (uint64_t)r * 16);
            h1 += row[0] >> 32; h0 += row[0] & 0xffffffffull;
            l1 += row[1] >> 32; l0 += row[1] & 0xffffffffull;
            bad += row[2];
        }
        h1 = wave_sum_u64(h1); h0 = wave_sum_u64(h0); l1 = wave_sum_u64(l1); l0 = wave_sum_u64(l0);
        bad = wave_sum_u64(bad);
        if (lane == 0) {
            chk[wave * 5] = h1; chk[wave * 5 + 1] = h0; chk[wave * 5 + 2] = l1; chk[wave * 5 + 3] = l0;
            chk[wave * 5 + 4] = bad;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < 16; w++)
                for (int k = 0; k < 5; k++) chk[k] += chk[w * 5 + k];
            // weights = 2^64 h1 + 2^32 (h0 + l1) + l0
            const bool over = chk[0] != 0ull || ((chk[1] + chk[2] + (chk[3] >> 32)) >> 32) != 0ull;
            status = chk[4] ? PASS_BAD : over ? PASS_OVERFLOW : PASS_OK;
        }
    }
    if (tid == 0) {
        if (status == PASS_OK && W == 0ull) status = PASS_ZERO;
        off[ng] = W;
        res->W = W;
        res->status = status;
        if (copy != res) copy->status = status;
    }
}

// One wavefront per sample first, first + 1, ... < k: t = floor(r W / 2^64),
// then x = min{j : C_j > t} by one 64-wide step per level (group prefix in two,
// chunks, sub-buckets, the four consecutive entries of a lane).  Five dependent loads, and nothing
// is read twice: bound by their latency over the resident wavefronts.  (A
// binary search over the bucket prefix in a kernel of its own, then a serial
// walk of the last 16 entries by one lane, took 0.6 ms for 10^5 samples at 30
// qubits.)
template <typename S, int G>
__global__ __launch_bounds__(RB) void k_resolve(const S *__restrict__ src, uint64_t N, int bs, uint64_t nb, int cg,
                                                const unsigned long long *__restrict__ off,
                                                const unsigned long long *__restrict__ csum,
                                                const unsigned long long *__restrict__ subsum,
                                                const PassResult *__restrict__ res, const uint64_t *__restrict__ words,
                                                uint64_t seed, int64_t first, int64_t k, uint64_t *__restrict__ out) {
    constexpr int sb = G == 1 ? 8 : G == 2 ? 9 : 10;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = first + (int64_t)blockIdx.x * (RB / 64) + wave;
    if (i >= k || res->status != PASS_OK) return;
    const int ng = (int)(nb / (uint64_t)cg);
    const uint64_t r = words ? words[i] : splitmix64(seed, (uint64_t)i);
    const unsigned long long t = __umul64hi(r, res->W);
    // the last group g with off[g] <= t (off[0] = 0): among every s1-th, then
    // among the s1 that follow
    const int s1 = (ng + 63) / 64;
    const int i1 = lane * s1;
    const unsigned long long o1 = i1 < ng ? off[i1] : ~0ull;
    int f = __popcll(__ballot(i1 < ng && o1 <= t)) - 1;
    f = f < 0 ? 0 : f;
    int g = f * s1;
    unsigned long long og = lane_u64(o1, f);
    for (int j = 0; j < s1; j += 64) {
        const int i2 = f * s1 + j + lane;
        const bool in = j + lane < s1 && i2 < ng;
        const unsigned long long o2 = in ? off[i2] : ~0ull;
        const int c2 = __popcll(__ballot(in && o2 <= t));
        if (c2 > 0) {
            g = f * s1 + j + c2 - 1;
            og = lane_u64(o2, c2 - 1);
        }
    }
    unsigned long long tl = t - og;
    // chunk of the group, sub-bucket of the chunk: the first whose inclusive
    // sum exceeds the target (it exists, since the target lies below the
    // total; the clamps keep every access in range all the same)
    const unsigned long long cw = lane < cg ? csum[(uint64_t)g * cg + lane] : 0ull;
    const unsigned long long ci = wave_incl_scan_u64(cw);
    int cl = __ffsll((long long)__ballot(lane < cg && ci > tl)) - 1;
    cl = cl < 0 ? cg - 1 : cl;
    tl -= lane_u64(ci - cw, cl);
    const uint64_t c = (uint64_t)g * cg + cl;
    const int nsub = 1 << (bs - sb);
    const unsigned long long sw = lane < nsub ? subsum[c * nsub + lane] : 0ull;
    const unsigned long long si = wave_incl_scan_u64(sw);
    int sl = __ffsll((long long)__ballot(lane < nsub && si > tl)) - 1;
    sl = sl < 0 ? nsub - 1 : sl;
    tl -= lane_u64(si - sw, sl);
    // entries: lane l holds entries 4 l .. 4 l + 3 of each run of 256
    const uint64_t start = (c << bs) + ((uint64_t)sl << sb);
    unsigned long long w[G][4], own[G];
    if (start + (256 * G) <= N) {
        S e[G][4];
#pragma unroll
        for (int q = 0; q < G; q++)
#pragma unroll
            for (int j = 0; j < 4; j++) e[q][j] = src[start + 256 * q + 4 * lane + j];
#pragma unroll
        for (int q = 0; q < G; q++)
#pragma unroll
            for (int j = 0; j < 4; j++) w[q][j] = weight_of(prob_of(e[q][j]));
    } else {
#pragma unroll
        for (int q = 0; q < G; q++)
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const uint64_t x = start + 256 * q + 4 * lane + j;
                w[q][j] = x < N ? weight_of(prob_of(src[x])) : 0ull;
            }
    }
#pragma unroll
    for (int q = 0; q < G; q++) own[q] = w[q][0] + w[q][1] + w[q][2] + w[q][3];
    bool done = false;
#pragma unroll
    for (int q = 0; q < G; q++) {
        const unsigned long long in = wave_incl_scan_u64(own[q]);
        const unsigned long long total = lane_u64(in, 63);
        if (!done && (total > tl || q == G - 1)) {
            int L = __ffsll((long long)__ballot(in > tl)) - 1;
            L = L < 0 ? 63 : L;
            if (lane == L) {
                unsigned long long s = in - own[q];
                int j = 0;
#pragma unroll
                for (int m = 0; m < 3; m++) {
                    s += w[q][m];
                    j += s <= tl ? 1 : 0;
                }
                out[i] = start + 256 * q + 4 * lane + j;
            }
            done = true;
        }
        if (!done) tl -= total;
    }
}

// Device scratch of the sampler: a workspace grown on demand, or a fixed
// buffer of cap bytes that must already be large enough.
struct ScratchSource {
    Workspace *ws = nullptr;
    void *fixed = nullptr;
    size_t cap = 0;
};

static sv_status take_scratch(const ScratchSource &scr, size_t need, uint8_t **out) {
    if (scr.ws) {
        SV_TRY(scr.ws->reserve(need));
        *out = (uint8_t *)scr.ws->ptr;
        return SV_OK;
    }
    if (need > scr.cap) {
        char b[160];
        snprintf(b, sizeof b, "needs %zu bytes of scratch, the fixed scratch holds %zu", need, scr.cap);
        return fail(SV_ERANGE, b);
    }
    *out = (uint8_t *)scr.fixed;
    return SV_OK;
}

// Layout of the sampler's scratch for 2^n entries: byte offsets of its parts
// and the total.  Sub-buckets of 2^8 entries (2 KiB of complex64 amplitudes
// read per sample) while their sums take at most 32 MiB, then 2^9 and 2^10.
struct SampleLayout {
    int bs, sb, cg;
    uint64_t nb;
    int blocks;
    size_t o_csum, o_off, o_sub, o_part, o_res, need;
};

static SampleLayout sample_layout(int n) {
    SampleLayout L{};
    L.sb = n <= 30 ? 8 : n == 31 ? 9 : 10;
    // chunks: at least a unit, at most 64 sub-buckets, and 8192 of them (a
    // full chip of wavefronts) before they grow
    L.bs = std::min(std::max(UNIT_BITS, n - 13), L.sb + 6);
    L.nb = n > L.bs ? 1ull << (n - L.bs) : 1ull;
    L.cg = 1;
    while (L.nb / (uint64_t)L.cg > (uint64_t)(L.cg < 16 ? MAX_GROUPS / 2 : MAX_GROUPS) && L.cg < 64) L.cg <<= 1;
    const uint64_t wgs = (L.nb + RB / 64 - 1) / (RB / 64);
    L.blocks = (int)(wgs < (uint64_t)PASS_BLOCKS ? wgs : (uint64_t)PASS_BLOCKS);
    size_t need = 0;
    auto take = [&](size_t bytes) { size_t o = need; need += (bytes + 255) & ~(size_t)255; return o; };
    L.o_res = take(sizeof(PassResult));
    L.o_csum = take(L.nb * 8);
    L.o_off = take((L.nb / (uint64_t)L.cg + 1) * 8);
    L.o_sub = take((L.nb << (L.bs - L.sb)) * 8);
    L.o_part = take((size_t)L.blocks * 16 * 8);
    L.need = need;
    return L;
}

// The sampler; with stats16 non-null (states only) the weights come from the
// fused statistics pass, whose 14 combined sums are copied to stats16 (and k
// may be 0).
// src holds N = 2^n entries, or (explicit distributions, which are checked)
// any N in (2^{n-1}, 2^n], the entries beyond N counting as weight 0.
// host_out, when not null, receives a copy of the samples.  Synchronises.
template <typename S>
static sv_status sample_impl(const ScratchSource &scr, hipStream_t s, const S *src, int n, const uint64_t *words,
                             uint64_t seed, int64_t k, uint64_t *dev_out, uint64_t *host_out,
                             double *stats16 = nullptr, uint64_t N = 0) {
    constexpr bool CHECK = std::is_same<S, double>::value;
    if (N == 0) N = 1ull << n;
    if (k <= 0 && !stats16 && !CHECK) return SV_OK;
    if (k < 0) k = 0;
    const SampleLayout L = sample_layout(n);
    uint8_t *w = nullptr;
    SV_TRY(take_scratch(scr, L.need, &w));
    auto *csum = (unsigned long long *)(w + L.o_csum);
    auto *off = (unsigned long long *)(w + L.o_off);
    auto *sub = (unsigned long long *)(w + L.o_sub);
    double *part = (double *)(w + L.o_part);
    auto *res = (PassResult *)(w + L.o_res);
    ResultSlot slot(scr.fixed ? SIZE_MAX : sizeof(PassResult), s);   // the no-allocation call copies
    const double Nd = std::ldexp(1.0, n);
    if constexpr (!CHECK) {
        if (stats16)
            hipLaunchKernelGGL((k_pass<S, true, false>), dim3(L.blocks), dim3(RB), 0, s, src, N, L.bs, L.sb, L.nb, Nd,
                               part, csum, sub);
        else
            hipLaunchKernelGGL((k_pass<S, false, false>), dim3(L.blocks), dim3(RB), 0, s, src, N, L.bs, L.sb, L.nb,
                               Nd, part, csum, sub);
    } else {
        hipLaunchKernelGGL((k_pass<S, false, true>), dim3(L.blocks), dim3(RB), 0, s, src, N, L.bs, L.sb, L.nb, Nd,
                           part, csum, sub);
    }
    hipLaunchKernelGGL(k_finish_pass, dim3(stats16 ? 2 : 1), dim3(CMB_THREADS), 0, s, csum, L.nb, L.cg, part,
                       stats16 ? L.blocks : 0, CHECK ? L.blocks : 0, off, res, slot.ptr ? (PassResult *)slot.ptr : res);
    SV_HIP(hipGetLastError());
    // a launch holds fewer than 2^32 threads: 2^25 samples take 2^31 of them
    for (int64_t first = 0; first < k; first += RESOLVE_SLICE) {
        const int64_t m = std::min(k - first, RESOLVE_SLICE);
        const unsigned rg = (unsigned)((m + RB / 64 - 1) / (RB / 64));
#define RESOLVE(G)                                                                                                 \
    hipLaunchKernelGGL((k_resolve<S, G>), dim3(rg), dim3(RB), 0, s, src, N, L.bs, L.nb, L.cg, off, csum, sub, res, \
                       words, seed, first, first + m, dev_out)
        if (L.sb == 8) RESOLVE(1);
        else if (L.sb == 9) RESOLVE(2);
        else RESOLVE(4);
#undef RESOLVE
        SV_HIP(hipGetLastError());
    }
    PassResult host;
    SV_TRY(fetch_result(slot, &host, res, sizeof host, s));
    if (stats16)
        for (int i = 0; i < 16; i++) stats16[i] = i <= NSTAT ? host.stats[i] : 0.0;
    if (host.status == PASS_BAD)
        return fail(SV_EINVAL, "sv_sample_from: a probability is negative, NaN, infinite or >= 4");
    if (host.status == PASS_OVERFLOW)
        return fail(SV_ERANGE, "sv_sample_from: the weights floor(p 2^62) sum to 2^64 or more (sum p >= 4)");
    if (k > 0 && host.status == PASS_ZERO) return fail(SV_ESTATE, "sampler: every probability rounds to weight 0");
    // only now: a call that fails leaves the caller's array as it was
    if (k > 0 && host_out) {
        SV_HIP(hipMemcpyAsync(host_out, dev_out, (size_t)k * 8, hipMemcpyDeviceToHost, s));
        SV_HIP(hipStreamSynchronize(s));
    }
    return SV_OK;
}

sv_status run_sample(sv_state *st, const void *psi, int64_t k, uint64_t seed, uint64_t *dev_out, uint64_t *host_out) {
    ScratchSource scr;
    scr.ws = &st->ws;
    if (st->dt == SV_C64)
        return sample_impl<cpx<float>>(scr, st->stream, (const cpx<float> *)psi, st->n, nullptr,
                                       seed, k, dev_out, host_out);
    return sample_impl<cpx<double>>(scr, st->stream, (const cpx<double> *)psi, st->n, nullptr,
                                    seed, k, dev_out, host_out);
}

static sv_status stats_sample_from(const ScratchSource &scr, sv_state *st, const void *psi, sv_stats *stats,
                                   int64_t k, uint64_t seed, uint64_t *dev_out, uint64_t *host_out) {
    double r[16] = {0};
    if (st->dt == SV_C64)
        SV_TRY(sample_impl<cpx<float>>(scr, st->stream, (const cpx<float> *)psi, st->n, nullptr, seed, k,
                                       dev_out, host_out, r));
    else
        SV_TRY(sample_impl<cpx<double>>(scr, st->stream, (const cpx<double> *)psi, st->n, nullptr, seed, k,
                                        dev_out, host_out, r));
    finish_stats(st->n, r, stats);
    return SV_OK;
}

sv_status run_stats_sample(sv_state *st, const void *psi, sv_stats *stats, int64_t k, uint64_t seed,
                           uint64_t *dev_out, uint64_t *host_out) {
    ScratchSource scr;
    scr.ws = &st->ws;
    return stats_sample_from(scr, st, psi, stats, k, seed, dev_out, host_out);
}

// ---------------------------------------------------------------------------
// allocation-free statistics and samples
// ---------------------------------------------------------------------------
// The scratch of sv_moments_sample_noalloc: device memory that comes with
// the code object on every GPU the library runs on (held until the process
// ends), so the call needs no allocation.  Host code never uses this name
// as an address: its device address on each GPU is looked up once, with
// that GPU current, and kept per device.
__device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_ptr[MAX_DEVICES] = {};

static sv_status noalloc_scratch(int device, void **out) {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (device < 0 || device >= MAX_DEVICES) return fail(SV_EDEVICE, "device index out of range");
    if (!g_scratch_ptr[device]) {
        int cur = 0;
        SV_HIP(hipGetDevice(&cur));
        if (cur != device) SV_HIP(hipSetDevice(device));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != device) (void)hipSetDevice(cur);
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_ptr[device] = p;
    }
    *out = g_scratch_ptr[device];
    return SV_OK;
}

// The documented limit of the call: 8 2^(n-10) + 16 2^(n-16) + 12 k bytes and
// the statistic rows.  The pass itself needs no room per sample.
size_t noalloc_scratch_need(int n, int64_t k) {
    const int bs = n < 16 ? n : 16, sb = bs < 10 ? bs : 10;
    const uint64_t nb = 1ull << (n - bs), rows = nb < 2048 ? nb : 2048;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t per_k = al((size_t)k * 4) + al((size_t)k * 8);
    const size_t limit = al(nb * 8) + al((nb + 1) * 8) + al((1ull << (n - sb)) * 8) + per_k + al(rows * 128) + 256;
    return std::max(limit, sample_layout(n).need);
}

sv_status run_stats_sample_noalloc(sv_state *st, sv_stats *stats, int64_t k, uint64_t seed, uint64_t *dev_out) {
    const size_t need = noalloc_scratch_need(st->n, k);
    if (need > NOALLOC_SCRATCH_BYTES) {
        char b[200];
        snprintf(b, sizeof b, "sv_moments_sample_noalloc: n = %d and k = %lld need %zu bytes of scratch, "
                 "the fixed scratch holds %zu", st->n, (long long)k, need, (size_t)NOALLOC_SCRATCH_BYTES);
        return fail(SV_ERANGE, b);
    }
    ScratchSource scr;
    SV_TRY(noalloc_scratch(st->device, &scr.fixed));
    scr.cap = NOALLOC_SCRATCH_BYTES;
    return stats_sample_from(scr, st, st->data, stats, k, seed, dev_out, nullptr);
}

// An explicit distribution: every p must be finite, >= 0 and < 4 (its weight
// floor(p 2^62) fits 64 bits), and the weights must sum below 2^64; the pass
// that sums the weights checks both (a separate validation read 46 workgroups
// of a 3-million-entry distribution in 103 us).
sv_status run_sample_from(const double *probs, uint64_t N, const uint64_t *r64, int64_t k,
                          uint64_t *out, hipStream_t s) {
    int n = 0;
    while ((1ull << n) < N) n++;
    // library-owned scratch for this standalone call; kept until the process
    // ends (never freed from a static destructor, after the runtime is gone),
    // one call at a time
    static Workspace *ws = new Workspace();
    static std::mutex *mu = new std::mutex();
    std::lock_guard<std::mutex> lock(*mu);
    ScratchSource scr;
    scr.ws = ws;
    return sample_impl<double>(scr, s, probs, n, r64, 0, k, out, nullptr, nullptr, N);
}

// ---------------------------------------------------------------------------
// sample cross entropy: sum_i ln p(x_i) and the number of p(x_i) = 0
// ---------------------------------------------------------------------------
// Samples are n-bit strings (checked on the host before the copy).
template <typename T>
__global__ __launch_bounds__(RB) void k_ce(const cpx<T> *__restrict__ psi,
                                           const uint64_t *__restrict__ x, int64_t k, int64_t per,
                                           double *__restrict__ part) {
    __shared__ double red[4 * 2];
    double v[2] = {0.0, 0.0};
    const int64_t b = (int64_t)blockIdx.x * per;
    const int64_t e = b + per < k ? b + per : k;
    for (int64_t i = b + threadIdx.x; i < e; i += RB) {
        const double p = prob_of(psi[x[i]]);
        if (p > 0.0) v[0] += log(p);
        else v[1] += 1.0;
    }
    block_sum<double, 2>(v, red);
    if (threadIdx.x < 2) part[(uint64_t)blockIdx.x * 16 + threadIdx.x] = red[threadIdx.x];
}

sv_status run_cross_entropy(sv_state *st, const void *psi, const uint64_t *dev_samples, int64_t k,
                            double S, double *sum_log, int64_t *zeros) {
    (void)S;
    if (k <= 0) { *sum_log = 0; *zeros = 0; return SV_OK; }
    // one sample per thread (latency-bound gathers) up to 2048 rows; with 4096
    // samples per workgroup 10^5 samples ran on 25 workgroups
    const int64_t per = std::max<int64_t>(RB, (k + 2047) / 2048);
    const int64_t nb = (k + per - 1) / per;
    SV_TRY(st->ws.reserve((size_t)(nb + 1) * 16 * sizeof(double)));
    double *part = (double *)st->ws.ptr;
    ResultSlot slot(2 * sizeof(double), st->stream);
    double *res = slot.ptr ? (double *)slot.ptr : part + (size_t)nb * 16;
    if (st->dt == SV_C64)
        hipLaunchKernelGGL(k_ce<float>, dim3((unsigned)nb), dim3(RB), 0, st->stream,
                           (const cpx<float> *)psi, dev_samples, k, per, part);
    else
        hipLaunchKernelGGL(k_ce<double>, dim3((unsigned)nb), dim3(RB), 0, st->stream,
                           (const cpx<double> *)psi, dev_samples, k, per, part);
    SV_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_combine, dim3(1), dim3(CMB_THREADS), 0, st->stream, part, (int)nb, 2, res);
    SV_HIP(hipGetLastError());
    double r[2];
    SV_TRY(fetch_result(slot, r, res, sizeof r, st->stream));
    *sum_log = r[0];
    *zeros = (int64_t)r[1];
    return SV_OK;
}

}  // namespace svi
