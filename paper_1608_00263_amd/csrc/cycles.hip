// Register-tile sweeps that also form the statistics of the state they store:
// the points of a per-cycle series (sv_cycle_moments).
#include <hip/hip_runtime.h>

#include <cmath>

#include "device_common.h"
#include "internal.h"
#include "reduce_common.h"

namespace svi {

// Adds the statistic sums of one stored tile to this wavefront's row in LDS.
// The probabilities replace the amplitudes before the sums start, so that the
// tile and the sums are not in registers together.
template <typename T>
struct TileStats {
    double *row;              // this wavefront's NSTAT sums
    unsigned *zrow;           // and its count of zeros
    const LnEntry *tab;
    double Nd;
    int lane;
    template <int NR>
    __device__ __forceinline__ void operator()(const cplx<T> (&a)[NR]) const {
        constexpr int K = NR < 2 ? NR : 2;
        double p[NR];
#pragma unroll
        for (int r = 0; r < NR; r++) {
            cpx<T> v;
            v.re = a[r].re;
            v.im = a[r].im;
            p[r] = prob_of(v);
        }
        __builtin_amdgcn_sched_barrier(0);
        double acc[NSTAT];
#pragma unroll
        for (int i = 0; i < NSTAT; i++) acc[i] = 0.0;
        unsigned zeros = 0;
#pragma unroll
        for (int r = 0; r < NR; r += K) {
            double q[K];
#pragma unroll
            for (int k = 0; k < K; k++) q[k] = p[r + k];
            stat_add_n<K>(acc, zeros, q, Nd, tab);
            __builtin_amdgcn_sched_barrier(0);
        }
        stat_finish(acc, Nd);
        zeros = wave_sum(zeros);
#pragma unroll
        for (int i = 0; i < NSTAT; i++) {
            const double s = wave_sum(acc[i]);
            if (lane == 0) row[i] += s;
        }
        if (lane == 0) *zrow += zeros;
    }
};

// The sweep of k_regtile over tiles blockIdx.x * 4 + wave, + 4 gridDim.x, ...
// and one row of partial sums per workgroup.  The statistics take about 45
// VALU issues per amplitude, which the sweep's memory time covers (a per-cycle
// sweep has few gates): 24 qubits complex128 one point took 87 us for the
// sweep and 47 us for a pass of its own over the state; the series of 39 points
// went from 5.73 to 4.5-4.7 ms, that of 28 qubits from 89.8 to 69.9.  (With four
// probabilities at a time and the lane's constants held across the tiles, 62
// registers spilled at 5 register qubits: 5.11 and 74.1 ms.)
template <typename T, int VB>
__global__ __launch_bounds__(BLOCK, VB == 4 ? 4 : 3) void k_regtile_stats(
    cplx<T> *__restrict__ psi, const uint8_t *__restrict__ prog, uint64_t ntiles, double Nd,
    double *__restrict__ part) {
    __shared__ LnEntry tab[LN_BINS];
    __shared__ double sums[4][NSTAT];
    __shared__ unsigned zsum[4];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    load_ln_table(tab);
    if (threadIdx.x < 4 * NSTAT) sums[threadIdx.x / NSTAT][threadIdx.x % NSTAT] = 0.0;
    if (threadIdx.x < 4) zsum[threadIdx.x] = 0u;
    __syncthreads();
    TileStats<T> after;
    after.row = sums[wave];
    after.zrow = &zsum[wave];
    after.tab = tab;
    after.Nd = Nd;
    after.lane = lane;
    const uint64_t stride = (uint64_t)gridDim.x * (BLOCK / 64);
#pragma unroll 1
    for (uint64_t tile = (uint64_t)blockIdx.x * (BLOCK / 64) + wave; tile < ntiles; tile += stride) {
        // opaque copies: what a tile derives from its lane and program is formed
        // anew (a few instructions) instead of being held across the loop
        // beside the tile and the sums
        const uint8_t *pr = prog;
        int ln = lane;
        asm volatile("" : "+s"(pr), "+v"(ln));
        regtile_apply<T, VB>(psi, pr, tile, ln, nullptr, 0, (T *)nullptr, after);
    }
    __syncthreads();
    double *row = part + (uint64_t)blockIdx.x * 16;
    if (threadIdx.x < NSTAT) row[threadIdx.x] = (sums[0][threadIdx.x] + sums[1][threadIdx.x]) + (sums[2][threadIdx.x] + sums[3][threadIdx.x]);
    if (threadIdx.x == NSTAT) row[NSTAT] = (double)((unsigned long long)zsum[0] + zsum[1] + zsum[2] + zsum[3]);
}

sv_status launch_stat_sweep(sv_state *st, const Plan &plan, const Op &op, double *part, int *nrows) {
    if (op.type != OP_REGTILE || op.wide || st->dt != SV_C128)
        return fail(SV_EINVAL, "a statistics sweep needs complex128 tiles of one wavefront");
    const uint8_t *prog = (const uint8_t *)plan.dprog + op.prog_off;
    const uint64_t ntiles = (1ull << st->n) >> (LANE_BITS + op.vbits);
    const uint64_t groups = (ntiles + BLOCK / 64 - 1) / (BLOCK / 64);
    // no more workgroups than are resident at the widths that matter (3 per CU
    // for 5 register qubits, 4 for 4): with more, the last round of a 28-qubit
    // sweep ran on a fraction of the chip.  Narrower tiles could hold 6 to 8 per
    // CU and run on 3 (24 qubits, 25 points: 5.16, 3.44 and 2.74 ms at 1, 2 and 3
    // register qubits, 2.60 at 4 and 2.73 at 5).
    const uint64_t resident = op.vbits == 4 ? 1024 : 768;
    static_assert(STATS_BLOCKS >= 1024, "a list of partial rows holds STATS_BLOCKS");
    *nrows = (int)(groups < resident ? groups : resident);
    const double Nd = std::ldexp(1.0, st->n);
#define STAT_CASE(VB)                                                                                         \
    case VB:                                                                                                  \
        hipLaunchKernelGGL((k_regtile_stats<double, VB>), dim3(*nrows), dim3(BLOCK), 0, st->stream,           \
                           (cplx<double> *)st->data, prog, ntiles, Nd, part);                                 \
        break;
    switch (op.vbits) {
        STAT_CASE(1) STAT_CASE(2) STAT_CASE(3) STAT_CASE(4) STAT_CASE(5)
    default: return fail(SV_EINVAL, "register tile width out of range");
    }
#undef STAT_CASE
    SV_HIP(hipGetLastError());
    return SV_OK;
}

}  // namespace svi
