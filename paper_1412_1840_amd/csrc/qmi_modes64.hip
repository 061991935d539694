// HIP kernel for gfx950 (MI355X): the mode sums (qmi_modes.hip) of Protopapas et al.,
// arXiv:1412.1840, with every step in FP64 (QMI_PREC_FP64).
#include <math.h>

#include "qmi_modes.h"

namespace qmi {

namespace {

typedef double double4v __attribute__((ext_vector_type(4)));

// One wave = (curve, 16 frequency slots): lane l works for slot l mod 16 and, in every block of 4
// samples, for sample l / 16, whose harmonics it feeds as the B operand of the 16 x 16 x 4 matrix
// instruction; the block's values of U in three blocks of 16 nodes are the A operands.  Node block k
// of a curve keeps its sums in accumulator k mod 3 (register i of lane group g: node 4 i + g); when
// the samples, in magnitude order, move on past it, they are folded into the lane's sums and the
// accumulator is taken over by node block k + 3.
//
// Three node blocks, so that a sample has the 33 nodes at least that nodes 0.36 sigma_y apart need to
// the rounding of a double: with two and 0.4 (29 nodes) a kernel value was off by up to 8e-14 where
// magnitudes all lie at the same place between two nodes (a wide sigma_y, few values), although not
// where they spread.
//
// Bound: FP64 arithmetic.  The matrix instruction takes 64 cycles of a SIMD and shares the FP64
// units with the vector instructions (measured: 71 cycles of 2.4 GHz, 4.3 more for every fma beside
// it), 18 of them and about 70 others per block and group of harmonics, 1600 cycles.
// The pairs take 26 instructions each: N^2 / 2 of them against N times 48 nodes, 2 x 33 harmonics
// (sigma_t 0.3) and the sines.  Measured, 16 survey curves, 1024 frequencies: 1.5 ms for the call
// against 4.3 (1.15 with two node blocks, four harmonics per pass).  Errors against extended precision
// are a rounding or two: V_J 3e-16 to 9e-16 rms against the pair sums' 4e-16 to 8e-15, IP_t and V_C
// 2e-16 to 8e-16 against 2e-16 to 7e-16 (N = 121 to 2500, sigma_t 0.05 to 2).
constexpr int kWaves64 = 4;
constexpr int kThreads64 = 64 * kWaves64;
constexpr int kS64 = 5;  // sums per harmonic and lane

template <bool SPLIT>
__global__ void __launch_bounds__(kThreads64, 2)
modes64_kernel(const CurveParams* __restrict__ cp, const int32_t* __restrict__ order, FreqPlan fp,
               ModeDev md, int n_work, int xcd_grouped, int gmax, PairOut out) {
    __shared__ double S_all[kWaves64][kModeGroup64 * kS64][64];
    const int lane = threadIdx.x & 63;
    const int wave = uni((int)(threadIdx.x >> 6));
    const int tiles = (fp.count + kLanes - 1) / kLanes;
    int rank, tile, g0 = 0;
    const unsigned blk = blockIdx.x;
    if (SPLIT) {
        rank = (int)(blk / (unsigned)(gmax * tiles));
        const int rem = (int)(blk - (unsigned)rank * (gmax * tiles));
        g0 = rem / tiles;
        tile = rem - g0 * tiles;
    } else if (xcd_grouped) {
        const int xcd = (int)(blk % kXcds);
        const int seq = (int)(blk / kXcds);
        // (turned by one die per round of curves: what is skipped in a pattern spreads over the dies)
        const int round = seq / tiles;
        rank = round * kXcds + (xcd + round) % kXcds;
        tile = seq - round * tiles;
    } else {
        rank = (int)(blk / tiles);
        tile = (int)(blk - (unsigned)rank * tiles);
    }
    if (rank >= n_work) return;
    const int c = order[rank];
    const CurveParams P = cp[c];
    const int n16 = lane & 15, kg = lane >> 4;
    const int slot = tile * kLanes + wave * 16 + n16;
    if (tile * kLanes + wave * 16 >= fp.count) return;
    bool active;
    const double f = mode_slot_freq(fp, c, slot, 0, active);
    const int64_t obase = (int64_t)c * fp.count + slot;
    if (P.status != 0) {
        if (active && kg == 0 && g0 == 0 && !SPLIT) mode_nan(obase, out);
        return;
    }
    const ModeCurve M = md.curves[c];
    const int g_end = SPLIT ? min(g0 + 1, M.groups) : M.groups;
    if (g0 >= g_end) return;  // no such group, or a curve left to the pair sums
    const double* ts = md.ts + 4 * M.boff + kg;
    const double* frag = reinterpret_cast<const double*>(md.frag) + 64 * kTiles64 * M.boff + lane;
    const double* bq = md.b + 16 * kTiles64 * M.boff + kg;
    const int32_t* rows = md.rows + M.boff;
    const double* coef = md.coef + (int64_t)c * mode_stride(md.mode_cap);
    double (*S)[64] = S_all[wave];

    const double n0 = (double)P.n;  // p sum_q b_q
    double SJ = M.c0 * M.sj0, ST = M.c0 * n0 * n0, SC = M.c0 * n0 * M.sj0;
    if (SPLIT) SJ = ST = SC = 0.0;
    for (int g = g0; g < g_end; ++g) {
        const int m0 = g * kModeGroup64 + 1;
        double4v acc[kTiles64][kModeGroup64][2];
#pragma unroll
        for (int m = 0; m < kModeGroup64; ++m) {
#pragma unroll
            for (int k = 0; k < kTiles64; ++k) acc[k][m][0] = acc[k][m][1] = double4v{0, 0, 0, 0};
#pragma unroll
            for (int q = 0; q < kS64; ++q) S[m * kS64 + q][lane] = 0.0;
        }
        int wb = 0, at = 0;  // first node block in the accumulators, and its accumulator
        // Folds the node blocks before `row`.  One uniform branch per accumulator, each block's own: a
        // loop over the blocks would have the accumulators merged, and moved, at every turn.
        auto retire_to = [&](int row) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < kTiles64; ++k) {
                const int blk = wb + (k < at ? k - at + kTiles64 : k - at);
                if (blk >= row) continue;
                double b[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) b[r] = bq[16 * (int64_t)blk + 4 * r];
#pragma unroll
                for (int m = 0; m < kModeGroup64; ++m) {
                    double v[kS64] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double x = acc[k][m][0][r], z = acc[k][m][1][r];
                        v[0] += fma(x, x, z * z);
                        v[1] += x;
                        v[2] += z;
                        v[3] = fma(b[r], x, v[3]);
                        v[4] = fma(b[r], z, v[4]);
                    }
                    acc[k][m][0] = acc[k][m][1] = double4v{0, 0, 0, 0};
#pragma unroll
                    for (int q = 0; q < kS64; ++q) lds_add(&S[m * kS64 + q][lane], v[q]);
                }
            }
            at = (at + row - wb) % kTiles64;
            wb = row;
        };
        double a[kTiles64], t = ts[0];
#pragma unroll
        for (int k = 0; k < kTiles64; ++k) a[k] = frag[64 * k];
        for (int kb = 0; kb < M.blocks; ++kb) {
            const int row = uni(rows[kb]);
            if (wb < row) retire_to(row);
            double u[kTiles64];
#pragma unroll
            for (int k = 0; k < kTiles64; ++k) u[k] = a[k];
            const double p = fma(f, t, -rint(f * t));  // the phase, in turns
            if (kb + 1 < M.blocks) {
#pragma unroll
                for (int k = 0; k < kTiles64; ++k) a[k] = frag[((int64_t)(kb + 1) * kTiles64 + k) * 64];
                t = ts[4 * (kb + 1)];
            }
            // z_m = exp(2 pi i m f t): z_m0 from its own phase, z_m0+1 = z_m0 z_1, and on from there
            // by z_m+1 = 2 cos(2 pi f t) z_m - z_m-1.
            double s1, c1, C, Sn;
            sincos_turns(p, &s1, &c1);
            C = c1;
            Sn = s1;
            if (g > 0) {
                const double md0 = (double)m0;
                sincos_turns(fma(md0, p, -rint(md0 * p)), &Sn, &C);
            }
            double Cp = 0.0, Sp = 0.0;
#pragma unroll
            for (int m = 0; m < kModeGroup64; ++m) {
#pragma unroll
                for (int k = 0; k < kTiles64; ++k) {
                    acc[k][m][0] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(u[k], C, acc[k][m][0], 0, 0, 0);
                    acc[k][m][1] =
                        __builtin_amdgcn_mfma_f64_16x16x4f64(u[k], Sn, acc[k][m][1], 0, 0, 0);
                }
                double x, y;
                if (m == 0) {
                    x = fma(C, c1, -(Sn * s1));
                    y = fma(C, s1, Sn * c1);
                    c1 += c1;
                } else {
                    x = fma(c1, C, -Cp);
                    y = fma(c1, Sn, -Sp);
                }
                Cp = C;
                Sp = Sn;
                C = x;
                Sn = y;
            }
        }
        retire_to(wb + kTiles64);
        // The four lanes of a slot hold a quarter of its nodes each: lane group kg adds them for
        // the harmonics kg, kg + 4, ... and forms their terms.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double gj = 0.0, gt = 0.0, gc = 0.0;
        for (int m = kg; m < kModeGroup64; m += 4) {
            double v[kS64];
#pragma unroll
            for (int q = 0; q < kS64; ++q) {
                v[q] = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) v[q] += S[m * kS64 + q][n16 + 16 * k];
            }
            const double cm = coef[m0 - 1 + m];
            const double ca = kNodeP64 * v[1], sa = kNodeP64 * v[2];
            // (every a_qm is b_q, as in the mixed mode)
            const bool together = v[2] == 0.0 && v[4] == 0.0 && fabs(ca - n0) <= 1e-5 * n0;
            gj = fma(cm, together ? M.sj0 : kNodeW64 * v[0], gj);
            gt = fma(cm, together ? n0 * n0 : ca * ca + sa * sa, gt);
            gc = fma(cm, together ? n0 * M.sj0 : kNodeW64 * (ca * v[3] + sa * v[4]), gc);
        }
        for (int o = 16; o < 64; o <<= 1) {
            gj += __shfl_xor(gj, o, 64);
            gt += __shfl_xor(gt, o, 64);
            gc += __shfl_xor(gc, o, 64);
        }
        SJ += gj;
        ST += gt;
        SC += gc;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (kg != 0 || !active) return;
    if (SPLIT) {
        double* pp = out.part + (((int64_t)rank * gmax + g0) * fp.count + slot) * 3;
        pp[0] = SJ;
        pp[1] = ST;
        pp[2] = SC;
        return;
    }
    mode_scores(P, SJ, ST, SC, obase, out);
}

}  // namespace

hipError_t launch_modes64(hipStream_t st, const CurveParams* cp, const int32_t* order,
                          int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                          const PairOut& out, int split_groups) {
    if (n_work_curves <= 0 || fp.count <= 0) return hipSuccess;
    const int64_t tiles = (fp.count + kLanes - 1) / kLanes;
    if (split_groups > 0 && out.part) {
        const int64_t blocks = (int64_t)n_work_curves * split_groups * tiles;
        modes64_kernel<true><<<(unsigned)blocks, kThreads64, 0, st>>>(
            cp, order, fp, md, n_work_curves, 0, split_groups, out);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_mode_epilogue(st, cp, order, n_work_curves, fp, md, out, split_groups);
    }
    const int xcd = n_work_curves >= 8 * kXcds;
    const int64_t rows = xcd ? (int64_t)(n_work_curves + kXcds - 1) / kXcds * kXcds
                             : (int64_t)n_work_curves;
    modes64_kernel<false><<<(unsigned)(rows * tiles), kThreads64, 0, st>>>(
        cp, order, fp, md, n_work_curves, xcd, 0, out);
    return hipGetLastError();
}

}  // namespace qmi
