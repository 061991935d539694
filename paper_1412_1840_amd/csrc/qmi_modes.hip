// HIP kernels for gfx950 (MI355X): the pair x frequency sums of Protopapas et al.,
// arXiv:1412.1840, as sums over harmonics and magnitude nodes (the mixed-precision path).
//
// Both kernels of the method (Sec. 2, Sec. 2.1) are sums of products of one-sample factors:
//   periodic:  exp(-2 sin^2(x/2) / st^2) = sum_m c_m cos(m x),  c_0 = e^-k I_0(k),
//              c_m = 2 e^-k I_m(k), k = 1 / st^2 (the Jacobi-Anger series; I_m decays faster than
//              exponentially past m ~ k^(1/2)),
//   Gaussian:  exp(-(y - y')^2 / (2 sy^2)) = w sum_q U_q(y) U_q(y'),  U_q(y) = exp(-((y - x_q)/sy)^2),
//              the trapezoid rule of the Gaussian product integral on nodes x_q of spacing h sy,
//              w = h sqrt(2/pi); its error is 2 exp(-pi^2 / (2 h^2)), and U_q is negligible a few
//              sy away from its node.  Also p sum_q U_q(y) = 1, p = h / sqrt(pi).
// With a_qm(f) = sum_i U_q(y_i) exp(2 pi i m f t_i) and b_q = a_q0 the sums over all ordered pairs
// are
//   sum K_y K_t / (A B) = w sum_m c_m sum_q |a_qm|^2
//   sum K_t / A         =   sum_m c_m |p sum_q a_qm|^2
//   sum_i r_i sum_j K_t / (A B) = sum_m c_m Re( conj(p sum_q a_qm) w sum_q b_q a_qm )
// so that a frequency costs N x (harmonics) x (nodes near a sample) instead of N^2 / 2 pairs, and
// the a_qm are a matrix product (nodes x samples) by (samples x frequencies and harmonics).  All
// three sums come from the same a_qm, so that their rounding errors cancel to first order in the
// QMI wherever time and magnitude are independent, and exactly where all phases coincide.
#include <math.h>

#include <algorithm>

#include "qmi_modes.h"

namespace qmi {

namespace {

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef double double2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef short short2v __attribute__((ext_vector_type(2)));

// exp(2 pi i p), exactly 1 at p = 0.  v_sin_f32 and v_cos_f32 round towards zero (sin^2 + cos^2 is
// 6.5e-8 below 1 on average): the factor 1 + (1 - sin^2 - cos^2) / 2 puts the value back on the
// circle, to rounding.
__device__ __forceinline__ void cis(float p, float& c, float& s) {
    c = __builtin_amdgcn_cosf(p);
    s = __builtin_amdgcn_sinf(p);
    const float e = 0.5f * fmaf(-s, s, fmaf(-c, c, 1.0f));
    c = fmaf(c, e, c);
    s = fmaf(s, e, s);
}

// --------------------------------------------------------------------------------------------
// Mode sums
// --------------------------------------------------------------------------------------------

// The sums of a window's nodes, kept where its points' scores will be: S_J and S_C in the first and
// second half of the window's score entries, S_T among its entries of the other score.
__device__ __forceinline__ void store_node_sums(const FreqPlan& fp, int c, int slot, int nodes,
                                                double SJ, double ST, double SC,
                                                const PairOut& out) {
    const int p = slot / nodes, j = slot - p * nodes;
    const int64_t o = (int64_t)c * fp.count + (int64_t)p * fp.n_fine + j;
    out.score[o] = SJ;
    out.score[o + nodes] = SC;
    out.score2[o] = ST;
}

// Eight single-precision values as a high and a low half-precision part (each rounded to nearest:
// together at least 22 bits).  minus_one is -1 in a scalar register whose value the compiler does
// not know, so that value minus high part is one v_fma_mix_f32 (v_fma_mixlo/hi_f16, which would
// also convert it, issue at half rate).
__device__ __forceinline__ void split8(const float (&v)[8], float minus_one, half8v& h,
                                       half8v& l) {
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const float2v x = {v[j], v[j + 1]};
        const half2v a = __builtin_convertvector(x, half2v);
        const float2v r = {fmaf((float)a.x, minus_one, v[j]),
                           fmaf((float)a.y, minus_one, v[j + 1])};
        const half2v b = __builtin_convertvector(r, half2v);
        h[j] = a.x;
        h[j + 1] = a.y;
        l[j] = b.x;
        l[j + 1] = b.y;
    }
}

// A copy that the compiler does not see through (an identity lane permutation), so that the
// accumulator that takes another one's sums over keeps its own registers in the loop.
__device__ __forceinline__ float4v copy4(float4v x) {
    float4v y;
#pragma unroll
    for (int r = 0; r < 4; ++r)
        y[r] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x[r]), 0xe4, 0xf, 0xf, true));
    return y;
}

__device__ __forceinline__ float4v mfma(half8v a, half8v b, float4v c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// A block's products, small parts first, summed from zero and then added: one rounding of the long
// sums per block, where products added to them one after the other would be three and more.
__device__ __forceinline__ void add_block(const float (&v)[8], float minus_one, half8v a0h, half8v a0l,
                                          half8v a1h, half8v a1l, float4v& acc0, float4v& acc1) {
    half8v h, l;
    split8(v, minus_one, h, l);
    const float4v zero = {0.f, 0.f, 0.f, 0.f};
    float4v x = mfma(a0l, h, zero), y = mfma(a1l, h, zero);
    x = mfma(a0h, l, x);
    y = mfma(a1h, l, y);
    x = mfma(a0h, h, x);
    y = mfma(a1h, h, y);
    acc0 += x;
    acc1 += y;
}

// The sums of a wave's nodes: single-precision accumulators, out of which whole units (kNodeScale,
// one sample at its node) are moved into 16-bit counts every few blocks, so that the accumulators
// stay small and a long sum is as exact as a short one.
struct Sum {
    float4v low;
    short2v high[2];
};
constexpr float kUnit = (float)kNodeScale;
static_assert(QMI_MAX_N < 32768, "counts of units");

__device__ __forceinline__ void carry(Sum& a) {
    constexpr float kC = 12582912.0f * kUnit;  // 1.5 2^23 units: rounds to whole units
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const float x = a.low[r] + kC, y = a.low[r + 1] + kC;
        a.low[r] -= x - kC;
        a.low[r + 1] -= y - kC;
        const unsigned units = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x),
                                                     0x05040100);  // the low halves of both
        short2v v;
        __builtin_memcpy(&v, &units, 4);
        a.high[r / 2] += v;
    }
}

__device__ __forceinline__ double value(const Sum& a, int r) {
    return fma((double)(int)a.high[r / 2][r & 1], (double)kUnit, (double)a.low[r]);
}

// One wave = (curve, 16 frequency slots): lane l works for slot l mod 16 and, in every block of 32
// samples (in magnitude order), for the samples 8 (l / 16) ... + 7.  Per block it forms
// exp(2 pi i m f t) of its eight samples for the kModeGroup harmonics of a group, splits them into
// two half-precision parts and feeds them as the B operand to the matrix unit: hi*hi + hi*lo +
// lo*hi with the U fragments of the block's two 16-node blocks as A.  Because samples are sorted, a
// node block that no later sample reaches is folded into the FP64 sums (sum_q a^2, sum_q a,
// sum_q b a, per lane in LDS) and its registers are taken over by the next.
// The harmonic groups of a slot are summed in order; with SPLIT a wave runs one group and stores
// its sums for mode_epilogue_kernel, which adds them in the same order.
//
// Precision.  A value of a harmonic is off by 4e-8 rms (22 bits of its two parts, and single
// precision before), each sample independently, a block's sum by two roundings of it, a node's sum
// by one rounding per block of what has come together since the last carry.  Times count from a
// sample's, so that the values are exact where phases coincide with it.  Measured against FP64 over
// 8 to 64 curves of each length (56 to 3000 samples) at 301 frequencies on [0.001, 10]: rms errors
// of V_J, IP_t and V_C 0.04 to 0.7 of the pair sums' (N = 617, sigma_t 0.3: 2.5e-9, 1.3e-9 and 1.8e-9
// against 1.2e-8, 1.1e-8 and 2.1e-8), of QMI and nCKP less (1.7e-9 against 4.2e-8; 2.1e-8 against
// 2.2e-7 of the highest nCKP).  The sums are largest at a curve's own frequency: of 16 curves of 1000
// samples V_J is off there by 9.2e-9, 9.6e-9 and 8.3e-9 at most for sigma_t 0.3, 0.1 and 0.6.
//
// Why this shape: N^2 / 2 pairs become N x 21 harmonics x 32 nodes (sigma_t 0.3) on the matrix
// unit.  Seven harmonics are what 256 registers of two waves per SIMD hold (112 accumulators and 56
// counts); the 16 x 16 x 32 instruction takes a lane's own eight samples as its B operand, so that
// the harmonics go from the recurrence to the matrix unit without LDS.  Bound: issue slots.  Per block
// and group a wave issues 84 MFMAs (17 cycles each) and, counted with carries and folds, 900 other VALU
// instructions (half of them conversions, FP64 and sines at 5 to 9 cycles), and the two overlap only
// in part (a conversion issued between MFMAs costs 2.7 of its 4.8 cycles): 4700 cycles of a SIMD in
// all, 30% of them MFMAs.  104 bytes a lane are spilled (2 GB written per 0.6 s launch of 4096
// curves, a thousandth of what HBM takes).  Measured, 768 survey curves (N 300..1000),
// 20 000 + 10 x 1000 frequencies with the windows interpolated: 134 ms of device time against 1010
// ms by the pair sums.  What the precision costs: 96 ms with products added to the long sums one by
// one, no carries and the sines as the hardware gives them, but errors of V_J up to 6e-8 at N = 617
// and 4e-7 at N = 8192; 126 ms with carries every eight blocks, but 1.7e-8 at a curve's own frequency
// with sigma_t 0.6, where the pair sums are within 1.3e-8; 131 ms every four (1.2e-8); 155 ms after
// every block.
constexpr int kModeWaves = 4;
constexpr int kModeThreads = 64 * kModeWaves;
constexpr int kCarry = 3;   // blocks between carries
constexpr int kMS = 5;  // FP64 sums per harmonic and lane

template <bool SPLIT>
__global__ void __launch_bounds__(kModeThreads, 2)
modes_kernel(const CurveParams* __restrict__ cp, const int32_t* __restrict__ order, FreqPlan fp,
             ModeDev md, int n_work, int xcd_grouped, int gmax, PairOut out) {
    __shared__ double S_all[kModeWaves][kModeGroup * kMS][64];
    const int lane = threadIdx.x & 63;
    const int wave = uni((int)(threadIdx.x >> 6));
    const int tiles = (fp.count + kLanes - 1) / kLanes;
    int rank, tile, g0 = 0;
    unsigned blk = blockIdx.x;
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
    const ModeCurve M = md.curves[c];
    const int nodes = fp.kind == 2 && P.status == 0 ? M.nodes : 0;
    if (tile * kLanes + wave * 16 >= (nodes > 0 ? fp.top_k * nodes : fp.count)) return;
    bool active;
    const double f = mode_slot_freq(fp, c, slot, nodes, active);
    const int64_t obase = (int64_t)c * fp.count + slot;
    if (P.status != 0) {
        if (active && kg == 0 && g0 == 0 && !SPLIT) mode_nan(obase, out);
        return;
    }
    const int g_end = SPLIT ? min(g0 + 1, M.groups) : M.groups;
    if (g0 >= g_end) return;  // no such group, or a curve left to the pair sums
    const double* ts = md.ts + 32 * M.boff + 8 * kg;
    const half8v* frag = reinterpret_cast<const half8v*>(md.frag) + M.boff * 256 + lane;
    const double* bq = md.b + M.boff * 32 + 4 * kg;
    const int32_t* rows = md.rows + M.boff;
    const double* coef = md.coef + (int64_t)c * mode_stride(md.mode_cap);
    double (*S)[64] = S_all[wave];
    float minus_one = -1.0f;
    asm volatile("" : "+s"(minus_one));

    const double n0 = (double)P.n;  // p sum_q b_q
    double SJ = M.c0 * M.sj0, ST = M.c0 * n0 * n0, SC = M.c0 * n0 * M.sj0;
    if (SPLIT) SJ = ST = SC = 0.0;
    for (int g = g0; g < g_end; ++g) {
        const int m0 = g * kModeGroup + 1;
        Sum acc[2][kModeGroup][2];
        const Sum zero = {{0.f, 0.f, 0.f, 0.f}, {{0, 0}, {0, 0}}};
#pragma unroll
        for (int m = 0; m < kModeGroup; ++m) {
            acc[0][m][0] = acc[0][m][1] = acc[1][m][0] = acc[1][m][1] = zero;
#pragma unroll
            for (int q = 0; q < kMS; ++q) S[m * kMS + q][lane] = 0.0;
        }
        int wb = 0;  // node block held by acc[0]
        // Folds harmonic m of the node block whose sums are (ac, as) and node sums b.
        auto fold = [&](int m, const Sum& ac, const Sum& as, const double (&b)[4]) {
            double sq = 0.0, ca = 0.0, sa = 0.0, cb = 0.0, sb = 0.0;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double x = value(ac, r), z = value(as, r);
                sq = fma(x, x, sq);
                sq = fma(z, z, sq);
                ca += x;
                sa += z;
                cb = fma(b[r], x, cb);
                sb = fma(b[r], z, sb);
            }
            lds_add(&S[m * kMS + 0][lane], sq);
            lds_add(&S[m * kMS + 1][lane], ca);
            lds_add(&S[m * kMS + 2][lane], sa);
            lds_add(&S[m * kMS + 3][lane], cb);
            lds_add(&S[m * kMS + 4][lane], sb);
        };
        auto load_b = [&](int row, double (&b)[4]) {
#pragma unroll
            for (int r = 0; r < 4; ++r) b[r] = bq[(int64_t)row * 16 + r];
        };
#pragma unroll 1
        for (int kb = 0; kb < M.blocks; ++kb) {
            const int row = uni(rows[kb]);
            while (wb < row) {  // at most two steps
                double b[4];
                load_b(wb, b);
#pragma unroll
                for (int m = 0; m < kModeGroup; ++m) {
                    fold(m, acc[0][m][0], acc[0][m][1], b);
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        acc[0][m][k].low = copy4(acc[1][m][k].low);
                        acc[0][m][k].high[0] = acc[1][m][k].high[0];
                        acc[0][m][k].high[1] = acc[1][m][k].high[1];
                        acc[1][m][k] = zero;
                    }
                }
                ++wb;
            }
            const half8v* fk = frag + (int64_t)kb * 256;
            const half8v a0h = fk[0], a0l = fk[64], a1h = fk[128], a1l = fk[192];
            const double2v* tp = reinterpret_cast<const double2v*>(ts + 32 * kb);
            double tv[8];
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const double2v v = tp[j / 2];
                tv[j] = v.x;
                tv[j + 1] = v.y;
            }
            // z_m = exp(2 pi i m f t): z_m0 from its own phase, z_m0+1 = z_m0 z_1, and on from
            // there by z_m+1 = 2 cos(2 pi f t) z_m - z_m-1, one multiply-add per value.
            float c1[8], s1[8], C[8], Sn[8], Cp[8], Sp[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                tv[j] = fma(f, tv[j], -rint(f * tv[j]));  // the phase, in turns
                cis((float)tv[j], c1[j], s1[j]);
            }
            if (g > 0) {
                const double md0 = (double)m0;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    cis((float)fma(md0, tv[j], -rint(md0 * tv[j])), C[j], Sn[j]);
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    C[j] = c1[j];
                    Sn[j] = s1[j];
                }
            }
#pragma unroll
            for (int m = 0; m < kModeGroup; ++m) {
                add_block(C, minus_one, a0h, a0l, a1h, a1l, acc[0][m][0].low, acc[1][m][0].low);
                add_block(Sn, minus_one, a0h, a0l, a1h, a1l, acc[0][m][1].low, acc[1][m][1].low);
                if (m == 0) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        Cp[j] = C[j];
                        Sp[j] = Sn[j];
                        C[j] = fmaf(Cp[j], c1[j], -(Sp[j] * s1[j]));
                        Sn[j] = fmaf(Cp[j], s1[j], Sp[j] * c1[j]);
                        c1[j] += c1[j];
                    }
                } else if (m + 1 < kModeGroup) {
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const float x = fmaf(c1[j], C[j], -Cp[j]);
                        const float y = fmaf(c1[j], Sn[j], -Sp[j]);
                        Cp[j] = C[j];
                        Sp[j] = Sn[j];
                        C[j] = x;
                        Sn[j] = y;
                    }
                }
            }
            if (kb % kCarry == kCarry - 1) {
#pragma unroll
                for (int m = 0; m < kModeGroup; ++m) {
                    carry(acc[0][m][0]);
                    carry(acc[0][m][1]);
                    carry(acc[1][m][0]);
                    carry(acc[1][m][1]);
                }
            }
        }
        {
            double b0[4], b1[4];
            load_b(wb, b0);
            load_b(wb + 1, b1);
#pragma unroll
            for (int m = 0; m < kModeGroup; ++m) {
                fold(m, acc[0][m][0], acc[0][m][1], b0);
                fold(m, acc[1][m][0], acc[1][m][1], b1);
            }
        }
        // The four lanes of a slot hold a quarter of its nodes each: lane group kg adds them for
        // the harmonics kg, kg + 4, ... and forms their terms.
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        double gj = 0.0, gt = 0.0, gc = 0.0;
        for (int m = kg; m < kModeGroup; m += 4) {
            double v[kMS];
#pragma unroll
            for (int q = 0; q < kMS; ++q) {
                v[q] = 0.0;
#pragma unroll
                for (int k = 0; k < 4; ++k) v[q] += S[m * kMS + q][n16 + 16 * k];
            }
            const double cm = coef[m0 - 1 + m];
            const double ca = kNodeP * v[1], sa = kNodeP * v[2];
            // Where all phases coincide (no sine left at all, and cosines of 1) every a_qm is b_q: the
            // sums are then exact.
            const bool together = v[2] == 0.0 && v[4] == 0.0 && fabs(ca - n0) <= 1e-5 * n0;
            gj = fma(cm, together ? M.sj0 : kNodeW * v[0], gj);
            gt = fma(cm, together ? n0 * n0 : ca * ca + sa * sa, gt);
            gc = fma(cm, together ? n0 * M.sj0 : kNodeW * (ca * v[3] + sa * v[4]), gc);
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
    if (nodes > 0) {
        store_node_sums(fp, c, slot, nodes, SJ, ST, SC, out);
        return;
    }
    mode_scores(P, SJ, ST, SC, obase, out);
}

constexpr int kModeEpiBlock = 256;

__global__ void __launch_bounds__(kModeEpiBlock)
mode_epilogue_kernel(const CurveParams* __restrict__ cp, const int32_t* __restrict__ order,
                     FreqPlan fp, ModeDev md, int n_work, int gmax, PairOut out) {
    const int64_t idx = (int64_t)blockIdx.x * kModeEpiBlock + threadIdx.x;
    const int64_t rank = idx / fp.count;
    if (rank >= n_work) return;
    const int slot = (int)(idx - rank * fp.count);
    const int c = order[rank];
    const CurveParams P = cp[c];
    const ModeCurve M = md.curves[c];
    const int nodes = fp.kind == 2 && P.status == 0 ? M.nodes : 0;
    bool active;
    (void)mode_slot_freq(fp, c, slot, nodes, active);
    if (!active) return;
    const int64_t obase = (int64_t)c * fp.count + slot;
    if (P.status != 0) {
        mode_nan(obase, out);
        return;
    }
    if (M.groups == 0) return;
    const double n0 = (double)P.n;  // p sum_q b_q
    double SJ = M.c0 * M.sj0, ST = M.c0 * n0 * n0, SC = M.c0 * n0 * M.sj0;
    for (int g = 0; g < M.groups; ++g) {
        const double* pp = out.part + ((rank * gmax + g) * fp.count + slot) * 3;
        SJ += pp[0];
        ST += pp[1];
        SC += pp[2];
    }
    if (nodes > 0) {
        store_node_sums(fp, c, slot, nodes, SJ, ST, SC, out);
        return;
    }
    mode_scores(P, SJ, ST, SC, obase, out);
}

// --------------------------------------------------------------------------------------------
// Refinement windows
// --------------------------------------------------------------------------------------------

// Within a refinement window the three sums are smooth in the frequency: harmonic m turns by at most
// m T W, and 1000 points of a window two coarse steps wide oversample them several times.  They are
// summed at the window's Chebyshev nodes only (ModeCurve::nodes, about 190 for 2500 days, a window
// of 1e-3 1/d and sigma_t 0.3) and every point's sums follow from the Chebyshev series through them
// (FP64; truncated below kWinTol), then its scores.  One workgroup per window.
// Bound: FP64 multiply-adds (two per point, coefficient and sum) in batches, latency for one curve.
// Measured, 768 survey curves, 10 windows of 1000 points: 0.41 ms, and 12 ms for the mode sums at the
// nodes, where they would take 62 at every point (half of the coarse grid's 124); one curve of 617
// samples 18 us.  (0.56 ms and 25 us without the symmetry of nodes and points.)
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK)
mode_window_kernel(const CurveParams* __restrict__ cp, FreqPlan fp, ModeDev md, PairOut out) {
    extern __shared__ double wsh[];
    const int c = blockIdx.x / fp.top_k, p = blockIdx.x - c * fp.top_k;
    const CurveParams P = cp[c];
    if (P.status != 0 || !md.curves[c].cap || !md.curves[c].groups) return;
    const int K = md.curves[c].nodes;
    if (K == 0 || p >= fp.npk[c]) return;
    const int H = (K + 1) / 2;  // node j and its mirror image K - 1 - j
    double* v = wsh;            // [H][2][3] sums and differences of the mirrored nodes' sums
    double* a = wsh + 6 * H;    // [H][2][3] coefficients 2 h and 2 h + 1
    const int64_t o = (int64_t)c * fp.count + (int64_t)p * fp.n_fine;
    for (int x = threadIdx.x; x < 3 * H; x += BLOCK) {
        const int j = x / 3, q = x - 3 * j;
        const double* from = q == 1 ? out.score2 + o : out.score + o + (q ? K : 0);
        const double v0 = from[j], v1 = from[K - 1 - j];
        const bool mid = j == K - 1 - j;
        v[6 * j + q] = mid ? v0 : v0 + v1;
        v[6 * j + 3 + q] = mid ? 0.0 : v0 - v1;
    }
    __syncthreads();
    // Coefficient k = (2 - [k = 0]) / K sum_j v_j cos(pi k (2 j + 1) / (2 K)): the cosines by their
    // recurrence over j, the mirrored node's being the same or, for odd k, its negative.
    for (int k = threadIdx.x; k < 2 * H; k += BLOCK) {
        const double th = (double)k / (double)K;
        const double tc = 2.0 * cospi(th);
        double c0 = cospi(0.5 * th), c1 = c0;  // at j = 0 and j = -1
        double s[3] = {0.0, 0.0, 0.0};
        const double* vk = v + 3 * (k & 1);
        for (int j = 0; j < H; ++j) {
#pragma unroll
            for (int q = 0; q < 3; ++q) s[q] = fma(vk[6 * j + q], c0, s[q]);
            const double c2 = fma(tc, c0, -c1);
            c1 = c0;
            c0 = c2;
        }
        const double w = k >= K ? 0.0 : (k ? 2.0 : 1.0) / (double)K;
#pragma unroll
        for (int q = 0; q < 3; ++q) a[3 * k + q] = s[q] * w;
    }
    __syncthreads();
    // Points m and n_fine - 1 - m mirror each other too: with y = T_2(x) the even terms are a
    // series in T_h(y), the odd ones x times a series with the same recurrence.
    const int half = (fp.n_fine + 1) / 2;
    for (int m = threadIdx.x; m < half; m += BLOCK) {
        const double x = 2.0 * (double)m / (double)(fp.n_fine - 1) - 1.0;
        const double y2 = 4.0 * x * x - 2.0;
        double b1[6], b2[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) b1[q] = b2[q] = 0.0;
        for (int h = H - 1; h > 0; --h) {  // Clenshaw's recurrence
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const double b = fma(y2, b1[q], a[6 * h + q] - b2[q]);
                b2[q] = b1[q];
                b1[q] = b;
            }
        }
        double sum[2][3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const double ev = fma(0.5 * y2, b1[q], a[q] - b2[q]);
            const double od = x * fma(y2 - 1.0, b1[3 + q], a[3 + q] - b2[3 + q]);
            sum[0][q] = ev + od;
            sum[1][q] = ev - od;
        }
        mode_scores(P, sum[0][0], sum[0][1], sum[0][2], o + m, out);
        if (fp.n_fine - 1 - m != m)
            mode_scores(P, sum[1][0], sum[1][1], sum[1][2], o + fp.n_fine - 1 - m, out);
    }
}

}  // namespace

hipError_t launch_mode_windows(hipStream_t st, const CurveParams* cp, int n_curves,
                               const FreqPlan& fp, const ModeDev& md, const PairOut& out) {
    const int64_t blocks = (int64_t)n_curves * fp.top_k;
    if (blocks <= 0) return hipSuccess;
    const size_t lds = (size_t)6 * 8 * (std::min(kWinNodesMax, fp.n_fine / 2) + 1);
    // A few windows: wide blocks, one point or two per thread.
    if (blocks < 512)
        mode_window_kernel<512><<<(unsigned)blocks, 512, lds, st>>>(cp, fp, md, out);
    else
        mode_window_kernel<256><<<(unsigned)blocks, 256, lds, st>>>(cp, fp, md, out);
    return hipGetLastError();
}

hipError_t launch_mode_epilogue(hipStream_t st, const CurveParams* cp, const int32_t* order,
                                int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                                const PairOut& out, int split_groups) {
    const int64_t threads = (int64_t)n_work_curves * fp.count;
    mode_epilogue_kernel<<<(unsigned)((threads + kModeEpiBlock - 1) / kModeEpiBlock), kModeEpiBlock,
                           0, st>>>(cp, order, fp, md, n_work_curves, split_groups, out);
    return hipGetLastError();
}

hipError_t launch_modes(hipStream_t st, const CurveParams* cp, const int32_t* order,
                        int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                        const PairOut& out, int split_groups) {
    if (n_work_curves <= 0 || fp.count <= 0) return hipSuccess;
    const int64_t tiles = (fp.count + kLanes - 1) / kLanes;
    if (split_groups > 0 && out.part) {
        const int64_t blocks = (int64_t)n_work_curves * split_groups * tiles;
        modes_kernel<true><<<(unsigned)blocks, kModeThreads, 0, st>>>(
            cp, order, fp, md, n_work_curves, 0, split_groups, out);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        return launch_mode_epilogue(st, cp, order, n_work_curves, fp, md, out, split_groups);
    }
    const int xcd = n_work_curves >= 8 * kXcds;
    const int64_t rows = xcd ? (int64_t)(n_work_curves + kXcds - 1) / kXcds * kXcds
                             : (int64_t)n_work_curves;
    modes_kernel<false><<<(unsigned)(rows * tiles), kModeThreads, 0, st>>>(
        cp, order, fp, md, n_work_curves, xcd, 0, out);
    return hipGetLastError();
}

}  // namespace qmi
