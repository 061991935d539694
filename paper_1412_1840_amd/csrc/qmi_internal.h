// Internal declarations shared by the device code (qmi_kernels.hip) and the host runtime
// (qmi_api.hip).  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qmi.h"

namespace qmi {

typedef _Float16 half8v __attribute__((ext_vector_type(8)));

// Pair-kernel geometry.  A work item is (curve, tile of kLanes frequency slots); one lane owns one
// frequency.  The pair triangle i < j is walked in passes of kPass rows; inside a pass wave w owns
// the interleaved rows base + w + kWaves*m (m < rows per wave), so every wave has nearly the same
// number of valid pairs in the diagonal region.  Columns j stream through LDS in chunks of kChunk.
constexpr int kLanes = 64;
constexpr int kWaves = 8;
constexpr int kThreads = kWaves * kLanes;
constexpr int kXcds = 8;    // accelerator complex dies of an MI355X, one L2 each
constexpr int kPass = 256;  // rows per pass; the K-table permutation is defined on it
constexpr int kChunk = 64;  // columns per LDS chunk

// Position of row i inside its pass in the K-table layout: rows of one wave are contiguous, so a
// wave reads its rows' kernel values for one column with scalar loads.
__host__ __device__ inline int64_t kperm(int64_t i) {
    int64_t b = i & ~int64_t(kPass - 1);
    int64_t r = i & (kPass - 1);
    return b + (r & (kWaves - 1)) * (kPass / kWaves) + (r >> 3);
}
__host__ __device__ inline int64_t kperm_inv(int64_t s) {
    int64_t b = s & ~int64_t(kPass - 1);
    int64_t r = s & (kPass - 1);
    return b + (r / (kPass / kWaves)) + kWaves * (r % (kPass / kWaves));
}

// Per-curve state, written by the host (off, koff, n, npad, status, sigma_t) and completed by the
// prologue and Gram kernels.
struct CurveParams {
    int64_t off;   // first sample in the packed t / y / e arrays
    int64_t koff;  // first element of this curve's K table
    int64_t poff;  // first element of this curve's permuted FP64 row-sum array (npad entries)
    int64_t ksoff; // first element of this curve's column K-sum table (passes * kWaves * n)
    int32_t n;     // samples
    int32_t npad;  // K-table row length (multiple of kPass)
    int32_t status;
    int32_t has_e;
    double sigma_t;       // > 0; QMI_SIGMA_T_SKEWNESS until the prologue sets it
    double sigma_y_rule;  // > 0 explicit, -1 Silverman, -2 median error bar
    double sigma_y;
    double A, B;   // 1 / (sqrt(2 pi) sigma)
    double ipy;    // IP_y
    double rsum;   // sum_i r_i
    double psnr;
    double bk;     // diagonal value of the stored K table (B rounded to the kernel type)
    double sjc;    // sum_{i<j} K(i,j)            (FP64, from the stored K table)
    int64_t pqoff; // first piece of this curve in a one-piece-per-workgroup launch's partial sums
    int32_t sparse; // set by the preparation: magnitudes too scattered for the mode sums
    int32_t pad;
};

// Mode sums (qmi_modes.hip).  Samples are taken in magnitude order in blocks of 32 that reach the
// same two blocks of 16 nodes; a block and each of its node blocks make a 16 x 32 operand of the
// matrix unit, in two half-precision parts.
// Groups of harmonics are kept until the rest of the series is below this share of the kernel's value
// where phases coincide (1); the rest goes with the last harmonic.
constexpr double kModeTail = 1e-8;
constexpr int kModeGroup = 7;      // harmonics per pass over the samples
constexpr int kModeCapMax = 256;     // most harmonics (sigma_t from 0.03)
// Which curves the mode sums take.  Measured per curve and frequency (4096 to 20 000 frequencies,
// batches): the pair sums take 9.2e-5 n^2 + 0.008 n + 0.25 ns, the mode sums 0.2 ns and, per group of
// harmonics, 0.107 ns per block and 0.06 per step to another node block (its sums are folded).  In
// units of half a block: mode_limit is what the pair sums' time buys, 2 blocks + steps what is spent.
// The host gives a curve to the mode sums when what it probably needs is a tenth less than that: its whole
// blocks, half a block lost at the end of each of the 4 runs and fewer that Silverman's width makes, and
// the steps.  It does so from n = 38, 77, 114, 225, 400 and 770 for sigma_t = 2, 0.6, 0.3, 0.2, 0.1 and
// 0.05 (1, 2, 3, 5, 9 and 17 groups); measured, the two sums take the same time at 32, 68, 118, 217, 385
// and 730.  The preparation gives a curve back to the pair sums when its samples
// are scattered over more node blocks than that and one block more (of curves with Silverman's
// width 3% and fewer where the mode sums begin, and none beyond): it then costs its part of one more
// section, 1% to 5% of the pair sums' time for searches of 64 curves.
inline double mode_even(int n, int groups) { return (8.6e-4 * n * n + 0.075 * n + 0.47) / groups; }
inline int mode_limit(int n, int groups) { return (int)(2.0 * mode_even(n, groups)) + 2; }
inline bool mode_takes(int n, int groups) {
    const int expect = (n + 31) / 32 + 2 + n / 200;
    return expect <= 0.9 * mode_even(n, groups) && expect <= n / 5;
}
// Blocks a curve has room for; n / 5 bounds the tables by the size of the pair sums' table of kernel
// values.
inline int mode_room(int n, int groups) {
    const int room = mode_limit(n, groups) / 2;
    return room < n / 5 ? room : n / 5;
}
// Coefficients stored per curve (whole groups).
__host__ __device__ constexpr int mode_stride(int cap) {
    return (cap + kModeGroup - 1) / kModeGroup * kModeGroup;
}

// Node spacing in units of sigma_y: the trapezoid error 2 exp(-pi^2 / (2 h^2)) is 1e-9 of a kernel
// value and alternates in sign along the magnitudes, so that it averages out over the pairs.  Values of
// U are held in units of 1 / kNodeScale: the low parts of values down to 1e-5 then are ordinary
// half-precision numbers (without, what is below 3e-8 is lost, and 4e-9 of sum_q U with it).
constexpr double kNodeStep = 0.48;
constexpr double kNodeScale = 16384.0;
constexpr double kNodeW =  // h sqrt(2/pi), for values of U in units of 1 / kNodeScale
    kNodeStep * 0.79788456080286535587989211986876 / (kNodeScale * kNodeScale);
constexpr double kNodeP = kNodeStep * 0.56418958354775628694807945156077 / kNodeScale;  // h / sqrt(pi)
// A sample uses the 16-node blocks rb and rb + 1, rb chosen so that they hold at least the
// 2 kReach + 1 nodes nearest to it (beyond, U < exp(-(8.5 h)^2) = 6e-8, which the last node takes over).
constexpr int kReach = 8;
// The mode sums in FP64 (qmi_modes64.hip): the same series and nodes, to the rounding of a double.
// Blocks of four samples that reach the same three blocks of 16 nodes: the 2 kReach64 + 1 nodes nearest
// to each sample at least (beyond, U < exp(-(16.5 h)^2) = 5e-16).
constexpr double kModeTail64 = 1e-16;
constexpr int kModeGroup64 = 3;  // harmonics per pass: their 144 registers of sums leave two waves a SIMD
constexpr double kNodeStep64 = 0.36;  // trapezoid error 6e-17 of a kernel value
constexpr double kNodeW64 = kNodeStep64 * 0.79788456080286535587989211986876;
constexpr double kNodeP64 = kNodeStep64 * 0.56418958354775628694807945156077;
constexpr int kReach64 = 16;
constexpr int kTiles64 = 3;
// Whether the host gives a curve to them.  Measured per curve and frequency (4096 frequencies,
// batches): the mode sums take 0.0105 n + 0.1 ns per group of harmonics, the pair sums 4.6e-4 n^2 and
// up to 1 ns; they meet at n = 138, 245, 690 and 1370 for sigma_t = 0.6, 0.3, 0.1 and 0.05 (7, 11, 29
// and 56 groups).
inline bool mode64_takes(int n, int groups) { return n >= 25 * groups - 30; }
// The same limit, in blocks of four samples: 0.042 ns each per group, a third of that per step.
inline int mode64_limit(int n, int groups) { return (int)(2.2e-2 * n * n / groups) + 16; }
// Blocks a curve has room for: its own, half as many again lost to the ends of runs (more and it
// is given back to the pair sums).
inline int mode64_room(int n) { return n / 4 + n / 8 + 8; }
struct ModeCurve {
    int64_t boff;   // first of its cap blocks
    int32_t cap;    // blocks there is room for; 0: the curve is left to the pair sums
    int32_t blocks; // blocks in use
    int32_t groups; // passes over the samples; 0: left to the pair sums
    int32_t limit;  // 2 blocks + steps from which the pair sums are faster
    int32_t pad;
    int32_t nodes;  // frequencies per refinement window whose sums the window's points are
                    // interpolated from; 0: every point is summed
    double c0;      // coefficient of the constant term
    double sj0;     // w sum_q b_q^2
};

struct ModeDev {
    ModeCurve* curves; // [curve]
    double* ts;        // [block][32] times in magnitude order
    int32_t* rows;     // [block] first node block, counted among the curve's
    void* frag;        // [block][node block][hi, lo][64 lanes] 8 half-precision values
    double* part;      // [block][node block][16] sums of U over the block's samples
    double* b;         // [node block (from 2 boff)][16] sums of U over all samples
    double* coef;      // [curve][mode_stride(mode_cap)]
    int32_t mode_cap;  // coefficients there is room for (past the harmonics kept)
    int32_t max_groups; // most groups of harmonics of any curve
    double win_width;  // width of a refinement window (0: no refinement)
    int32_t n_fine;    // its points
    int32_t pad;
};
// Interpolated refinement windows (mode_window_kernel): most frequencies per window, and the error
// allowed, as a share of the periodic kernel's value where phases coincide.
constexpr int kWinNodesMax = 512;
constexpr double kWinTol = 1e-10;


// Interleaved partial sums of a column's terms over a wave's rows (row m goes to partial
// m mod kPartials), combined at the end of the column: the pair kernel and the column-sum tables
// it subtracts use the same order.  Two partials issue 1% faster than four (two adds fewer per
// column and sum) and as fast as one.
constexpr int kPartials = 2;
static_assert(kPartials == 1 || kPartials == 2 || kPartials == 4, "1, 2 or 4 partial sums");

template <typename R>
__host__ __device__ inline R combine_partials(const R* p) {
    if constexpr (kPartials == 1) return p[0];
    else if constexpr (kPartials == 2) return p[0] + p[1];
    else return (p[0] + p[1]) + (p[2] + p[3]);
}

// Rows per wave of the pair kernel for each arithmetic type (a pass is kWaves times this).
template <typename R>
constexpr int rows_per_wave() {
    return sizeof(R) == 4 ? 32 : 16;
}

// How frequency slot s of curve c maps to a frequency.
struct FreqPlan {
    int32_t kind;   // 0 linear grid, 1 explicit list, 2 refinement windows, 3 per-curve lists
    int32_t count;  // slots per curve
    int32_t n_fine;
    int32_t top_k;
    int32_t stride;  // kind 3: row length of the per-curve lists
    int32_t tile_cap;  // > 0: the pair kernel runs only the first tile_cap tiles of kLanes slots
    double f0, df;           // kind 0: f = f0 + s * df
    const double* list;      // kind 1: [count]; kind 3: [curve][stride], NaN = no frequency
    const double* win;       // kind 2: [curve][top_k][2] = (lo, step)
    const int32_t* npk;      // kind 2: [curve] refined peaks
};

struct PairOut {
    double* score;   // [curve][count] primary score
    double* score2;  // nullable: [curve][count] the other score
    double* ips;     // nullable: [curve][count][3] V_J, IP_t, V_C
    int32_t score_kind;
    int32_t pad;
    double* part;    // one piece per workgroup: [piece (pqoff + q)][count][3] FP64 piece sums
};

struct PeakOut {
    int32_t* peak_k;   // [curve][top_k]
    int32_t* npk;      // [curve]
    double* win;       // [curve][top_k][2]
    int32_t* argmax;   // [curve]
};

// Refined points of a curve too close to the best for the mixed sums to tell them apart
// (best_kernel): they are scored again by the pair sums, which so decide near ties on every path.
constexpr int kTieMax = 32;
struct TieDev {
    int32_t* count;  // [curve] listed points, 0 where one is clearly the best; nullptr: no lists
    int32_t* slot;   // [curve][kTieMax] their slots
    const ModeCurve* curves;
};

// Spurious-period masks (Sec. 6.1), passed to the selection kernels by value.  A candidate (f, s)
// is inside mask i when s < amp[i] exp(-(1/f - period[i])^2 / (2 sigma[i]^2)).
struct MaskDev {
    int32_t n;
    int32_t pad;
    double period[QMI_MAX_MASKS];
    double sigma[QMI_MAX_MASKS];
    double amp[QMI_MAX_MASKS];
};

__device__ __forceinline__ bool in_mask(const MaskDev& md, double f, double s) {
    if (md.n == 0) return false;
    const double P = 1.0 / f;
    for (int i = 0; i < md.n; ++i) {
        const double d = P - md.period[i];
        if (s < md.amp[i] * exp(-(d * d) / (2.0 * md.sigma[i] * md.sigma[i]))) return true;
    }
    return false;
}

// Result record written by the best-of kernel (mirrors qmi_result field order).
struct DevResult {
    double f_best, period, score, score_qmi, score_nckp, sigma_y, psnr, coarse_best;
    int32_t coarse_index, peak_rank, fine_index, coarse_argmax, n_peaks, n, status, reserved;
    double sigma_t;
};

// Bands method (qmi_bands.hip): per-group device buffers and parameters.
struct BandsDev {
    double f_lo, df;      // spectral-window grid f_k = f_lo + k df
    int32_t n_grid, n_bands, n_keep, n_trials;
    int32_t stride;       // band_t row length (at least the largest band)
    int32_t pad;
    double* ts;           // [samples] times in time order (at each curve's offset)
    double* ys;           // [samples] magnitudes in the same order
    double* band_t;       // [curve][n_keep][stride] sample times of the kept bands
    int32_t* band_cnt;    // [curve][n_keep]
    int32_t* band_id;     // [curve][n_keep] band index of each kept band
    double* S;            // [curve][n_keep][n_grid] spectral windows
    double* trials;       // [curve][n_keep * n_trials] trial frequencies, NaN = none
    int32_t* trial_k;     // [curve][n_keep * n_trials] their grid indices, -1 = none
};
hipError_t launch_bands(hipStream_t st, const CurveParams* cp, int n_curves, int max_n,
                        const double* t, const double* y, const BandsDev& bd);
hipError_t launch_bands_best(hipStream_t st, const CurveParams* cp, int n_curves,
                             const double* score, const double* score2, int score_kind,
                             const BandsDev& bd, const MaskDev& md, DevResult* res);

// Preprocessing and whitening (qmi_prep.hip).
struct PrepDev {
    int32_t error_cut, detrend, min_samples, pad;
    const int32_t* status_in;  // [curve] host validation (nonzero: skip the curve)
    int32_t* counts;           // [curve] samples kept
    int32_t* status;           // [curve] QMI_OK or QMI_EINVAL (too short)
    uint8_t* detrended;        // [curve] 1 if the chi^2 line was subtracted
    double* t_out;             // kept samples, compacted inside each curve's input span
    double* y_out;
    double* e_out;
};
hipError_t launch_prep(hipStream_t st, int n_curves, const int64_t* offsets, const double* t,
                       const double* y, const double* e, const PrepDev& pd);
hipError_t launch_whiten(hipStream_t st, int n_curves, int max_n, const int64_t* offsets,
                         const double* t, const double* y, const double* periods, int window,
                         const int32_t* status, double* y_out);

// Launchers (qmi_kernels.hip).  All launch on `st` and return hipGetLastError().
// Per-curve preparation (qmi_prepare.hip): kernel widths and pSNR, and with md.curves the node
// tables of the curves summed over modes.  skew_lambda, skew_mu: constants of the sigma_t rule,
// applied to curves whose sigma_t is QMI_SIGMA_T_SKEWNESS.
hipError_t launch_prepare(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                          const double* t, const double* y, const double* e, double skew_lambda,
                          double skew_mu, const ModeDev& md);
template <typename R>
hipError_t launch_gram(hipStream_t st, CurveParams* cp, int n_curves, int64_t total_rows,
                       const int64_t* row_curve_start, const double* y, R* K, double* rp,
                       double* rd);
template <typename R>
hipError_t launch_gram_finalize(hipStream_t st, CurveParams* cp, int n_curves, const double* rd,
                                double* rp);
template <typename R>
hipError_t launch_ksum(hipStream_t st, const CurveParams* cp, int n_curves, int max_n, const R* K,
                       R* ks);
// Pair-kernel variants: ids 0 .. pair_variants<R>() - 1 (0 is the default), and for R = float
// kVariantFold32, the shape of variant 0 with the phase fold in FP32 (a precision control).
// split_pmax > 0 (with out.part): one (pass, column segment) piece per workgroup, at most
// split_pmax pieces per curve, then the epilogue kernel; 0: every piece of a (curve, tile) in one
// workgroup.  Both give the same bits.
constexpr int kVariantFold32 = -1;
template <typename R>
int pair_variants();
template <typename R>
hipError_t launch_pairs(hipStream_t st, const CurveParams* cp, const int32_t* order,
                        int n_work_curves, const FreqPlan& fp, const double* t, const R* K,
                        const double* rd, const double* rp, const R* ks, const PairOut& out,
                        int variant, int split_pmax);
// The last kRemSlots slots of per-curve frequency lists (fp.kind 3) from slot0 on, one row per
// lane (FP32 path; pairs with fp.tile_cap = slot0 / kLanes on the main launch).
constexpr int kRemSlots = kLanes / 32;
hipError_t launch_pairs_rows(hipStream_t st, const CurveParams* cp, const int32_t* order,
                             int n_work_curves, const FreqPlan& fp, int slot0, const double* t,
                             const float* K, const double* rd, const PairOut& out);
// Mode sums of a frequency plan.  split_groups > 0 (with out.part,
// [rank][split_groups][count][3]): one harmonic group per wave, then the epilogue kernel; 0: every
// group in one wave.  Both give the same bits.
hipError_t launch_modes(hipStream_t st, const CurveParams* cp, const int32_t* order,
                        int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                        const PairOut& out, int split_groups);
hipError_t launch_mode_epilogue(hipStream_t st, const CurveParams* cp, const int32_t* order,
                                int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                                const PairOut& out, int split_groups);
// The same in FP64.  md: ts [block][4], rows the first of a block's node blocks (counted among the
// curve's), frag [block][kTiles64][64 lanes] values of U, node block k at k mod kTiles64,
// b [node block (from kTiles64 boff)][16].
hipError_t launch_prepare64(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                            const double* t, const double* y, const ModeDev& md);
hipError_t launch_modes64(hipStream_t st, const CurveParams* cp, const int32_t* order,
                          int n_work_curves, const FreqPlan& fp, const ModeDev& md,
                          const PairOut& out, int split_groups);
// The refinement windows of the curves with nodes > 0: every point's scores from the node sums that
// launch_modes left in out.score and out.score2.
hipError_t launch_mode_windows(hipStream_t st, const CurveParams* cp, int n_curves,
                               const FreqPlan& fp, const ModeDev& md, const PairOut& out);
// parts: nullable scratch of a split scan, parts_stride doubles per curve.
hipError_t launch_peaks(hipStream_t st, const CurveParams* cp, int n_curves, const double* coarse,
                        int n_coarse, double f0, double df, int top_k, int n_fine,
                        const MaskDev& md, const PeakOut& po, double* parts,
                        int64_t parts_stride);
hipError_t launch_best(hipStream_t st, const CurveParams* cp, int n_curves, const double* coarse,
                       const double* coarse2, int n_coarse, const double* fine,
                       const double* fine2, int top_k, int n_fine, int score_kind, double f0,
                       double df, const MaskDev& md, const PeakOut& po, const TieDev& tie,
                       DevResult* res);
// After launch_best with lists, for the curves idx[0 .. m): list[j][kTieMax], the frequencies of the
// points listed for curve idx[j] (NaN past the last); and the records rewritten with the best of them
// by their pair-sum scores score[j][kTieMax].
hipError_t launch_tie_lists(hipStream_t st, int m, const int32_t* idx, int top_k, int n_fine,
                            const PeakOut& po, const TieDev& tie, double* list);
hipError_t launch_best_of_ties(hipStream_t st, int m, const int32_t* idx, const double* score,
                               const double* fine, const double* fine2, int top_k, int n_fine,
                               int score_kind, const PeakOut& po, const TieDev& tie,
                               DevResult* res);

}  // namespace qmi
