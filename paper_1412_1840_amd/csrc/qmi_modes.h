// What the mode sums of both precisions (and the bands method) share: frequencies, scores, sines
// (device code).
#ifndef QMI_MODES_H
#define QMI_MODES_H

#include <math.h>

#include "qmi_internal.h"

namespace qmi {

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Frequency of slot s of curve c.  nodes > 0 (refinement windows): slots are the Chebyshev nodes of
// the curve's windows, nodes per window.
__device__ __forceinline__ double mode_slot_freq(const FreqPlan& fp, int c, int s, int nodes,
                                                 bool& active) {
    if (nodes > 0) {
        const int p = s / nodes, j = s - p * nodes;
        active = p < fp.npk[c];
        if (!active) return 0.0;
        const double* w = fp.win + ((int64_t)c * fp.top_k + p) * 2;
        const double half = 0.5 * w[1] * (double)(fp.n_fine - 1);
        return w[0] + half * (1.0 + cospi(((double)j + 0.5) / (double)nodes));
    }
    active = s < fp.count;
    if (!active) return 0.0;
    if (fp.kind == 0) return __dadd_rn(fp.f0, __dmul_rn((double)s, fp.df));
    if (fp.kind == 1) return fp.list[s];
    if (fp.kind == 3) {
        const double v = fp.list[(int64_t)c * fp.stride + s];
        active = v == v;
        return active ? v : 0.0;
    }
    const int p = s / fp.n_fine, m = s - p * fp.n_fine;
    if (p >= fp.npk[c]) {
        active = false;
        return 0.0;
    }
    const double* w = fp.win + ((int64_t)c * fp.top_k + p) * 2;
    return __dadd_rn(w[0], __dmul_rn((double)m, w[1]));
}

__device__ __forceinline__ void mode_nan(int64_t o, const PairOut& out) {
    out.score[o] = NAN;
    if (out.score2) out.score2[o] = NAN;
    if (out.ips) out.ips[o * 3 + 0] = out.ips[o * 3 + 1] = out.ips[o * 3 + 2] = NAN;
}

// V_J, IP_t, V_C and the scores from the three sums over ordered pairs without their constants.
__device__ __forceinline__ void mode_scores(const CurveParams& P, double SJ, double ST, double SC,
                                            int64_t o, const PairOut& out) {
    const double N = (double)P.n;
    const double VJ = P.A * P.B * SJ / (N * N);
    const double IPt = P.A * ST / (N * N);
    const double VC = P.A * P.B * SC / (N * N * N);
    const double VM = P.ipy * IPt;
    const double q = log(VJ) + log(VM) - 2.0 * log(VC);
    const double nckp = sqrt(N * P.sigma_t) / P.ipy * (VJ - VM);
    out.score[o] = out.score_kind == 0 ? q : nckp;
    if (out.score2) out.score2[o] = out.score_kind == 0 ? nckp : q;
    if (out.ips) {
        out.ips[o * 3 + 0] = VJ;
        out.ips[o * 3 + 1] = IPt;
        out.ips[o * 3 + 2] = VC;
    }
}

__device__ __forceinline__ void lds_add(double* p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

// sin and cos of p turns, |p| <= 1/2: the Taylor series of both at the nearest quarter turn
// (|r| <= 1/2 of a quarter; the first omitted terms are below 3e-19) and the quadrant identities.
// 33 instructions, where sincospi takes 61.
__device__ __forceinline__ void sincos_turns(double p, double* sn, double* cs) {
    constexpr double S[9] = {1.5707963267948966, -0.6459640975062463, 0.07969262624616705,
                             -0.004681754135318688, 0.00016044118478735983, -3.598843235212085e-06,
                             5.692172921967927e-08, -6.688035109811468e-10, 6.0669357311061955e-12};
    constexpr double C[9] = {1.0, -1.2337005501361697, 0.25366950790104803,
                             -0.02086348076335296, 0.0009192602748394266, -2.5202042373060607e-05,
                             4.710874778818172e-07, -6.386603083791852e-09, 6.565963114979473e-11};
    const double x = 4.0 * p, q = rint(x), r = x - q, u = r * r;
    double s = S[8], c = C[8];
#pragma unroll
    for (int k = 7; k >= 0; --k) {
        s = fma(u, s, S[k]);
        c = fma(u, c, C[k]);
    }
    s *= r;
    const int iq = (int)q;
    const double a = (iq & 1) ? c : s, b = (iq & 1) ? s : c;
    *sn = (iq & 2) ? -a : a;
    *cs = ((iq + 1) & 2) ? -b : b;
}

}  // namespace qmi

#endif  // QMI_MODES_H
