// HIP kernels for gfx950 (MI355X): the search around the pair sums of Protopapas et al.,
// arXiv:1412.1840 - the top local maxima of the coarse periodogram and their refinement windows
// (the trial periods are kept at the highest maxima of a spectrum, Sec. 3.1), and the best
// frequency of a curve (the score is maximised over trial frequencies, Sec. 3).
#include <math.h>

#include <algorithm>

#include "qmi_internal.h"

namespace qmi {

namespace {

// --------------------------------------------------------------------------------------------
// Peaks: local maxima of the coarse scores, best top_k by (score desc, k asc), and their
// refinement windows.  Candidates inside a spurious-period mask (Sec. 6.1) are left out of the
// argmax and of the maxima kept.  One block per curve.
// --------------------------------------------------------------------------------------------

constexpr int kWideBelow = 256;  // curves in a launch: one wide block per compute unit, or narrow ones

__device__ __forceinline__ bool better(double qa, int ka, double qb, int kb) {
    // a ranks before b: higher score, ties to lower index.  NaN never ranks.
    if (!(qa == qa)) return false;
    if (!(qb == qb)) return true;
    return qa > qb || (qa == qb && ka < kb);
}

__device__ __forceinline__ double grid_f(double f0, double df, int k) {
    return __dadd_rn(f0, __dmul_rn((double)k, df));
}

// The wave's best (score, index) by the rank order of better(), in every lane (butterfly).
__device__ __forceinline__ void wave_best(double& q, int& k) {
    for (int o = 32; o > 0; o >>= 1) {
        const double q2 = __shfl_xor(q, o, 64);
        const int k2 = __shfl_xor(k, o, 64);
        if (better(q2, k2, q, k)) {
            q = q2;
            k = k2;
        }
    }
}

// The value of one lane (wave-uniform), and of the lane below (lane 0: its own).
__device__ __forceinline__ double read_lane(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ int lane_below(int v) {
    return __builtin_amdgcn_update_dpp(v, v, 0x138, 0xf, 0xf, false);  // wave_shr:1
}
__device__ __forceinline__ double lane_below(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = lane_below((int)(b & 0xffffffffll)), hi = lane_below((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Ranks the entries of n_lists lists (each in rank order, [list][top_k]) and writes the best count
// of them and their refinement windows.
__device__ __forceinline__ void merge_lists(const double* lq, const int* lk, int n_lists,
                                            int count, int c, int F, double f0, double df,
                                            int top_k, int n_fine, const PeakOut& po) {
    for (int x = threadIdx.x; x < n_lists * top_k; x += blockDim.x) {
        const double xq = lq[x];
        const int k = lk[x];
        if (k == 0x7fffffff) continue;
        int p = 0;
        for (int v = 0; v < n_lists && p < count; ++v)
            for (int i = 0; i < top_k && better(lq[v * top_k + i], lk[v * top_k + i], xq, k); ++i)
                ++p;
        if (p >= count) continue;
        int a = k - 1, b = k + 1;
        if (F == 1) { a = 0; b = 0; }
        else if (k == 0) { a = 0; b = 1; }
        else if (k == F - 1) { a = F - 2; b = F - 1; }
        const double lo = grid_f(f0, df, a), hi = grid_f(f0, df, b);
        po.peak_k[(int64_t)c * top_k + p] = k;
        po.win[((int64_t)c * top_k + p) * 2 + 0] = lo;
        po.win[((int64_t)c * top_k + p) * 2 + 1] = (hi - lo) / (double)(n_fine - 1);
    }
}

// A part's list in the scratch of a split scan: scores, grid indices, the argmax's score and index.
__host__ __device__ constexpr int part_doubles(int top_k) { return 2 * top_k + 2; }

// Bound: the reads of the scores (8 bytes per grid point) for batches, latency for one curve.  A
// wave keeps its best top_k maxima in rank order, entry i in lane i, and takes a maximum in only
// where it beats the last of them: the longer the scan, the rarer (about 50 times in 1250 points
// for the best 10, 40 instructions each).  PART: the grid is cut into gridDim.y parts, one block
// each, whose lists peaks_merge_kernel joins.  Measured, 20 000 grid points, best 10, against a
// list per thread in LDS and a merge in top_k rounds: one curve 68 -> 30 us with the merge, 256
// curves 119 -> 51, 768 curves 142 -> 73.
constexpr int kPeakBlock = 256;
constexpr int kPeakParts = 32;    // most parts of a grid
constexpr int kPeakPart = 1024;  // fewest points of a part (a block's step)

template <bool PART>
__global__ void __launch_bounds__(kPeakBlock)
peaks_kernel(const CurveParams* __restrict__ cp, const double* __restrict__ coarse, int F,
             double f0, double df, int top_k, int n_fine, MaskDev md, PeakOut po,
             double* __restrict__ parts, int64_t parts_stride) {
    constexpr int BLOCK = kPeakBlock;
    constexpr int NW = BLOCK / 64;
    constexpr int kUnroll = 4;  // grid points of a lane whose loads are issued together
    __shared__ double wq[NW], lq[NW * QMI_MAX_TOPK];
    __shared__ int wk[NW], lk[NW * QMI_MAX_TOPK];
    __shared__ int wn[NW];
    const int c = blockIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double* q = coarse + (int64_t)c * F;
    const bool ok = cp[c].status == 0 && !cp[c].sparse;  // (no scores: left to the pair sums)
    int k_lo = 0, k_hi = F;  // this block's points
    if (PART) {
        const int len = (F + (int)gridDim.y - 1) / (int)gridDim.y;
        k_lo = min(F, (int)blockIdx.y * len);
        k_hi = min(F, k_lo + len);
    }
    double bq = NAN, hq = NAN;  // this lane's argmax; entry `lane` of the wave's list
    int bk = 0x7fffffff, hk = 0x7fffffff, n_loc = 0;
    double last_q = NAN;  // entry top_k - 1 of the wave's list (NaN until there is one)
    int last_k = 0x7fffffff;
    for (int k0 = k_lo + threadIdx.x; ok && k0 - lane < k_hi; k0 += kUnroll * BLOCK) {
        double v[kUnroll], lft[kUnroll], rgt[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + u * BLOCK;
            v[u] = k < k_hi ? q[k] : NAN;
            lft[u] = (k < k_hi && k > 0) ? q[k - 1] : NAN;
            rgt[u] = (k < k_hi && k + 1 < F) ? q[k + 1] : NAN;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int k = k0 + u * BLOCK;
            if (better(v[u], k, bq, bk) && !in_mask(md, grid_f(f0, df, k), v[u])) {
                bq = v[u];
                bk = k;
            }
            if (top_k <= 0) continue;
            bool peak;
            if (F == 1) peak = (v[u] == v[u]);
            else if (k == 0) peak = v[u] >= rgt[u];
            else if (k == F - 1) peak = v[u] > lft[u];
            else peak = v[u] > lft[u] && v[u] >= rgt[u];
            peak = peak && better(v[u], k, last_q, last_k) &&
                   !in_mask(md, grid_f(f0, df, k), v[u]);
            unsigned long long todo = __ballot(peak);
            while (todo) {
                const int src = __builtin_ctzll(todo);
                todo &= todo - 1;
                const double vq = read_lane(v[u], src);
                const int vk = k - lane + src;
                if (!better(vq, vk, last_q, last_k)) continue;
                const int at = __popcll(__ballot(better(hq, hk, vq, vk)));
                const double up_q = lane_below(hq);
                const int up_k = lane_below(hk);
                if (lane >= at) {
                    hq = lane == at ? vq : up_q;
                    hk = lane == at ? vk : up_k;
                }
                n_loc = min(n_loc + 1, top_k);
                if (lane >= top_k) {
                    hq = NAN;
                    hk = 0x7fffffff;
                }
                last_q = read_lane(hq, top_k - 1);
                last_k = __builtin_amdgcn_readlane(hk, top_k - 1);
            }
        }
    }
    wave_best(bq, bk);
    if (lane == 0) {
        wq[w] = bq;
        wk[w] = bk;
        wn[w] = n_loc;
    }
    if (lane < top_k) {
        lq[w * top_k + lane] = hq;
        lk[w * top_k + lane] = hk;
    }
    __syncthreads();
    int count = 0;
    for (int v = 0; v < NW; ++v) count += wn[v];
    count = min(count, top_k);
    if (threadIdx.x == 0) {
        for (int v = 1; v < NW; ++v)
            if (better(wq[v], wk[v], bq, bk)) {
                bq = wq[v];
                bk = wk[v];
            }
        if (!PART) {
            po.argmax[c] = (bk == 0x7fffffff) ? -1 : bk;
            po.npk[c] = count;
        }
    }
    if (!PART) {
        merge_lists(lq, lk, NW, count, c, F, f0, df, top_k, n_fine, po);
        return;
    }
    double* to = parts + (int64_t)c * parts_stride + (int64_t)blockIdx.y * part_doubles(top_k);
    for (int x = threadIdx.x; x < NW * top_k; x += BLOCK) {
        int p = 0;
        for (int v = 0; v < NW; ++v)
            for (int i = 0; i < top_k && better(lq[v * top_k + i], lk[v * top_k + i], lq[x], lk[x]);
                 ++i)
                ++p;
        if (lk[x] == 0x7fffffff || p >= top_k) continue;
        to[p] = lq[x];
        to[top_k + p] = (double)lk[x];
    }
    if (threadIdx.x == 0) {
        for (int p = count; p < top_k; ++p) to[top_k + p] = -1.0;
        to[2 * top_k] = bq;
        to[2 * top_k + 1] = bk == 0x7fffffff ? -1.0 : (double)bk;
    }
}

// The lists of a split scan joined: one block per curve.
__global__ void __launch_bounds__(kPeakBlock)
peaks_merge_kernel(int n_parts, int F, double f0, double df, int top_k, int n_fine, PeakOut po,
                   const double* __restrict__ parts, int64_t parts_stride) {
    __shared__ double lq[kPeakParts * QMI_MAX_TOPK];
    __shared__ int lk[kPeakParts * QMI_MAX_TOPK];
    __shared__ double aq[kPeakParts];
    __shared__ int ak[kPeakParts];
    __shared__ int total;
    const int c = blockIdx.x;
    const double* from = parts + (int64_t)c * parts_stride;
    if (threadIdx.x == 0) total = 0;
    __syncthreads();
    int mine = 0;
    for (int x = threadIdx.x; x < n_parts * top_k; x += kPeakBlock) {
        const double* pp = from + (int64_t)(x / top_k) * part_doubles(top_k);
        const double k = pp[top_k + x % top_k];
        lq[x] = k >= 0.0 ? pp[x % top_k] : NAN;
        lk[x] = k >= 0.0 ? (int)k : 0x7fffffff;
        mine += k >= 0.0;
    }
    if (mine) atomicAdd(&total, mine);
    if (threadIdx.x < n_parts) {
        const double* pp = from + (int64_t)threadIdx.x * part_doubles(top_k) + 2 * top_k;
        aq[threadIdx.x] = pp[0];
        ak[threadIdx.x] = pp[1] >= 0.0 ? (int)pp[1] : 0x7fffffff;
    }
    __syncthreads();
    const int count = min(total, top_k);
    if (threadIdx.x == 0) {
        double bq = aq[0];
        int bk = ak[0];
        for (int v = 1; v < n_parts; ++v)
            if (better(aq[v], ak[v], bq, bk)) {
                bq = aq[v];
                bk = ak[v];
            }
        po.argmax[c] = (bk == 0x7fffffff) ? -1 : bk;
        po.npk[c] = count;
    }
    merge_lists(lq, lk, n_parts, count, c, F, f0, df, top_k, n_fine, po);
}

// --------------------------------------------------------------------------------------------
// Best-of: highest refined score outside every mask, ties to the lower frequency then the lower
// peak rank; without a refined candidate, the coarse argmax; without that, an empty result.
// --------------------------------------------------------------------------------------------

// Points closer to the best than this are told apart by the pair sums.  Of QMI: the largest
// difference of two points' errors, mode sums (1e-7 at 40 samples, 5e-8 and less from 100 on) and pair
// sums (4e-7 at 121 samples, 2e-7 at 617) together.  nCKP = sqrt(N st) / IP_y (V_J - V_M), with
// relative errors of the V's of the same size.
__device__ __forceinline__ double tie_margin(const CurveParams& P, int score_kind, double best) {
    const double e = 4e-7 + 7e-5 / (double)P.n;
    return score_kind == 0 ? e : e * (fabs(best) + 2.0 * P.A * sqrt((double)P.n * P.sigma_t));
}

// The point that ranks first: higher score, ties to the lower frequency, then the lower slot.
struct BestPoint {
    double q, f;
    int s;
};
__device__ __forceinline__ bool ranks_before(const BestPoint& a, const BestPoint& b) {
    return a.q == a.q && (!(b.q == b.q) || a.q > b.q ||
                          (a.q == b.q && (a.f < b.f || (a.f == b.f && a.s < b.s))));
}

// Bound: latency of the two passes over the refined scores (the second, for near ties, from
// cache).  Measured, 10 windows of 1000 points, against one load in flight per thread and blocks
// of 256: one curve 27 -> 10 us (1024 threads),
// 768 curves 47 -> 24.
template <int BLOCK>
__global__ void __launch_bounds__(BLOCK)
best_kernel(const CurveParams* __restrict__ cp, const double* __restrict__ coarse,
            const double* __restrict__ coarse2, int F,
            const double* __restrict__ fine, const double* __restrict__ fine2, int top_k,
            int n_fine, int score_kind, double f0, double df, MaskDev md, PeakOut po, TieDev tie,
            DevResult* __restrict__ res) {
    constexpr int kUnroll = 4;
    __shared__ BestPoint wb[BLOCK / 64];
    __shared__ int n_ties;
    const int c = blockIdx.x;
    const CurveParams P = cp[c];
    const int npk = (top_k > 0 && n_fine > 0 && P.status == 0 && !P.sparse) ? po.npk[c] : 0;
    const int64_t S = (int64_t)top_k * n_fine;
    const int n_pts = npk * n_fine;
    const double* q = fine + (int64_t)c * S;
    auto freq = [&](int s) {
        const int p = s / n_fine, m = s - p * n_fine;
        const double* w = po.win + ((int64_t)c * top_k + p) * 2;
        return __dadd_rn(w[0], __dmul_rn((double)m, w[1]));
    };
    BestPoint best{NAN, INFINITY, 0x7fffffff};
    for (int s0 = threadIdx.x; s0 < n_pts; s0 += kUnroll * BLOCK) {
        double v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int s = s0 + u * BLOCK;
            v[u] = s < n_pts ? q[s] : NAN;
        }
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            if (!(v[u] == v[u]) || v[u] < best.q) continue;
            const int s = s0 + u * BLOCK;
            const BestPoint x{v[u], freq(s), s};
            if (ranks_before(x, best) && !in_mask(md, x.f, x.q)) best = x;
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        const BestPoint x{__shfl_xor(best.q, o, 64), __shfl_xor(best.f, o, 64),
                          __shfl_xor(best.s, o, 64)};
        if (ranks_before(x, best)) best = x;
    }
    if ((threadIdx.x & 63) == 0) wb[threadIdx.x >> 6] = best;
    if (threadIdx.x == 0) n_ties = 0;
    __syncthreads();
    best = wb[0];
    for (int v = 1; v < BLOCK / 64; ++v)
        if (ranks_before(wb[v], best)) best = wb[v];
    // The points that the mode sums cannot tell from the best (tie_margin), where there are any
    // besides it; with more than kTieMax the margin is halved until they fit.  After kTieHalvings
    // (1e-7 of the margin, below the sums' rounding) they count as equal: the first one stays.  A wave
    // counts its points at once, and a pass ends when there are too many of them.
    int listed = 0;
    if (tie.count && P.status == 0 && npk > 0 && best.s != 0x7fffffff &&
        tie.curves[c].groups > 0) {
        constexpr int kTieHalvings = 24;
        const int lane = threadIdx.x & 63;
        volatile int* total = &n_ties;
        double margin = tie_margin(P, score_kind, best.q);
        int found;
        for (int halvings = 0;; ++halvings) {
            for (int s0 = threadIdx.x; s0 - lane < n_pts; s0 += kUnroll * BLOCK) {
                if (*total > kTieMax) break;
                double v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int s = s0 + u * BLOCK;
                    v[u] = s < n_pts ? q[s] : NAN;
                }
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int s = s0 + u * BLOCK;
                    const bool in = v[u] >= best.q - margin && !in_mask(md, freq(s), v[u]);
                    const unsigned long long m = __ballot(in);
                    if (m == 0) continue;
                    int at = 0;
                    if (lane == 0) at = atomicAdd(&n_ties, __popcll(m));
                    at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1));
                    if (in && at < kTieMax) tie.slot[c * kTieMax + at] = s;
                }
            }
            __syncthreads();
            found = n_ties;
            if (found <= kTieMax) break;
            if (halvings == kTieHalvings) {
                found = 1;
                break;
            }
            margin *= 0.5;
            __syncthreads();
            if (threadIdx.x == 0) n_ties = 0;
            __syncthreads();
        }
        listed = found > 1 ? found : 0;
        if (threadIdx.x == 0) tie.count[c] = listed;
    } else if (tie.count && threadIdx.x == 0) {
        tie.count[c] = 0;
    }
    if (threadIdx.x != 0) return;
    DevResult r;
    r.sigma_y = P.sigma_y;
    r.sigma_t = P.sigma_t > 0.0 ? P.sigma_t : NAN;  // the rule flag until the prologue ran
    r.psnr = P.psnr;
    r.n = P.n;
    r.status = P.status;
    // 1: the pair sums take the curve over; 2: they decide its near ties.
    r.reserved = P.sparse ? 1 : listed ? 2 : 0;
    r.n_peaks = npk;
    const int am = (P.status == 0) ? po.argmax[c] : -1;
    r.coarse_argmax = am;
    r.coarse_best = (am >= 0) ? coarse[(int64_t)c * F + am] : NAN;
    if (P.status != 0 || ((npk == 0 || best.s == 0x7fffffff) && am < 0)) {
        r.f_best = r.period = r.score = r.score_qmi = r.score_nckp = NAN;
        r.coarse_index = r.peak_rank = r.fine_index = -1;
    } else if (npk == 0 || best.s == 0x7fffffff) {
        r.f_best = grid_f(f0, df, am);
        r.period = 1.0 / r.f_best;
        r.score = r.coarse_best;
        r.coarse_index = am;
        r.peak_rank = -1;
        r.fine_index = -1;
        const double other = coarse2 ? coarse2[(int64_t)c * F + am] : NAN;
        r.score_qmi = score_kind == 0 ? r.coarse_best : other;
        r.score_nckp = score_kind == 0 ? other : r.coarse_best;
    } else {
        const int s = best.s;
        const int p = s / n_fine, m = s - p * n_fine;
        r.f_best = best.f;
        r.period = 1.0 / r.f_best;
        r.score = best.q;
        const double other = fine2 ? fine2[(int64_t)c * S + s] : NAN;
        r.score_qmi = score_kind == 0 ? best.q : other;
        r.score_nckp = score_kind == 0 ? other : best.q;
        r.coarse_index = po.peak_k[(int64_t)c * top_k + p];
        r.peak_rank = p;
        r.fine_index = m;
    }
    res[c] = r;
}

__device__ __forceinline__ double slot_of_window(const PeakOut& po, int c, int top_k, int n_fine,
                                                 int s) {
    const double* w = po.win + ((int64_t)c * top_k + s / n_fine) * 2;
    return __dadd_rn(w[0], __dmul_rn((double)(s % n_fine), w[1]));
}

__global__ void tie_lists_kernel(int m, const int32_t* __restrict__ idx, int top_k, int n_fine,
                                 PeakOut po, TieDev tie, double* __restrict__ list) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x, j = x / kTieMax, k = x % kTieMax;
    if (j >= m) return;
    const int c = idx[j];
    list[x] = k < tie.count[c] ? slot_of_window(po, c, top_k, n_fine, tie.slot[c * kTieMax + k])
                               : NAN;
}

// The record of a curve with a list of near ties: the point with the highest pair-sum score (ties to
// the lower frequency, then the lower peak rank), with its scores as the refinement formed them.
__global__ void best_of_ties_kernel(int m, const int32_t* __restrict__ idx,
                                    const double* __restrict__ score,
                                    const double* __restrict__ fine,
                                    const double* __restrict__ fine2, int top_k, int n_fine,
                                    int score_kind, PeakOut po, TieDev tie,
                                    DevResult* __restrict__ res) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= m) return;
    const int c = idx[j];
    const int64_t S = (int64_t)top_k * n_fine;
    double bq = NAN, bf = INFINITY;
    int bs = 0x7fffffff;
    for (int k = 0; k < tie.count[c]; ++k) {
        const double v = score[j * kTieMax + k];
        const int s = tie.slot[c * kTieMax + k];
        const double fr = slot_of_window(po, c, top_k, n_fine, s);
        if ((v == v) &&
            (!(bq == bq) || v > bq || (v == bq && (fr < bf || (fr == bf && s < bs))))) {
            bq = v;
            bf = fr;
            bs = s;
        }
    }
    if (bs == 0x7fffffff) return;
    DevResult& r = res[c];
    r.f_best = bf;
    r.period = 1.0 / bf;
    r.score = fine[(int64_t)c * S + bs];
    const double other = fine2 ? fine2[(int64_t)c * S + bs] : NAN;
    r.score_qmi = score_kind == 0 ? r.score : other;
    r.score_nckp = score_kind == 0 ? other : r.score;
    r.coarse_index = po.peak_k[(int64_t)c * top_k + bs / n_fine];
    r.peak_rank = bs / n_fine;
    r.fine_index = bs % n_fine;
}

}  // namespace

hipError_t launch_peaks(hipStream_t st, const CurveParams* cp, int n_curves, const double* coarse,
                        int n_coarse, double f0, double df, int top_k, int n_fine,
                        const MaskDev& md, const PeakOut& po, double* parts,
                        int64_t parts_stride) {
    if (n_curves <= 0) return hipSuccess;
    // Few curves leave most of the chip idle: their grids are cut into parts until there are about
    // two blocks per compute unit, where the scratch has room for the parts' lists.  One curve:
    // 47 us by one block of 1024 threads, 30 by 19 parts and their merge.
    int64_t n_parts = std::min<int64_t>({kPeakParts, 512 / n_curves, n_coarse / kPeakPart,
                                         parts ? parts_stride / part_doubles(top_k) : 0});
    if (n_parts < 2) {
        peaks_kernel<false><<<n_curves, kPeakBlock, 0, st>>>(cp, coarse, n_coarse, f0, df, top_k,
                                                             n_fine, md, po, nullptr, 0);
        return hipGetLastError();
    }
    peaks_kernel<true><<<dim3(n_curves, (unsigned)n_parts), kPeakBlock, 0, st>>>(
        cp, coarse, n_coarse, f0, df, top_k, n_fine, md, po, parts, parts_stride);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    peaks_merge_kernel<<<n_curves, kPeakBlock, 0, st>>>((int)n_parts, n_coarse, f0, df, top_k,
                                                        n_fine, po, parts, parts_stride);
    return hipGetLastError();
}

hipError_t launch_best(hipStream_t st, const CurveParams* cp, int n_curves, const double* coarse,
                       const double* coarse2, int n_coarse, const double* fine,
                       const double* fine2, int top_k, int n_fine, int score_kind, double f0,
                       double df, const MaskDev& md, const PeakOut& po, const TieDev& tie,
                       DevResult* res) {
    if (n_curves <= 0) return hipSuccess;
    if (n_curves < kWideBelow)
        best_kernel<1024><<<n_curves, 1024, 0, st>>>(cp, coarse, coarse2, n_coarse, fine, fine2,
                                                     top_k, n_fine, score_kind, f0, df, md, po, tie,
                                                     res);
    else
        best_kernel<256><<<n_curves, 256, 0, st>>>(cp, coarse, coarse2, n_coarse, fine, fine2,
                                                   top_k, n_fine, score_kind, f0, df, md, po, tie,
                                                   res);
    return hipGetLastError();
}

hipError_t launch_tie_lists(hipStream_t st, int m, const int32_t* idx, int top_k, int n_fine,
                            const PeakOut& po, const TieDev& tie, double* list) {
    tie_lists_kernel<<<(m * kTieMax + 255) / 256, 256, 0, st>>>(m, idx, top_k, n_fine, po, tie,
                                                                list);
    return hipGetLastError();
}

hipError_t launch_best_of_ties(hipStream_t st, int m, const int32_t* idx, const double* score,
                               const double* fine, const double* fine2, int top_k, int n_fine,
                               int score_kind, const PeakOut& po, const TieDev& tie,
                               DevResult* res) {
    best_of_ties_kernel<<<(m + 63) / 64, 64, 0, st>>>(m, idx, score, fine, fine2, top_k, n_fine,
                                                      score_kind, po, tie, res);
    return hipGetLastError();
}

}  // namespace qmi
