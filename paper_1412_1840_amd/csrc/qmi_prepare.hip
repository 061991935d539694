// HIP kernel for gfx950 (MI355X): the per-curve preparation of the sums of Protopapas et al.,
// arXiv:1412.1840 - kernel widths (Sec. 2, Sec. 3), pSNR (Sec. 5.2), and the node tables of the mode
// sums (qmi_modes.hip).  One workgroup per curve.
#include <math.h>

#include <algorithm>

#include "qmi_internal.h"
#include "qmi_sort.h"

namespace qmi {

namespace {

constexpr double kInvSqrt2Pi = 0.39894228040143267793994605993438187;

// Sums over a curve are formed by the first kSumThreads threads whatever the block (a curve's
// results do not depend on the longest curve of its batch): wave shuffles, then the waves in order.
constexpr int kSumThreads = 256;

__device__ double block_sum(double v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0 && threadIdx.x < kSumThreads) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (int k = 0; k < kSumThreads / 64; ++k) s += sh[k];
    __syncthreads();
    return s;
}

// Exclusive prefix sum of one value per thread; *total receives the sum.
template <int BLOCK>
__device__ int block_scan(int v, int* sh, int* total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int s = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(s, o, 64);
        if (lane >= o) s += u;
    }
    __syncthreads();
    if (lane == 63) sh[w] = s;
    __syncthreads();
    int base = 0, all = 0;
    for (int k = 0; k < BLOCK / 64; ++k) {
        if (k < w) base += sh[k];
        all += sh[k];
    }
    __syncthreads();
    *total = all;
    return base + s - v;
}

// Quantile by linear interpolation at position (n-1) p of sorted a[0..n).
__device__ double sorted_quantile(const double* a, int n, double p) {
    double h = (n - 1) * p;
    int lo = (int)floor(h);
    int hi = lo + 1 < n ? lo + 1 : n - 1;
    return a[lo] + (h - lo) * (a[hi] - a[lo]);
}

__device__ double sorted_median(const double* a, int n) {
    return (n & 1) ? a[n / 2] : 0.5 * (a[n / 2 - 1] + a[n / 2]);
}

// Distance (y - y0) inv in two parts, exact but for the rounding of inv (an outlier puts the others
// far from y0).
struct Exact {
    double hi, lo;
};
__device__ __forceinline__ Exact node_units(double y, double y0, double inv) {
    const double s = y - y0, v = s - y;
    const double err = (y - (s - v)) - (y0 + v);
    const double x = s * inv;
    return Exact{x, fma(s, inv, -x) + err * inv};
}

// Coefficients cs[0..cap] of the periodic kernel's cosine series by the trapezoid rule over the
// circle (exact up to the coefficients past L - m).  ev, ct: L = 3 cap + 32 entries each.
template <int BLOCK>
__device__ void series_coefficients(double sigma_t, int cap, double* ev, double* ct, double* cs) {
    const int L = 3 * cap + 32, tid = threadIdx.x;
    const double kap = 1.0 / (sigma_t * sigma_t);
    for (int j = tid; j < L; j += BLOCK) {
        const double x = (double)j / (double)L, sn = sinpi(x);
        ct[j] = cospi(2.0 * x);
        ev[j] = exp(-2.0 * kap * sn * sn);  // (cos - 1 would lose kap roundings where it is small)
    }
    __syncthreads();
    for (int m = tid; m <= cap; m += BLOCK) {
        double a = 0.0;
        int k = 0;
#pragma unroll 4
        for (int j = 0; j < L; ++j) {
            a = fma(ev[j], ct[k], a);
            k += m;
            if (k >= L) k -= L;
        }
        cs[m] = (m ? 2.0 : 1.0) * a / (double)L;
    }
}

// Waves that form operand tiles, and the bytes of a tile (two node blocks, two parts, 64 lanes).
template <int BLOCK>
constexpr int tile_waves() {
    return BLOCK <= 512 ? BLOCK / 64 : 8;
}
constexpr int kTileBytes = 4096;

// LDS bytes of the sort keys, which the series tables (2 L + cap + 1 doubles) take over: a multiple
// of 16, since the operand tiles that follow are read 16 bytes at a time.
int key_bytes_of(int room, int mode_cap) {
    const int series = mode_cap ? 2 * (3 * mode_cap + 32) + mode_cap + 2 : 0;
    return (8 * std::max(room, series) + 15) / 16 * 16;
}

// Bound: latency (one curve per call: a chain of sorts, scans and reductions by one workgroup),
// FP64 exponentials where one workgroup has a long curve.  Measured against separate prologue and
// node kernels with sorts in LDS and one exponential per node and sample: one curve of 617 samples
// 119 -> 46 us (55 by the small block), one of 8192 1274 -> 300 us, 768 survey curves 206 -> 104 us.
template <int BLOCK, int EMAX>
__global__ void __launch_bounds__(BLOCK)
prepare_kernel(CurveParams* __restrict__ cp, const double* __restrict__ t_all,
               const double* __restrict__ y_all, const double* __restrict__ e_all,
               double skew_lambda, double skew_mu, int room, int key_bytes, int group_room,
               ModeDev md) {
    extern __shared__ __attribute__((aligned(16))) double psh[];
    __shared__ double red[kSumThreads / 64];
    __shared__ int ired[BLOCK / 64];
    __shared__ int bad;
    __shared__ double s_sy, s_st;
    __shared__ double s_lo[BLOCK / 64], s_hi[BLOCK / 64];
    const int c = blockIdx.x, tid = threadIdx.x;
    const CurveParams P = cp[c];
    const int n = P.n;
    if (P.status != 0) return;
    double* key = psh;
    int32_t* idx = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(psh) + key_bytes);
    const double* t = t_all + P.off;
    const double* y = y_all + P.off;
    const double* e = P.has_e ? e_all + P.off : nullptr;
    if (tid == 0) bad = 0;
    __syncthreads();
    double s = 0.0, t_lo = INFINITY, t_hi = -INFINITY;
    for (int i = tid; i < n; i += BLOCK) {
        const double ti = t[i];
        const bool ok = isfinite(ti) && isfinite(y[i]) && (!e || isfinite(e[i]));
        if (!ok) bad = 1;
        t_lo = fmin(t_lo, ti);
        t_hi = fmax(t_hi, ti);
    }
    for (int o = 32; o > 0; o >>= 1) {
        t_lo = fmin(t_lo, __shfl_xor(t_lo, o, 64));
        t_hi = fmax(t_hi, __shfl_xor(t_hi, o, 64));
    }
    if ((tid & 63) == 0) {
        s_lo[tid >> 6] = t_lo;
        s_hi[tid >> 6] = t_hi;
    }
    if (tid < kSumThreads)
        for (int i = tid; i < n; i += kSumThreads) s += y[i];
    __syncthreads();
    if (bad || n < 2) {
        if (tid == 0) cp[c].status = -1;  // QMI_EINVAL
        return;
    }
    // Mean and sample deviation of y.
    const double mean = block_sum(s, red) / n;
    s = 0.0;
    if (tid < kSumThreads)
        for (int i = tid; i < n; i += kSumThreads) {
            const double d = y[i] - mean;
            s += d * d;
        }
    const double sdev = sqrt(block_sum(s, red) / (n - 1));
    double med_e = NAN;
    if (e) {
        for (int i = tid; i < n; i += BLOCK) key[i] = e[i];
        sort_block<BLOCK, EMAX, false>(key, idx, n);
        med_e = sorted_median(key, n);
        __syncthreads();
    }
    for (int i = tid; i < n; i += BLOCK) {
        key[i] = y[i];
        idx[i] = i;
    }
    sort_block<BLOCK, EMAX, true>(key, idx, n);
    if (tid == 0) {
        const double iqr = sorted_quantile(key, n, 0.75) - sorted_quantile(key, n, 0.25);
        // sigma_t rule (Sec. 3): S = (Q3 + Q1 - 2 Q2) / (Q3 - Q1) with Q2 the median and Q1, Q3 the
        // medians of the lower and upper n / 2 sorted magnitudes; S = 0 when Q3 = Q1.
        double sigma_t = P.sigma_t;
        if (!(sigma_t > 0.0)) {
            const int h = n / 2;
            const double q1 = sorted_median(key, h), q2 = sorted_median(key, n);
            const double q3 = sorted_median(key + (n - h), h);
            const double S = (q3 == q1) ? 0.0 : (q3 + q1 - 2.0 * q2) / (q3 - q1);
            sigma_t = skew_lambda + 0.5 * exp(-skew_mu * S * S);
        }
        double sy = 0.0;
        int status = 0;
        if (P.sigma_y_rule > 0.0) {
            sy = P.sigma_y_rule;
        } else if (P.sigma_y_rule == -1.0) {
            if (sdev == 0.0) {
                status = -4;  // QMI_EDEGENERATE
            } else {
                double spread = (iqr == 0.0) ? sdev : fmin(sdev, iqr / 1.34);
                sy = 0.9 * spread * pow((double)n, -0.2);
            }
        } else {
            if (!(med_e > 0.0)) status = e ? -4 : -1;
            sy = med_e;
        }
        cp[c].status = status;
        cp[c].sigma_y = status ? NAN : sy;
        cp[c].sigma_t = sigma_t;
        cp[c].A = kInvSqrt2Pi / sigma_t;
        cp[c].B = status ? NAN : kInvSqrt2Pi / sy;
        cp[c].psnr = (e && med_e > 0.0) ? 0.7413 * iqr / med_e : NAN;
        s_sy = status ? NAN : sy;
        s_st = sigma_t;
    }
    if (!md.curves) return;
    ModeCurve M = md.curves[c];
    if (M.cap == 0) return;
    __syncthreads();
    const double sigma_y = s_sy, sigma_t = s_st;
    if (!(sigma_y == sigma_y)) return;

    // ---- Node tables.  Groups of samples (in magnitude order) with the same first node block.
    int* g_first = reinterpret_cast<int*>(idx) + std::max(room, tile_waves<BLOCK>() * kTileBytes / 4);
    int* g_block = g_first + group_room + 1;  // first block of samples of a group
    int* g_row = g_block + group_room + 1;    // first node block, counted among those in use
    int* g_rb = g_row + group_room;           // and by magnitude
    const double y0 = key[0];
    const double inv = 1.0 / (kNodeStep * sigma_y);
    bool sparse = !((key[n - 1] - y0) * inv < 1e9);  // far more nodes than samples can use
    // Position of a sample in node units from node kReach, and its first node block.
    auto pos = [&](int i) { return node_units(key[i], y0, inv); };
    auto blk = [&](int i) { return (int)rint(pos(i).hi) >> 4; };
    int n_groups = 0, n_rows = 0, n_blocks = 0;
    if (!sparse) {
        const int per = (n + BLOCK - 1) / BLOCK;
        const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
        int cnt = 0, all = 0;  // groups in the low, node blocks in the high half
        // A group brings two new node blocks, or one where the group before it starts one lower.
        for (int i = i0; i < i1; ++i) {
            const int d = i == 0 ? 2 : min(2, blk(i) - blk(i - 1));
            if (d > 0) cnt += 1 + (d << 16);
        }
        int at = block_scan<BLOCK>(cnt, ired, &all);
        n_groups = all & 0xffff;
        n_rows = all >> 16;
        sparse = n_groups > M.cap;
        if (!sparse) {
            for (int i = i0; i < i1; ++i) {
                const int b = blk(i);
                const int d = i == 0 ? 2 : min(2, b - blk(i - 1));
                if (d <= 0) continue;
                const int g = at & 0xffff;
                at += 1 + (d << 16);
                g_first[g] = i;
                g_rb[g] = b;
                g_row[g] = (at >> 16) - 2;
            }
            if (tid == 0) g_first[n_groups] = n;
            __syncthreads();
            // Blocks of 32 samples: every group starts a new one.
            const int gper = (n_groups + BLOCK - 1) / BLOCK;
            const int a0 = min(n_groups, tid * gper), a1 = min(n_groups, a0 + gper);
            int nb = 0;
            for (int g = a0; g < a1; ++g) nb += (g_first[g + 1] - g_first[g] + 31) >> 5;
            int f = block_scan<BLOCK>(nb, ired, &n_blocks);
            for (int g = a0; g < a1; ++g) {
                g_block[g] = f;
                f += (g_first[g + 1] - g_first[g] + 31) >> 5;
            }
            if (tid == 0) g_block[n_groups] = n_blocks;
            sparse = n_blocks > M.cap || 2 * n_blocks + n_groups > M.limit;
        }
        __syncthreads();
    }
    if (sparse) {
        if (tid == 0) {
            md.curves[c].groups = 0;
            cp[c].sparse = 1;
        }
        return;
    }
    auto group_of = [&](int block) {
        int lo = 0, hi = n_groups - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (g_block[mid] <= block) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    // Times in magnitude order, every group padded to whole blocks; counted from a sample's, so that
    // phases that coincide are near 0 (qmi_modes.hip).
    const double t0 = t[idx[n / 2]];
    double* ts = md.ts + 32 * M.boff;
    int32_t* rows = md.rows + M.boff;
    for (int q = tid; q < 32 * n_blocks; q += BLOCK) {
        const int g = group_of(q >> 5);
        const int i = g_first[g] + q - 32 * g_block[g];
        ts[q] = i < g_first[g + 1] ? t[idx[i]] - t0 : 0.0;
        if ((q & 31) == 0) rows[q >> 5] = g_row[g];
    }
    __syncthreads();  // idx is free from here
    // Fragments of U in the operand layout of the 16x16x32 matrix instruction: lane l holds node
    // l mod 16 and samples 8 (l / 16) ... + 7 of the block, as a high and a low half-precision
    // part; and each node's sum over the block's samples.  A lane forms the 16 nodes of one node
    // block for one sample from the middle outwards: U at the next node is U times a ratio, and
    // the ratio falls by exp(-2 h^2) per node, so that a block of 16 takes three exponentials.
    half8v* frag = reinterpret_cast<half8v*>(md.frag) + M.boff * 256;
    double* part = md.part + M.boff * 32;
    double* bsum = md.b + M.boff * 32;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave < tile_waves<BLOCK>()) {
        _Float16* tile = reinterpret_cast<_Float16*>(idx) + wave * (kTileBytes / 2);
        const double fall = exp(-2.0 * kNodeStep * kNodeStep);
        for (int b = wave; b < n_blocks; b += tile_waves<BLOCK>()) {
            const int g = group_of(b);
            const int i = lane & 31, nb = lane >> 5;
            const int smp = g_first[g] + 32 * (b - g_block[g]) + i;
            double v = 0.0, up = 0.0, down = 0.0;
            if (smp < g_first[g + 1]) {
                const Exact x = pos(smp);
                const double d =
                    ((double)(16 * (g_rb[g] + nb) + 8 - kReach) - x.hi - x.lo) * kNodeStep;
                v = kNodeScale * exp(-d * d);
                up = exp(-2.0 * kNodeStep * d - kNodeStep * kNodeStep);
                down = exp(2.0 * kNodeStep * d - kNodeStep * kNodeStep);
            }
            // Element of node r: part hl of node block nb at ((nb 2 + hl) 64 + 16 (i/8) + r) 8 + i%8.
            _Float16* to = tile + (nb * 128 + 16 * (i >> 3)) * 8 + (i & 7);
            auto put = [&](int r, double x) {
                const _Float16 h = (_Float16)(float)x;
                to[r * 8] = h;
                to[512 + r * 8] = (_Float16)(float)(x - (double)(float)h);
            };
            // Nodes past either end of the two blocks add their values to the last node, so that
            // sum_q U is the same for every sample (three of them: the next is below 1e-9 of these).
            put(8, v);
            double x = v, last = 0.0;
#pragma unroll
            for (int r = 9; r < 19; ++r) {
                x *= up;
                up *= fall;
                if (r < 15) put(r, x);
                else if (r == 15 || nb == 1) last += x;
            }
            put(15, last);
            x = v;
            last = 0.0;
#pragma unroll
            for (int r = 7; r >= -3; --r) {
                x *= down;
                down *= fall;
                if (r > 0) put(r, x);
                else if (r == 0 || nb == 0) last += x;
            }
            put(0, last);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const half8v* tv = reinterpret_cast<const half8v*>(tile);
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const half8v h = tv[k * 128 + lane], l = tv[k * 128 + 64 + lane];
                frag[(int64_t)b * 256 + k * 128 + lane] = h;
                frag[(int64_t)b * 256 + k * 128 + 64 + lane] = l;
                double sum = 0.0;
#pragma unroll
                for (int j = 0; j < 8; ++j) sum += (double)(float)h[j] + (double)(float)l[j];
                sum += __shfl_xor(sum, 16, 64);
                sum += __shfl_xor(sum, 32, 64);
                if (lane < 16) part[(int64_t)(2 * b + k) * 16 + lane] = sum;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    double sq = 0.0;
    if (tid < kSumThreads)
        for (int q = tid; q < 16 * n_rows; q += kSumThreads) {
            const int row = q >> 4;
            int lo = 0, hi = n_groups - 1;  // first group that reaches the node block
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (g_row[mid] + 1 >= row) hi = mid; else lo = mid + 1;
            }
            double b = 0.0;
            for (int g = lo; g < n_groups && g_row[g] <= row; ++g)
                for (int r = g_block[g]; r < g_block[g + 1]; ++r)
                    b += part[(int64_t)(2 * r + row - g_row[g]) * 16 + (q & 15)];
            bsum[q] = b;
            sq = fma(b, b, sq);
        }
    sq = block_sum(sq, red);
    // Coefficients, and the number of harmonics to keep.
    const int cap = md.mode_cap, L = 3 * cap + 32;
    double* ev = psh;
    double* ct = psh + L;
    double* cs = ct + L;  // [cap + 1]
    series_coefficients<BLOCK>(sigma_t, cap, ev, ct, cs);
    // Frequencies per refinement window.  Harmonic m of the sums runs through at most
    // w = pi m T W (T the curve's time span, W the window) radians from the window's middle to its
    // end, and its Chebyshev coefficients fall below eps past the degree
    // w + s (w/2)^(1/3) + 0.12 s^2 / (w/2)^(1/3), s = (3/2 ln(2/eps))^(2/3) (the Bessel functions
    // J_d(w) past their turning point; checked against them for w in [0.01, 600], eps in
    // [1e-11, 0.1]: never short, at most a tenth over from w = 10 on).
    if (tid == 0) ired[1] = 0;
    __syncthreads();
    if (md.win_width > 0.0) {
        double lo = s_lo[0], hi = s_hi[0];
        for (int k = 1; k < BLOCK / 64; ++k) {
            lo = fmin(lo, s_lo[k]);
            hi = fmax(hi, s_hi[k]);
        }
        for (int m = tid; m <= cap; m += BLOCK) {
            if (m == 0 || cs[m] <= kWinTol) continue;
            const double w = M_PI * m * (hi - lo) * md.win_width;
            const double q = 1.5 * log(2.0 * cs[m] / kWinTol);
            const double r = cbrt(q), h = fmax(cbrt(0.5 * w), 0.6);
            const double d = w + r * r * cbrt(0.5 * w) + 0.12 * r * r * r * r / h;
            atomicMax(&ired[1], d < 1e6 ? (int)d + 2 : 1000000);
        }
    }
    __syncthreads();
    if (tid == 0) {
        int m = cap;
        double tail = 0.0;
        for (; m > 1; --m) {
            tail += cs[m];
            if (tail > kModeTail) break;
        }
        M.groups = min((m + kModeGroup - 1) / kModeGroup, md.max_groups);
        // All harmonics of the groups, and what is left of the series with the last of them, so that
        // the kernel is 1 where phases coincide.
        m = M.groups * kModeGroup;
        ired[0] = m;
        for (int k = m + 1; k <= cap; ++k) cs[m] += cs[k];
        M.blocks = n_blocks;
        // Windows are interpolated where that takes at most half of their points (whose score
        // arrays hold the node sums meanwhile).
        M.nodes = (ired[1] > 0 && ired[1] <= kWinNodesMax && 2 * ired[1] <= md.n_fine) ? ired[1] : 0;
        M.c0 = cs[0];
        M.sj0 = kNodeW * sq;
        md.curves[c] = M;
        cp[c].ipy = kInvSqrt2Pi / sigma_y * M.sj0 / ((double)n * (double)n);
    }
    __syncthreads();
    // Coefficient of harmonic m at m - 1.
    const int keep = ired[0];
    double* coef = md.coef + (int64_t)c * mode_stride(cap);
    for (int m = tid + 1; m <= keep; m += BLOCK) coef[m - 1] = cs[m];
}

template <int BLOCK, int EMAX>
hipError_t launch_prepare_b(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                            const double* t, const double* y, const double* e,
                            double skew_lambda, double skew_mu, const ModeDev& md) {
    const int room = sort_room(BLOCK, max_n);
    const int key_bytes = key_bytes_of(room, md.curves ? md.mode_cap : 0);
    if (key_bytes % (int)sizeof(half8v) != 0) return hipErrorInvalidValue;
    const int group_room = max_n / 5 + 1;
    size_t lds = (size_t)key_bytes + 4 * (size_t)room;
    if (md.curves)
        lds = (size_t)key_bytes + std::max(4 * room, tile_waves<BLOCK>() * kTileBytes) +
              4 * (size_t)(4 * group_room + 2);
    prepare_kernel<BLOCK, EMAX><<<n_curves, BLOCK, lds, st>>>(
        cp, t, y, e, skew_lambda, skew_mu, room, key_bytes, group_room, md);
    return hipGetLastError();
}

// The node tables of the FP64 mode sums, as above but for exact operands: three node blocks per sample,
// blocks of 4 samples, the value of every node and sample by its own exponential.  Bound: latency
// (sort, scans, reductions); measured, 16 survey curves 62 us.
template <int BLOCK, int EMAX>
__global__ void __launch_bounds__(BLOCK)
prepare64_kernel(CurveParams* __restrict__ cp, const double* __restrict__ t_all,
                 const double* __restrict__ y_all, int room, int key_bytes, int group_room,
                 ModeDev md) {
    extern __shared__ __attribute__((aligned(16))) double psh[];
    __shared__ double red[kSumThreads / 64];
    __shared__ int ired[BLOCK / 64];
    const int c = blockIdx.x, tid = threadIdx.x;
    const CurveParams P = cp[c];
    ModeCurve M = md.curves[c];
    if (P.status != 0 || M.cap == 0) return;
    const int n = P.n;
    const double* t = t_all + P.off;
    const double* y = y_all + P.off;
    double* key = psh;
    int32_t* idx = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(psh) + key_bytes);
    int* g_first = reinterpret_cast<int*>(idx) + room;
    int* g_block = g_first + group_room + 1;  // first block of samples of a group
    int* g_row = g_block + group_room + 1;    // first node block, counted among those in use
    int* g_rb = g_row + group_room;           // and by magnitude
    for (int i = tid; i < n; i += BLOCK) {
        key[i] = y[i];
        idx[i] = i;
    }
    sort_block<BLOCK, EMAX, true>(key, idx, n);
    const double y0 = key[0], inv = 1.0 / (kNodeStep64 * P.sigma_y);
    bool sparse = !((key[n - 1] - y0) * inv < 1e9);
    auto pos = [&](int i) { return node_units(key[i], y0, inv); };  // from node kReach64
    auto blk = [&](int i) { return (int)rint(pos(i).hi) >> 4; };
    int n_groups = 0, n_rows = 0, n_blocks = 0;
    if (!sparse) {
        constexpr int kShift = 14;  // groups (at most 8192) below, node blocks (3 per group) above
        static_assert(QMI_MAX_N < (1 << kShift) && QMI_MAX_N * kTiles64 < (1 << 17), "packed counts");
        const int per = (n + BLOCK - 1) / BLOCK;
        const int i0 = min(n, tid * per), i1 = min(n, i0 + per);
        int cnt = 0, all = 0;
        for (int i = i0; i < i1; ++i) {
            const int d = i == 0 ? kTiles64 : min(kTiles64, blk(i) - blk(i - 1));
            if (d > 0) cnt += 1 + (d << kShift);
        }
        int at = block_scan<BLOCK>(cnt, ired, &all);
        n_groups = all & ((1 << kShift) - 1);
        n_rows = all >> kShift;
        sparse = n_groups > M.cap;
        if (!sparse) {
            for (int i = i0; i < i1; ++i) {
                const int b = blk(i);
                const int d = i == 0 ? kTiles64 : min(kTiles64, b - blk(i - 1));
                if (d <= 0) continue;
                const int g = at & ((1 << kShift) - 1);
                at += 1 + (d << kShift);
                g_first[g] = i;
                g_rb[g] = b;
                g_row[g] = (at >> kShift) - kTiles64;
            }
            if (tid == 0) g_first[n_groups] = n;
            __syncthreads();
            const int gper = (n_groups + BLOCK - 1) / BLOCK;
            const int a0 = min(n_groups, tid * gper), a1 = min(n_groups, a0 + gper);
            int nb = 0;
            for (int g = a0; g < a1; ++g) nb += (g_first[g + 1] - g_first[g] + 3) >> 2;
            int f = block_scan<BLOCK>(nb, ired, &n_blocks);
            for (int g = a0; g < a1; ++g) {
                g_block[g] = f;
                f += (g_first[g + 1] - g_first[g] + 3) >> 2;
            }
            if (tid == 0) g_block[n_groups] = n_blocks;
            sparse = n_blocks > M.cap || 2 * n_blocks + n_groups > M.limit;
        }
        __syncthreads();
    }
    if (sparse) {
        if (tid == 0) {
            md.curves[c].groups = 0;
            cp[c].sparse = 1;
        }
        return;
    }
    auto group_of = [&](int block) {
        int lo = 0, hi = n_groups - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (g_block[mid] <= block) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    double* ts = md.ts + 4 * M.boff;
    int32_t* rows = md.rows + M.boff;
    double* frag = reinterpret_cast<double*>(md.frag) + 64 * kTiles64 * M.boff;
    double* bsum = md.b + 16 * kTiles64 * M.boff;
    const int lane = tid & 63, wave = tid >> 6;
    for (int b = wave; b < n_blocks; b += BLOCK / 64) {
        const int g = group_of(b), r0 = g_row[g];
        const int smp = g_first[g] + 4 * (b - g_block[g]) + (lane >> 4);
        const bool has = smp < g_first[g + 1];
        const Exact x = has ? pos(smp) : Exact{0.0, 0.0};
        for (int k = 0; k < kTiles64; ++k) {
            const int node = 16 * (g_rb[g] + k) + (lane & 15) - kReach64;
            const double d = ((double)node - x.hi - x.lo) * kNodeStep64;
            frag[((int64_t)b * kTiles64 + (r0 + k) % kTiles64) * 64 + lane] =
                has ? exp(-d * d) : 0.0;
        }
        if ((lane & 15) == 0) ts[4 * b + (lane >> 4)] = has ? t[idx[smp]] : 0.0;
        if (lane == 0) rows[b] = r0;
    }
    __syncthreads();
    // Sums of a node block's 16 nodes over all samples: one wave, four lanes per node.
    for (int k = wave; k < n_rows; k += BLOCK / 64) {
        int lo = 0, hi = n_groups - 1;  // first group that reaches the node block
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (g_row[mid] + kTiles64 > k) hi = mid; else lo = mid + 1;
        }
        int last = lo;
        while (last + 1 < n_groups && g_row[last + 1] <= k) ++last;
        const double* from = frag + 64 * (k % kTiles64) + lane;
        double v = 0.0;
#pragma unroll 4
        for (int b = g_block[lo]; b < g_block[last + 1]; ++b) v += from[(int64_t)b * kTiles64 * 64];
        v += __shfl_xor(v, 16, 64);
        v += __shfl_xor(v, 32, 64);
        if (lane < 16) bsum[16 * k + lane] = v;
    }
    __syncthreads();
    double sq = 0.0;
    if (tid < kSumThreads)
        for (int q = tid; q < 16 * n_rows; q += kSumThreads) {
            const double b = bsum[q];
            sq = fma(b, b, sq);
        }
    sq = block_sum(sq, red);
    const int cap = md.mode_cap, L = 3 * cap + 32;
    double* ev = psh;
    double* ct = psh + L;
    double* cs = ct + L;
    series_coefficients<BLOCK>(P.sigma_t, cap, ev, ct, cs);
    __syncthreads();
    if (tid == 0) {
        int m = cap;
        double tail = 0.0;
        for (; m > 1; --m) {
            tail += cs[m];
            if (tail > kModeTail64) break;
        }
        m = min(m, md.max_groups * kModeGroup64);
        ired[0] = m;
        M.groups = (m + kModeGroup64 - 1) / kModeGroup64;
        M.blocks = n_blocks;
        M.nodes = 0;
        M.c0 = cs[0];
        M.sj0 = kNodeW64 * sq;
        md.curves[c] = M;
        cp[c].ipy = kInvSqrt2Pi / P.sigma_y * M.sj0 / ((double)n * (double)n);
    }
    __syncthreads();
    const int keep = ired[0];
    double* coef = md.coef + (int64_t)c * mode_stride(cap);
    for (int m = tid + 1; m <= mode_stride(cap); m += BLOCK)
        coef[m - 1] = m <= keep ? cs[m] : 0.0;
}

template <int BLOCK, int EMAX>
hipError_t launch_prepare64_b(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                              const double* t, const double* y, const ModeDev& md) {
    const int room = sort_room(BLOCK, max_n);
    const int key_bytes = key_bytes_of(room, md.mode_cap);
    const int group_room = mode64_room(max_n);
    const size_t lds = (size_t)key_bytes + 4 * (size_t)(room + 4 * group_room + 2);
    prepare64_kernel<BLOCK, EMAX><<<n_curves, BLOCK, lds, st>>>(cp, t, y, room, key_bytes,
                                                                group_room, md);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_prepare64(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                            const double* t, const double* y, const ModeDev& md) {
    if (n_curves <= 0) return hipSuccess;
    if (!sort_big(n_curves, max_n))
        return launch_prepare64_b<kSortBlock, kSortE>(st, cp, n_curves, max_n, t, y, md);
    return launch_prepare64_b<kSortBlockBig, kSortEBig>(st, cp, n_curves, max_n, t, y, md);
}

hipError_t launch_prepare(hipStream_t st, CurveParams* cp, int n_curves, int max_n,
                          const double* t, const double* y, const double* e, double skew_lambda,
                          double skew_mu, const ModeDev& md) {
    if (n_curves <= 0) return hipSuccess;
    if (!sort_big(n_curves, max_n))
        return launch_prepare_b<kSortBlock, kSortE>(st, cp, n_curves, max_n, t, y, e, skew_lambda,
                                                    skew_mu, md);
    return launch_prepare_b<kSortBlockBig, kSortEBig>(st, cp, n_curves, max_n, t, y, e,
                                                      skew_lambda, skew_mu, md);
}

}  // namespace qmi
