// Block-wide sorts for the per-curve preparation kernels: a bitonic network with the keys in
// registers.
//
// Thread t holds elements t E ... t E + E - 1, so that of the network's log^2 steps those of
// stride below E stay inside a thread, those below 64 E are lane exchanges within a wave, and only
// the longest strides go through LDS with barriers (for 1024 keys and 256 threads 3 of 55 steps).
// Measured with the kernels around it: 8192 keys twice 640 -> 100 us, the time and magnitude orders
// of 768 survey curves 470 -> 89 us, against one key pair per thread and step in LDS.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qmi {

// Exchange of one element with a partner's: keeps the smaller (first) or the larger by (key, idx),
// a total order, so that the result is the stable order of the keys.
template <bool IDX>
__device__ __forceinline__ void sort_keep(double& k, int32_t& v, double ok, int32_t ov,
                                          bool smaller) {
    if constexpr (IDX) {
        const bool gt = (k > ok) || (k == ok && v > ov);
        if (gt == smaller) {
            k = ok;
            v = ov;
        }
    } else {
        k = smaller ? fmin(k, ok) : fmax(k, ok);
    }
}

template <int BLOCK, int E, bool IDX>
__device__ __forceinline__ void sort_regs(double (&k)[E], int32_t (&v)[E], int m, double* lk,
                                          int32_t* lv) {
    const int t = threadIdx.x, base = t * E;
    for (int kk = 2; kk <= m; kk <<= 1) {
        int j = kk >> 1;
        for (; j >= 64 * E; j >>= 1) {
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) {
                lk[base + e] = k[e];
                if (IDX) lv[base + e] = v[e];
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int i = base + e;
                sort_keep<IDX>(k[e], v[e], lk[i ^ j], IDX ? lv[i ^ j] : 0,
                               ((i & kk) == 0) == ((i & j) == 0));
            }
        }
        for (; j >= E && j > 0; j >>= 1) {
            const int mask = j / E;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int i = base + e;
                const double ok = __shfl_xor(k[e], mask, 64);
                const int32_t ov = IDX ? __shfl_xor(v[e], mask, 64) : 0;
                sort_keep<IDX>(k[e], v[e], ok, ov, ((i & kk) == 0) == ((i & j) == 0));
            }
        }
#pragma unroll
        for (int s = E / 2; s > 0; s >>= 1) {
            if (s > j) continue;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int l = e ^ s;
                if (l < e) continue;
                const bool up = ((base + e) & kk) == 0;
                const bool gt = IDX ? (k[e] > k[l]) || (k[e] == k[l] && v[e] > v[l])
                                    : k[e] > k[l];
                if (gt == up) {
                    const double a = k[e];
                    k[e] = k[l];
                    k[l] = a;
                    const int32_t b = v[e];
                    v[e] = v[l];
                    v[l] = b;
                }
            }
        }
    }
}

template <int BLOCK, int E, bool IDX>
__device__ void sort_block_e(double* lk, int32_t* lv, int n, int m) {
    double k[E];
    int32_t v[E];
    const int base = threadIdx.x * E;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = base + e;
        k[e] = i < n ? lk[i] : INFINITY;
        v[e] = IDX ? (i < n ? lv[i] : 0x7fffffff) : 0;
    }
    sort_regs<BLOCK, E, IDX>(k, v, m, lk, lv);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int i = base + e;
        if (i < n) {
            lk[i] = k[e];
            if (IDX) lv[i] = v[e];
        }
    }
    __syncthreads();
}

// Sorts lk[0..n) (LDS, no NaN) in place, with IDX together with lv[0..n) by (key, value): the
// stable order of the keys where lv starts as 0, 1, ....  lk and lv have the entries that sort_room
// says; n <= BLOCK * EMAX.  Every thread of the block calls it.
template <int BLOCK, int EMAX, bool IDX>
__device__ void sort_block(double* lk, int32_t* lv, int n) {
    int m = 1;
    while (m < n) m <<= 1;
    __syncthreads();
    if (n <= BLOCK) {
        sort_block_e<BLOCK, 1, IDX>(lk, lv, n, m);
    } else if (EMAX >= 2 && n <= 2 * BLOCK) {
        sort_block_e<BLOCK, EMAX >= 2 ? 2 : 1, IDX>(lk, lv, n, m);
    } else if (EMAX >= 4 && n <= 4 * BLOCK) {
        sort_block_e<BLOCK, EMAX >= 4 ? 4 : 1, IDX>(lk, lv, n, m);
    } else if (EMAX >= 8) {
        sort_block_e<BLOCK, EMAX >= 8 ? 8 : 1, IDX>(lk, lv, n, m);
    }
}

// Threads of a preparation block, and elements per thread: the small one where the batch fills the
// chip, the big one for long curves and for a few curves, whose blocks have the chip to themselves.
constexpr int kSortBlock = 256, kSortE = 4;         // up to 1024
constexpr int kSortBlockBig = 1024, kSortEBig = 8;  // up to 8192
inline bool sort_big(int n_curves, int max_n) {
    return max_n > kSortBlock * kSortE || n_curves < 128;
}

// LDS entries that sort_block needs for n keys: the block's padded size.
inline int sort_room(int block, int max_n) {
    int m = block;
    while (m < max_n) m <<= 1;
    return m;
}

}  // namespace qmi
