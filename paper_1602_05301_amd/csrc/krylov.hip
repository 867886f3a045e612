// Device building blocks of GMRES on the QBX-FMM matvec (Sec. 8.3): the
// Arnoldi step's Gram-Schmidt products over the stored Krylov vectors, the
// normalisation, and the interpolation of densities to oversampled panels
// (Sec. 3.2, Table 1).  Every sum runs in a fixed order, so results do not
// depend on timing.  These loops stream the Krylov basis from HBM once per
// call: they are bandwidth-bound.
#include <hip/hip_runtime.h>

#include "krylov.hpp"

namespace qbx {

namespace {

__device__ __forceinline__ cd kc_mul(cd a, cd b) { return {fma(a.x, b.x, -a.y * b.y), fma(a.x, b.y, a.y * b.x)}; }
__device__ __forceinline__ cd kc_cmul(cd a, cd b)     // conj(a) b
{
    return {fma(a.x, b.x, a.y * b.y), fma(a.x, b.y, -a.y * b.x)};
}

constexpr int KD_THREADS = 256;
constexpr int KD_COLS = 4;                    // columns per thread
constexpr int KD_CHUNK = KD_THREADS * KD_COLS;
constexpr int KD_ROWS = 8;                    // Krylov vectors per block

__device__ __forceinline__ cd wave_sum(cd a)
{
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        a.x += __shfl_xor(a.x, s, 64);
        a.y += __shfl_xor(a.y, s, 64);
    }
    return a;
}

// partial[r * nchunk + c] = sum over chunk c of conj(V[r][j]) w[j], for the
// KD_ROWS rows of block y.  A lane sums its columns in order for every row
// (all loads independent), each wave its lanes by a fixed butterfly, and the
// block its waves in order: one barrier for all rows, where a block-wide tree
// per row had eight each (71 to 69 us for 200 vectors of
// 107552, 5.0 TB/s, the copy rate).
__global__ void __launch_bounds__(KD_THREADS) k_kdot_partial(long long n, int k, const cd *V, long long ldv,
                                                             const cd *w, cd *partial, int nchunk)
{
    __shared__ cd red[KD_THREADS / 64][KD_ROWS];
    int c = blockIdx.x, r0 = blockIdx.y * KD_ROWS, rows = min(KD_ROWS, k - r0);
    long long j0 = (long long)c * KD_CHUNK + threadIdx.x;
    bool ok[KD_COLS];
    cd wj[KD_COLS];
#pragma unroll
    for (int t = 0; t < KD_COLS; ++t) {
        long long j = j0 + (long long)t * KD_THREADS;
        ok[t] = j < n;
        wj[t] = ok[t] ? w[j] : cd{0.0, 0.0};
    }
#pragma unroll
    for (int rr = 0; rr < KD_ROWS; ++rr) {
        if (rr >= rows) break;                  // uniform across the block
        const cd *vr = V + (long long)(r0 + rr) * ldv + j0;
        cd acc{0.0, 0.0};
#pragma unroll
        for (int t = 0; t < KD_COLS; ++t)
            if (ok[t]) {
                cd p = kc_cmul(vr[t * KD_THREADS], wj[t]);
                acc.x += p.x;
                acc.y += p.y;
            }
        acc = wave_sum(acc);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][rr] = acc;
    }
    __syncthreads();
    if ((int)threadIdx.x < rows) {
        cd sum = red[0][threadIdx.x];
#pragma unroll
        for (int i = 1; i < KD_THREADS / 64; ++i) {
            sum.x += red[i][threadIdx.x].x;
            sum.y += red[i][threadIdx.x].y;
        }
        partial[(long long)(r0 + threadIdx.x) * nchunk + c] = sum;
    }
}

// h[r] = sum over chunks of partial[r][.]: a wave per row, lane l takes chunks
// l, l + 64, ... in order, the lanes by a fixed butterfly.  (One thread per
// row walked the chunks one after the other: 18 us for 105 chunks, now 4.9.)
constexpr int KF_THREADS = 256;

__global__ void __launch_bounds__(KF_THREADS) k_kdot_final(int k, const cd *partial, int nchunk, cd *h)
{
    int r = blockIdx.x * (KF_THREADS / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (r >= k) return;                         // uniform across the wave
    cd acc{0.0, 0.0};
    for (int c = lane; c < nchunk; c += 64) {
        cd p = partial[(long long)r * nchunk + c];
        acc.x += p.x;
        acc.y += p.y;
    }
    acc = wave_sum(acc);
    if (lane == 0) h[r] = acc;
}

constexpr int KU_THREADS = 256;
constexpr int KU_HTILE = 256;                 // coefficients staged in LDS at a time

// w[j] -= sum_i h[i] V[i][j], i in order.
__global__ void __launch_bounds__(KU_THREADS) k_kupdate(long long n, int k, const cd *V, long long ldv,
                                                        const cd *h, cd *w)
{
    __shared__ cd hs[KU_HTILE];
    long long j = (long long)blockIdx.x * KU_THREADS + threadIdx.x;
    cd acc{0.0, 0.0};
    for (int i0 = 0; i0 < k; i0 += KU_HTILE) {
        int m = min(KU_HTILE, k - i0);
        __syncthreads();
        if ((int)threadIdx.x < m) hs[threadIdx.x] = h[i0 + threadIdx.x];
        __syncthreads();
        if (j < n) {
            const cd *v = V + (long long)i0 * ldv + j;
            for (int i = 0; i < m; ++i) {
                cd p = kc_mul(hs[i], v[(long long)i * ldv]);
                acc.x += p.x;
                acc.y += p.y;
            }
        }
    }
    if (j < n) {
        cd x = w[j];
        w[j] = cd{x.x - acc.x, x.y - acc.y};
    }
}

// v[j] = w[j] / sqrt(Re nrm2[0]) (0 when the norm is 0).
__global__ void k_knormalize(long long n, const cd *w, const cd *nrm2, cd *v)
{
    long long j = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    double s = nrm2[0].x;
    double inv = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    cd x = w[j];
    v[j] = cd{inv * x.x, inv * x.y};
}

// Panel p's density at its q nodes, x[p q + b], carried to its qs nodes:
// yd[p qs + a] = sum_b L[a q + b] x[p q + b]; ys = alpha yd.
// A block takes KP_PANELS panels: their densities and a row-padded copy of L
// are staged in LDS, so that the inner sums read no global memory (each
// thread reading its row of L and the panel through the caches: 20 us for 6722
// panels, q = 16 to 64; now 8).
constexpr int KP_THREADS = 256;
constexpr int KP_PANELS = 8;

__global__ void __launch_bounds__(KP_THREADS) k_upsample(long long n_panels, int q, int qs, const double *L, cd alpha,
                                                         const cd *x, cd *ys, cd *yd)
{
    extern __shared__ double kp_lds[];
    cd *xs = reinterpret_cast<cd *>(kp_lds);            // [KP_PANELS][q]
    double *Ls = kp_lds + 2 * KP_PANELS * q;            // [qs][q + 1]
    long long p0 = (long long)blockIdx.x * KP_PANELS;
    int np = (int)min((long long)KP_PANELS, n_panels - p0);
    for (int i = threadIdx.x; i < np * q; i += KP_THREADS) xs[i] = x[p0 * q + i];
    for (int i = threadIdx.x; i < qs * q; i += KP_THREADS) Ls[i / q * (q + 1) + i % q] = L[i];
    __syncthreads();
    for (int t = threadIdx.x; t < np * qs; t += KP_THREADS) {
        int p = t / qs, a = t - p * qs;
        const cd *xp = xs + p * q;
        const double *La = Ls + a * (q + 1);
        cd acc{0.0, 0.0};
        for (int b = 0; b < q; ++b) {
            acc.x = fma(La[b], xp[b].x, acc.x);
            acc.y = fma(La[b], xp[b].y, acc.y);
        }
        if (yd) yd[p0 * qs + t] = acc;
        if (ys) ys[p0 * qs + t] = kc_mul(alpha, acc);
    }
}

// The same for panels too long for LDS, or too short for its staging: one thread per fine node.
__global__ void k_upsample_long(long long n_panels, int q, int qs, const double *L, cd alpha, const cd *x, cd *ys,
                                cd *yd)
{
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n_panels * qs) return;
    long long p = t / qs;
    int a = (int)(t - p * qs);
    const cd *xp = x + p * q;
    const double *La = L + (long long)a * q;
    cd acc{0.0, 0.0};
    for (int b = 0; b < q; ++b) {
        acc.x = fma(La[b], xp[b].x, acc.x);
        acc.y = fma(La[b], xp[b].y, acc.y);
    }
    if (yd) yd[t] = acc;
    if (ys) ys[t] = kc_mul(alpha, acc);
}

}  // namespace

int krylov_dot_chunks(long long n) { return (int)((n + KD_CHUNK - 1) / KD_CHUNK); }

hipError_t launch_krylov_dot(long long n, int k, const cd *V, long long ldv, const cd *w, cd *partial, cd *h,
                             hipStream_t s)
{
    if (k <= 0) return hipSuccess;
    int nchunk = krylov_dot_chunks(n);
    if (nchunk > 0) {
        dim3 grid(nchunk, (k + KD_ROWS - 1) / KD_ROWS);
        k_kdot_partial<<<grid, KD_THREADS, 0, s>>>(n, k, V, ldv, w, partial, nchunk);
    }
    k_kdot_final<<<(k + KF_THREADS / 64 - 1) / (KF_THREADS / 64), KF_THREADS, 0, s>>>(k, partial, nchunk, h);
    return hipGetLastError();
}

hipError_t launch_krylov_update(long long n, int k, const cd *V, long long ldv, const cd *h, cd *w, hipStream_t s)
{
    if (n <= 0 || k <= 0) return hipSuccess;
    k_kupdate<<<(unsigned)((n + KU_THREADS - 1) / KU_THREADS), KU_THREADS, 0, s>>>(n, k, V, ldv, h, w);
    return hipGetLastError();
}

hipError_t launch_krylov_normalize(long long n, const cd *w, const cd *nrm2, cd *v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    k_knormalize<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(n, w, nrm2, v);
    return hipGetLastError();
}

hipError_t launch_upsample(long long n_panels, int q, int qs, const double *L, cd alpha, const cd *x, cd *ys,
                           cd *yd, hipStream_t s)
{
    long long t = n_panels * qs;
    if (t <= 0) return hipSuccess;
    // LDS of the staged form; sizes past 64 KiB (q and qs about 80) read through
    // the caches, and so do panels and rows so short that staging a block's takes
    // longer than its few sums: 200000 panels, 4 to 4 nodes 9.6 us a call and 14.5
    // staged, 1 to 4 8.2 and 13.3, 16 to 1 22.5 and 23.5, 64 to 2 68 and 82; but 8
    // to 8 29 and 18, 16 to 4 39 and 23, 64 to 4 123 and 77.
    size_t lds = sizeof(double) * (2 * (size_t)KP_PANELS * q + (size_t)qs * (q + 1));
    if (lds <= 64 * 1024 && q >= 8 && qs >= 4)
        k_upsample<<<(unsigned)((n_panels + KP_PANELS - 1) / KP_PANELS), KP_THREADS, lds, s>>>(n_panels, q, qs, L, alpha, x, ys, yd);
    else
        k_upsample_long<<<(unsigned)((t + 255) / 256), 256, 0, s>>>(n_panels, q, qs, L, alpha, x, ys, yd);
    return hipGetLastError();
}

}  // namespace qbx
