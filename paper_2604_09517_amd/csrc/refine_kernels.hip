// Kernels of the FP64 iterative refinement (Sec. III-A.2: residuals and
// corrections in FP64; Sec. II-B: refinement based on GMRES) and of its
// preconditioner M = U^-1 L^-1 P applied in FP32 to the low-precision factors.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "asource.h"
#include "common.h"
#include "lp_common.h"
#include "refine_kernels.h"

namespace {

using namespace mxlu;

__device__ __forceinline__ void atomic_max_abs(unsigned long long *dst, double v) {
    atomicMax(dst, (unsigned long long)__double_as_longlong(fabs(v)));
}

__device__ __forceinline__ double bits_to_double(unsigned long long b) {
    return __longlong_as_double((long long)b);
}

// ---------------------------------------------------------------- GEMV
// partial[s][i] = sum over columns j of split s of A[i, j] x[j] (ascending
// j); with asum, the |A[i, j]| row sums of the split go to asum_part.  The
// seeded form regenerates each A[i, j] from its counter (consecutive j of a
// row step the counter by G n), so the matrix is never read from memory; its
// terms are taken in the same order, so both forms give the same bits.
template <bool SEEDED>
__global__ __launch_bounds__(256) void gemv_n_partial_kernel(int64_t n, ASource src,
                                                             const double *__restrict__ x,
                                                             int64_t cps, double *__restrict__ part,
                                                             double *__restrict__ asum_part) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t j0 = (int64_t)blockIdx.y * cps;
    const int64_t j1 = (j0 + cps < n) ? j0 + cps : n;
    if (i >= n) return;
    double acc = 0.0, as = 0.0;
    if constexpr (!SEEDED) {
        const double *__restrict__ A = src.A;
        const int64_t lda = src.lda;
        int64_t j = j0;
        // sixteen columns of 8-byte loads in flight
        for (; j + 16 <= j1; j += 16) {
            double a[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) a[q] = MXLU_AT(A, i, j + q, lda);
#pragma unroll
            for (int q = 0; q < 16; ++q) acc = fma(a[q], x[j + q], acc);
            if (asum_part)
#pragma unroll
                for (int q = 0; q < 16; q += 4)
                    as += fabs(a[q]) + fabs(a[q + 1]) + fabs(a[q + 2]) + fabs(a[q + 3]);
        }
        for (; j + 4 <= j1; j += 4) {
            const double a0 = MXLU_AT(A, i, j, lda), a1 = MXLU_AT(A, i, j + 1, lda);
            const double a2 = MXLU_AT(A, i, j + 2, lda), a3 = MXLU_AT(A, i, j + 3, lda);
            acc = fma(a0, x[j], acc);
            acc = fma(a1, x[j + 1], acc);
            acc = fma(a2, x[j + 2], acc);
            acc = fma(a3, x[j + 3], acc);
            if (asum_part) as += fabs(a0) + fabs(a1) + fabs(a2) + fabs(a3);
        }
        for (; j < j1; ++j) {
            const double a = MXLU_AT(A, i, j, lda);
            acc = fma(a, x[j], acc);
            if (asum_part) as += fabs(a);
        }
    } else {
        // |a| sums of generator values are exact in any order (multiples of
        // 2^-32 below 2^21 in size), so the grouping above does not matter
        const uint64_t step = kGenGolden * (uint64_t)n;
        uint64_t z = src.key + kGenGolden * ((uint64_t)j0 * (uint64_t)n + (uint64_t)i + 1ull);
        for (int64_t j = j0; j < j1; ++j, z += step) {
            const double a = (src.diag && j == i) ? src.diag[i] : gen_value(z);
            acc = fma(a, x[j], acc);
            if (asum_part) as += fabs(a);
        }
    }
    part[(size_t)blockIdx.y * n + i] = acc;
    if (asum_part) asum_part[(size_t)blockIdx.y * n + i] = as;
}

// The same for a stored A with even lda and 16-byte alignment: two adjacent
// rows per thread (one 16-byte load per column covers both), each row's
// terms still in ascending j, eight columns per iteration in flight.
__global__ __launch_bounds__(256) void gemv_n_partial2_kernel(int64_t n, const double *__restrict__ A,
                                                              int64_t lda,
                                                              const double *__restrict__ x,
                                                              int64_t cps, double *__restrict__ part,
                                                              double *__restrict__ asum_part) {
    const int64_t i = 2 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
    const int64_t j0 = (int64_t)blockIdx.y * cps;
    const int64_t j1 = (j0 + cps < n) ? j0 + cps : n;
    if (i >= n) return;
    double acc0 = 0.0, acc1 = 0.0, as0 = 0.0, as1 = 0.0;
    if (i + 1 < n) {
        int64_t j = j0;
        for (; j + 8 <= j1; j += 8) {
            double2 a[8];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                a[q] = *reinterpret_cast<const double2 *>(&A[(size_t)i + (size_t)(j + q) * lda]);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const double xq = x[j + q];
                acc0 = fma(a[q].x, xq, acc0);
                acc1 = fma(a[q].y, xq, acc1);
            }
            if (asum_part) {
                // the same grouping as the one-row form: four terms, then added
#pragma unroll
                for (int h = 0; h < 8; h += 4) {
                    as0 += fabs(a[h].x) + fabs(a[h + 1].x) + fabs(a[h + 2].x) + fabs(a[h + 3].x);
                    as1 += fabs(a[h].y) + fabs(a[h + 1].y) + fabs(a[h + 2].y) + fabs(a[h + 3].y);
                }
            }
        }
        for (; j + 4 <= j1; j += 4) {
            double2 a[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a[q] = *reinterpret_cast<const double2 *>(&A[(size_t)i + (size_t)(j + q) * lda]);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double xq = x[j + q];
                acc0 = fma(a[q].x, xq, acc0);
                acc1 = fma(a[q].y, xq, acc1);
            }
            if (asum_part) {
                as0 += fabs(a[0].x) + fabs(a[1].x) + fabs(a[2].x) + fabs(a[3].x);
                as1 += fabs(a[0].y) + fabs(a[1].y) + fabs(a[2].y) + fabs(a[3].y);
            }
        }
        for (; j < j1; ++j) {
            const double2 a = *reinterpret_cast<const double2 *>(&A[(size_t)i + (size_t)j * lda]);
            acc0 = fma(a.x, x[j], acc0);
            acc1 = fma(a.y, x[j], acc1);
            if (asum_part) {
                as0 += fabs(a.x);
                as1 += fabs(a.y);
            }
        }
        part[(size_t)blockIdx.y * n + i + 1] = acc1;
        if (asum_part) asum_part[(size_t)blockIdx.y * n + i + 1] = as1;
    } else {   // the last row of an odd n
        int64_t j = j0;
        for (; j + 4 <= j1; j += 4) {
            const double a0 = MXLU_AT(A, i, j, lda), a1 = MXLU_AT(A, i, j + 1, lda);
            const double a2 = MXLU_AT(A, i, j + 2, lda), a3 = MXLU_AT(A, i, j + 3, lda);
            acc0 = fma(a0, x[j], acc0);
            acc0 = fma(a1, x[j + 1], acc0);
            acc0 = fma(a2, x[j + 2], acc0);
            acc0 = fma(a3, x[j + 3], acc0);
            if (asum_part) as0 += fabs(a0) + fabs(a1) + fabs(a2) + fabs(a3);
        }
        for (; j < j1; ++j) {
            const double a = MXLU_AT(A, i, j, lda);
            acc0 = fma(a, x[j], acc0);
            if (asum_part) as0 += fabs(a);
        }
    }
    part[(size_t)blockIdx.y * n + i] = acc0;
    if (asum_part) asum_part[(size_t)blockIdx.y * n + i] = as0;
}

// Transposed: part[s][i] = sum over rows j of split s of A[j, i] x[j]; one
// wave per i (column i of A is contiguous).
template <bool SEEDED>
__global__ __launch_bounds__(256) void gemv_t_partial_kernel(int64_t n, ASource src,
                                                             const double *__restrict__ x,
                                                             int64_t cps, double *__restrict__ part,
                                                             double *__restrict__ asum_part) {
    const int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int64_t j0 = (int64_t)blockIdx.y * cps;
    const int64_t j1 = (j0 + cps < n) ? j0 + cps : n;
    if (i >= n) return;
    double acc = 0.0, as = 0.0;
    if constexpr (!SEEDED) {
        for (int64_t j = j0 + lane; j < j1; j += 64) {
            const double a = MXLU_AT(src.A, j, i, src.lda);
            acc = fma(a, x[j], acc);
            as += fabs(a);
        }
    } else {
        uint64_t z = src.key + kGenGolden * ((uint64_t)i * (uint64_t)n + (uint64_t)(j0 + lane) + 1ull);
        for (int64_t j = j0 + lane; j < j1; j += 64, z += 64ull * kGenGolden) {
            const double a = (src.diag && j == i) ? src.diag[i] : gen_value(z);
            acc = fma(a, x[j], acc);
            as += fabs(a);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        acc += __shfl_xor(acc, off);
        as += __shfl_xor(as, off);
    }
    if (lane == 0) {
        part[(size_t)blockIdx.y * n + i] = acc;
        if (asum_part) asum_part[(size_t)blockIdx.y * n + i] = as;
    }
}

// y[i] = (b ? b[i] - sum_s part : sum_s part); maxima of |y| and of the
// |A| row sums go to stats[0] and stats[1] (bit patterns), |x| to stats[2];
// that of |y| to ymax as well.
__global__ void gemv_finish_kernel(int64_t n, int nsplit, const double *__restrict__ part,
                                   const double *__restrict__ asum_part,
                                   const double *__restrict__ b, double *__restrict__ y,
                                   const double *__restrict__ xv,
                                   unsigned long long *__restrict__ stats,
                                   unsigned long long *__restrict__ ymax) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double m_y = 0.0, m_a = 0.0, m_x = 0.0;
    if (i < n) {
        // the partial sums in order, sixteen loads in flight
        auto total = [&](const double *__restrict__ p) {
            double s = 0.0;
            int k = 0;
            for (; k + 16 <= nsplit; k += 16) {
                double v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = p[(size_t)(k + q) * n + i];
#pragma unroll
                for (int q = 0; q < 16; ++q) s += v[q];
            }
            for (; k < nsplit; ++k) s += p[(size_t)k * n + i];
            return s;
        };
        const double s = total(part);
        const double v = b ? b[i] - s : s;
        y[i] = v;
        m_y = fabs(v);
        if (asum_part) {
            m_a = total(asum_part);
        }
        if (xv) m_x = fabs(xv[i]);
    }
    if (stats || ymax) {
        for (int off = 32; off > 0; off >>= 1) {
            m_y = fmax(m_y, __shfl_xor(m_y, off));
            m_a = fmax(m_a, __shfl_xor(m_a, off));
            m_x = fmax(m_x, __shfl_xor(m_x, off));
        }
        if ((threadIdx.x & 63) == 0) {
            if (stats) {
                atomic_max_abs(&stats[0], m_y);
                if (asum_part) atomic_max_abs(&stats[1], m_a);
                if (xv) atomic_max_abs(&stats[2], m_x);
            }
            if (ymax) atomic_max_abs(ymax, fmax(0.0, m_y));   // (a NaN alone counts as none)
        }
    }
}

// ---------------------------------------------------------------- BLAS-1/2
// part[c][chunk] = sum over the chunk of V[:, c] * z
__global__ __launch_bounds__(256) void dots_partial_kernel(int64_t n, const double *__restrict__ V,
                                                           int64_t ldv,
                                                           const double *__restrict__ z,
                                                           int64_t chunk, double *__restrict__ part,
                                                           int nchunks) {
    __shared__ double red[256];
    const int c = blockIdx.y;
    const int64_t i0 = (int64_t)blockIdx.x * chunk;
    const int64_t i1 = (i0 + chunk < n) ? i0 + chunk : n;
    double acc = 0.0;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += 256) acc = fma(MXLU_AT(V, i, c, ldv), z[i], acc);
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)c * nchunks + blockIdx.x] = red[0];
}

__global__ void dots_reduce_kernel(int ncols, int nchunks, const double *__restrict__ part,
                                   double *__restrict__ out) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncols) return;
    double s = 0.0;
    for (int k = 0; k < nchunks; ++k) s += part[(size_t)c * nchunks + k];
    out[c] = s;
}

// z[i] += sign * sum_c V[i, c] h[c]   (c ascending)
__global__ void gemv_small_kernel(int64_t n, int k, const double *__restrict__ V, int64_t ldv,
                                  const double *__restrict__ h, double sign,
                                  double *__restrict__ z) {
    __shared__ double hs[256];
    if ((int)threadIdx.x < k) hs[threadIdx.x] = h[threadIdx.x];
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double acc = z[i];
    for (int c = 0; c < k; ++c) acc = fma(sign * MXLU_AT(V, i, c, ldv), hs[c], acc);
    z[i] = acc;
}

// One step of the orthogonalization by a single workgroup, n < 2048 (one chunk
// of the sums above): classical Gram-Schmidt twice against V's k columns, then
// the norm and the next column: h1 = V^T z, z -= V h1, h2 = V^T z, z -= V h2,
// *hn = z^T z, vnext = z / sqrt(*hn); with k = 0 only the last two.  The same
// sums in the same order as dots_partial_kernel (256 strided partial sums and
// its tree, four of them per lane) and gemv_small_kernel: eight launches in
// one.  At n = 1000 those took 3 to 5 us each and about as much between them.
constexpr int kArnoldiMaxN = 2048;

__global__ __launch_bounds__(1024) void arnoldi_small_kernel(int n, int k, const double *__restrict__ V,
                                                             int64_t ldv, const double *__restrict__ z,
                                                             double *__restrict__ h1,
                                                             double *__restrict__ h2,
                                                             double *__restrict__ hn,
                                                             double *__restrict__ vnext) {
    __shared__ double zs[kArnoldiMaxN];
    __shared__ double hs[256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int i = tid; i < n; i += 1024) zs[i] = z[i];
    __syncthreads();
    auto dot = [&](const double *x) {   // x^T z in lane 0; every lane of the wave takes part
        double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
        for (int i0 = 0; i0 < n; i0 += 256)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + 64 * q + lane;
                if (i < n) a[q] = fma(x[i], zs[i], a[q]);
            }
        double s = (a[0] + a[2]) + (a[1] + a[3]);
        for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off);
        return s;
    };
    for (int pass = 0; pass < (k > 0 ? 2 : 0); ++pass) {
        for (int c = wave; c < k; c += 16) {
            const double s = dot(V + (size_t)c * ldv);
            if (lane == 0) {
                hs[c] = s;
                (pass ? h2 : h1)[c] = s;
            }
        }
        __syncthreads();
        for (int i = tid; i < n; i += 1024) {
            double acc = zs[i];
#pragma unroll 8
            for (int c = 0; c < k; ++c) acc = fma(-V[(size_t)i + (size_t)c * ldv], hs[c], acc);
            zs[i] = acc;
        }
        __syncthreads();
    }
    if (wave == 0) {
        const double s = dot(zs);
        if (lane == 0) {
            hs[0] = s;
            *hn = s;
        }
    }
    __syncthreads();
    const double alpha = 1.0 / sqrt(hs[0]);   // (not finite: the caller stops here)
    for (int i = tid; i < n; i += 1024) vnext[i] = zs[i] * alpha;
}

__global__ void scale_copy_kernel(int64_t n, const double *__restrict__ z, double alpha,
                                  double *__restrict__ v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] = z[i] * alpha;
}

__global__ void axpy_kernel(int64_t n, const double *__restrict__ z, double *__restrict__ x) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = x[i] + z[i];
}

__global__ void absmax_kernel(int64_t n, const double *__restrict__ v,
                              unsigned long long *__restrict__ out) {
    double m = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        m = fmax(m, fabs(v[i]));
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) atomic_max_abs(out, m);
}

// ---------------------------------------------------------------- precond
// (FP32 factors; those of 16 bits do both steps in their solves)
// v32[i] = fp32( r[src(i)] / s ), s = *smax (bits) or 1 when zero;
// src(i) = perm[i] when perm is given (apply P), else i.
__global__ void precond_in_kernel(int64_t n, const double *__restrict__ r,
                                  const int32_t *__restrict__ perm,
                                  const unsigned long long *__restrict__ smax,
                                  unsigned long long *smax_next, float *__restrict__ v32) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *smax_next = 0;
    if (i >= n) return;
    const double s = bits_to_double(*smax);
    const double ri = r[perm ? perm[i] : i];
    v32[i] = s > 0.0 ? (float)(ri / s) : 0.0f;
}

// d[i] = s * fp64(v32[i])
__global__ void precond_out_kernel(int64_t n, const float *__restrict__ v32,
                                   const unsigned long long *__restrict__ smax,
                                   double *__restrict__ d) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double s = bits_to_double(*smax);
    d[i] = s > 0.0 ? s * (double)v32[i] : 0.0;
}

unsigned g1(int64_t n) { return (unsigned)((n + 255) / 256); }

// FP32-storage preconditioner: the factors are FP32 numbers, solved block by
// block (kTrsv32Bs rows) in solve order with two launches per block: one
// workgroup solves the diagonal block (its rows staged in LDS, thread = row,
// each finished value broadcast through LDS), then a grid applies the block's
// solution to the rows still to be solved (thread = row, the block's values in
// LDS, the factor streamed column by column).  Every element takes its terms in
// the order of the column-oriented substitution: ascending k for L, descending
// k for U (then the division by the diagonal), one fused multiply-add each.
constexpr int kTrsv32Bs = 128;

template <bool LOWER>
__global__ __launch_bounds__(kTrsv32Bs) void trsv_f32_diag_kernel(const float *__restrict__ F,
                                                                  int64_t ldf, int64_t b0,
                                                                  int rows, float *__restrict__ v) {
    __shared__ float Ld[kTrsv32Bs][kTrsv32Bs + 1];
    __shared__ float xk[2];
    const int t = threadIdx.x;
    for (int c = 0; c < rows; ++c)
        if (t < rows) Ld[t][c] = F[(size_t)(b0 + t) + (size_t)(b0 + c) * ldf];
    __syncthreads();
    float x = t < rows ? v[b0 + t] : 0.0f;
    // slot k & 1 is rewritten at step k + 2, after every thread has passed the
    // barrier of step k + 1 and so has read it at step k
    if constexpr (LOWER) {
        for (int k = 0; k < rows; ++k) {
            if (t == k) xk[k & 1] = x;
            __syncthreads();
            const float xv = xk[k & 1];
            if (t > k && t < rows) x = fmaf(-Ld[t][k], xv, x);
        }
    } else {
        for (int k = rows - 1; k >= 0; --k) {
            if (t == k) {
                x = x / Ld[k][k];
                xk[k & 1] = x;
            }
            __syncthreads();
            const float xv = xk[k & 1];
            if (t < k) x = fmaf(-Ld[t][k], xv, x);
        }
    }
    if (t < rows) v[b0 + t] = x;
}

// rows i >= b0 + rows (LOWER) or i < b0 (upper): v_i -= sum over the block
template <bool LOWER>
__global__ __launch_bounds__(256) void trsv_f32_apply_kernel(int64_t n, const float *__restrict__ F,
                                                             int64_t ldf, int64_t b0, int rows,
                                                             float *__restrict__ v) {
    __shared__ float xb[kTrsv32Bs];
    const int t = threadIdx.x;
    if (t < rows) xb[t] = v[b0 + t];
    __syncthreads();
    const int64_t i = (LOWER ? b0 + rows : 0) + (int64_t)blockIdx.x * 256 + t;
    if (i >= (LOWER ? n : b0)) return;
    float x = v[i];
    if constexpr (LOWER) {
#pragma unroll 16
        for (int k = 0; k < rows; ++k) x = fmaf(-F[(size_t)i + (size_t)(b0 + k) * ldf], xb[k], x);
    } else {
#pragma unroll 16
        for (int k = rows - 1; k >= 0; --k)
            x = fmaf(-F[(size_t)i + (size_t)(b0 + k) * ldf], xb[k], x);
    }
    v[i] = x;
}

}  // namespace

namespace mxlu {

int gemv_f64(int trans, int64_t n, const ASource &src, const double *x,
             const double *b, double *y, double *part, double *asum_part, int nsplit,
             unsigned long long *stats, unsigned long long *ymax, hipStream_t s) {
    if (n <= 0) return 0;
    const int64_t cps = (n + nsplit - 1) / nsplit;
    const dim3 gn(g1(n), (unsigned)nsplit), gt((unsigned)((n + 3) / 4), (unsigned)nsplit);
    if (trans == 0 && !src.seeded() && src.lda % 2 == 0 && (uintptr_t)src.A % 16 == 0)
        hipLaunchKernelGGL(gemv_n_partial2_kernel, dim3((unsigned)((n + 511) / 512), (unsigned)nsplit),
                           dim3(256), 0, s, n, src.A, src.lda, x, cps, part, asum_part);
    else if (trans == 0 && !src.seeded())
        hipLaunchKernelGGL(gemv_n_partial_kernel<false>, gn, dim3(256), 0, s, n, src, x, cps, part,
                           asum_part);
    else if (trans == 0)
        hipLaunchKernelGGL(gemv_n_partial_kernel<true>, gn, dim3(256), 0, s, n, src, x, cps, part,
                           asum_part);
    else if (!src.seeded())
        hipLaunchKernelGGL(gemv_t_partial_kernel<false>, gt, dim3(256), 0, s, n, src, x, cps, part,
                           asum_part);
    else
        hipLaunchKernelGGL(gemv_t_partial_kernel<true>, gt, dim3(256), 0, s, n, src, x, cps, part,
                           asum_part);
    MXLU_LAUNCH_CHECK();
    hipLaunchKernelGGL(gemv_finish_kernel, dim3(g1(n)), dim3(256), 0, s, n, nsplit, part,
                       asum_part, b, y, x, stats, ymax);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int dots_f64(int64_t n, int ncols, const double *V, int64_t ldv, const double *z, double *part,
             int nchunks, double *out, hipStream_t s) {
    if (ncols <= 0) return 0;
    const int64_t chunk = (n + nchunks - 1) / nchunks;
    hipLaunchKernelGGL(dots_partial_kernel, dim3((unsigned)nchunks, (unsigned)ncols), dim3(256), 0,
                       s, n, V, ldv, z, chunk, part, nchunks);
    MXLU_LAUNCH_CHECK();
    hipLaunchKernelGGL(dots_reduce_kernel, dim3((unsigned)((ncols + 63) / 64)), dim3(64), 0, s,
                       ncols, nchunks, part, out);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int gemv_small_f64(int64_t n, int k, const double *V, int64_t ldv, const double *h, double sign,
                   double *z, hipStream_t s) {
    if (n <= 0 || k <= 0) return 0;
    if (k > 256) {
        set_error_msg("gemv_small_f64: more than 256 columns");
        return MXLU_E_NOMEM;
    }
    hipLaunchKernelGGL(gemv_small_kernel, dim3(g1(n)), dim3(256), 0, s, n, k, V, ldv, h, sign, z);
    MXLU_LAUNCH_CHECK();
    return 0;
}

bool arnoldi_small_ok(int64_t n, int nchunks, int k) {
    return nchunks == 1 && n < kArnoldiMaxN && k <= 256;
}

int arnoldi_small_f64(int64_t n, int k, const double *V, int64_t ldv, const double *z, double *h1,
                      double *h2, double *hn, double *vnext, hipStream_t s) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(arnoldi_small_kernel, dim3(1), dim3(1024), 0, s, (int)n, k, V, ldv, z, h1, h2,
                       hn, vnext);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int scale_copy_f64(int64_t n, const double *z, double alpha, double *v, hipStream_t s) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(scale_copy_kernel, dim3(g1(n)), dim3(256), 0, s, n, z, alpha, v);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int axpy_f64(int64_t n, const double *z, double *x, hipStream_t s) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(axpy_kernel, dim3(g1(n)), dim3(256), 0, s, n, z, x);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int absmax_f64(int64_t n, const double *v, unsigned long long *out, hipStream_t s) {
    if (n <= 0) return 0;
    const unsigned grid = (unsigned)((n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024);
    hipLaunchKernelGGL(absmax_kernel, dim3(grid), dim3(256), 0, s, n, v, out);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int lp_precond_apply_f32(int64_t n, const float *F, int64_t ldf, const int32_t *perm,
                         const double *r, double *d, float *v32, const unsigned long long *smax,
                         unsigned long long *smax_next, hipStream_t s) {
    if (n <= 0) return 0;
    hipLaunchKernelGGL(precond_in_kernel, dim3(g1(n)), dim3(256), 0, s, n, r, perm, smax, smax_next,
                       v32);
    MXLU_LAUNCH_CHECK();
    for (int64_t b0 = 0; b0 < n; b0 += kTrsv32Bs) {   // L, forward
        const int rows = (int)std::min<int64_t>(kTrsv32Bs, n - b0);
        hipLaunchKernelGGL(trsv_f32_diag_kernel<true>, dim3(1), dim3(kTrsv32Bs), 0, s, F, ldf, b0,
                           rows, v32);
        MXLU_LAUNCH_CHECK();
        const int64_t below = n - b0 - rows;
        if (below > 0) {
            hipLaunchKernelGGL(trsv_f32_apply_kernel<true>, dim3((unsigned)((below + 255) / 256)),
                               dim3(256), 0, s, n, F, ldf, b0, rows, v32);
            MXLU_LAUNCH_CHECK();
        }
    }
    for (int64_t b0 = (n - 1) / kTrsv32Bs * kTrsv32Bs; b0 >= 0; b0 -= kTrsv32Bs) {   // U, backward
        const int rows = (int)std::min<int64_t>(kTrsv32Bs, n - b0);
        hipLaunchKernelGGL(trsv_f32_diag_kernel<false>, dim3(1), dim3(kTrsv32Bs), 0, s, F, ldf, b0,
                           rows, v32);
        MXLU_LAUNCH_CHECK();
        if (b0 > 0) {
            hipLaunchKernelGGL(trsv_f32_apply_kernel<false>, dim3((unsigned)((b0 + 255) / 256)),
                               dim3(256), 0, s, n, F, ldf, b0, rows, v32);
            MXLU_LAUNCH_CHECK();
        }
    }
    hipLaunchKernelGGL(precond_out_kernel, dim3(g1(n)), dim3(256), 0, s, n, v32, smax,
                       d);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace mxlu
