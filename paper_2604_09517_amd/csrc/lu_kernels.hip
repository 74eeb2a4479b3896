// SWAP of the right-looking LU: row interchanges, composed, then applied
// column-strip-wise, and the deferred ones left of the panels (Sec. III-A.1).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

#include "common.h"
#include "kernels.h"

namespace {

// ---------------------------------------------------------------------------
// SWAP.  compose: one workgroup turns the interchange sequence
// ipiv[j0 .. j0+cnt) (rows >= j0) into a list of moves (dst row <- src row).
// The rows that can change are rows j0 .. j0+cnt-1 and the distinct pivot
// rows beyond them (taken in order of first appearance).  For each such row
// d, the row whose contents end up in d is found by applying the
// interchanges to d in reverse order (each thread follows its own rows; the
// pivot list is read from LDS by all threads in step); every row whose
// source differs is one move.  apply: each workgroup copies the moves for a
// strip of columns, staging the gathered values in LDS so that all reads of
// a column precede all of its writes.
// ---------------------------------------------------------------------------
constexpr int kMaxSwaps = 1024;

__global__ __launch_bounds__(256) void swap_compose_kernel(const int32_t *__restrict__ ipiv,
                                                           int64_t j0, int cnt, int64_t nrows,
                                                           int *__restrict__ moves) {
    __shared__ int s_piv[kMaxSwaps];
    __shared__ int s_wsum[4];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    // relative pivot rows; an entry outside [t, nrows - j0) (possible only in
    // a sequence left by an expired wait) is taken as no interchange, so the
    // moves never address a row outside the matrix
    for (int t = tid; t < cnt; t += 256) {
        const int64_t q = (int64_t)ipiv[j0 + t] - j0;
        s_piv[t] = (q >= t && q < nrows - j0) ? (int)q : t;
    }
    __syncthreads();
    // candidate t < cnt is row t; candidate cnt + u is the pivot row of
    // interchange u when it lies beyond the block and appears there first
    int base = 0;
    for (int t0 = 0; t0 < 2 * cnt; t0 += 256) {
        const int t = t0 + tid;
        int d = -1;
        if (t < cnt) {
            d = t;
        } else if (t < 2 * cnt) {
            const int u = t - cnt;
            const int q = s_piv[u];
            if (q >= cnt) {
                d = q;
                for (int v = 0; v < u; ++v)
                    if (s_piv[v] == q) {
                        d = -1;
                        break;
                    }
            }
        }
        int src = d;
        for (int u = cnt - 1; u >= 0; --u) {
            const int q = s_piv[u];
            src = (src == u) ? q : ((src == q) ? u : src);
        }
        const bool moved = (d >= 0) && (src != d);
        // compact in candidate order: moves = [count, dst..., src...]
        const unsigned long long mask = __ballot(moved);
        const int before = __popcll(mask & ((1ull << lane) - 1ull));
        if (lane == 0) s_wsum[wv] = __popcll(mask);
        __syncthreads();
        int off = base;
        for (int k = 0; k < wv; ++k) off += s_wsum[k];
        if (moved) {
            moves[1 + off + before] = d;
            moves[1 + 2 * kMaxSwaps + off + before] = src;
        }
        const int total = s_wsum[0] + s_wsum[1] + s_wsum[2] + s_wsum[3];
        __syncthreads();
        base += total;
    }
    if (tid == 0) moves[0] = base;
}

constexpr int kSwapColsPerBlock = 32;
constexpr int kSwapBatch = 4;   // columns staged per round

template <typename T>
__global__ __launch_bounds__(256) void swap_apply_kernel(T *__restrict__ A, int64_t lda,
                                                         int64_t j0, const int *__restrict__ moves,
                                                         int64_t c_begin, int64_t ncols,
                                                         int64_t skip_begin, int64_t skip_len) {
    __shared__ int s_dst[2 * kMaxSwaps];
    __shared__ int s_src[2 * kMaxSwaps];
    __shared__ T s_val[kSwapBatch * 2 * kMaxSwaps / 2];   // 4 x 1024
    const int tid = threadIdx.x;
    const int nm = moves[0];
    for (int t = tid; t < nm; t += 256) {
        s_dst[t] = moves[1 + t];
        s_src[t] = moves[1 + 2 * kMaxSwaps + t];
    }
    __syncthreads();
    if (nm == 0) return;
    const int64_t q0 = (int64_t)blockIdx.x * kSwapColsPerBlock;
    const int64_t q1 = (q0 + kSwapColsPerBlock < ncols) ? q0 + kSwapColsPerBlock : ncols;
    const int per_round = (nm <= 1024) ? kSwapBatch : 2;   // s_val holds 4096 values
    const int64_t skip_rel = skip_begin - c_begin;
    for (int64_t qb = q0; qb < q1; qb += per_round) {
        const int nb = (int)((q1 - qb < per_round) ? q1 - qb : per_round);
        for (int t = tid; t < nb * nm; t += 256) {
            const int b = t / nm, mv = t - b * nm;
            const int64_t q = qb + b;
            const int64_t c = c_begin + ((q < skip_rel) ? q : q + skip_len);
            s_val[t] = MXLU_AT(A, j0 + s_src[mv], c, lda);
        }
        __syncthreads();
        for (int t = tid; t < nb * nm; t += 256) {
            const int b = t / nm, mv = t - b * nm;
            const int64_t q = qb + b;
            const int64_t c = c_begin + ((q < skip_rel) ? q : q + skip_len);
            MXLU_AT(A, j0 + s_dst[mv], c, lda) = s_val[t];
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Deferred interchanges of the columns left of the panels.  No later step
// reads the L columns of a finished panel, so their row interchanges can wait
// until the factorization is done; then each element moves once.  Panel j's
// rows below it end up gathered through q_j = r_{j+1} o ... o r_{K-1}, the
// composition of the gather maps of the later steps' interchanges (r_s(i) is
// the row whose content step s moves to row i: the identity but for the
// moves of step s).  q is built from the last step backwards.
__global__ void perm_iota_kernel(int64_t n, int32_t *__restrict__ q) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) q[i] = (int32_t)i;
}

// r at the moved rows of one step: their sources (set) or themselves (reset)
__global__ void perm_moves_kernel(const int *__restrict__ moves, int64_t j0,
                                  int32_t *__restrict__ r, int reset) {
    const int nm = moves[0];
    for (int t = threadIdx.x; t < nm; t += 256) {
        const int d = moves[1 + t];
        r[j0 + d] = (int32_t)(j0 + (reset ? d : moves[1 + 2 * kMaxSwaps + t]));
    }
}

// q[i] <- r[q[i]] for rows [i0, n)
__global__ void perm_compose_kernel(int64_t i0, int64_t n, const int32_t *__restrict__ r,
                                    int32_t *__restrict__ q) {
    const int64_t i = i0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) q[i] = r[q[i]];
}

// T (rows x cols, leading dimension rows) <- A[q[r0 + i], c0 + c]
__global__ void gather_panel_rows_kernel(const double *__restrict__ A, int64_t lda, int64_t r0,
                                         int64_t rows, int64_t c0, const int32_t *__restrict__ q,
                                   double *__restrict__ T) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t c = blockIdx.y;
    if (i < rows) T[i + c * rows] = MXLU_AT(A, q[r0 + i], c0 + c, lda);
}

// A[r0 + i, c0 + c] <- T
__global__ void put_panel_rows_kernel(const double *__restrict__ T, int64_t rows, double *__restrict__ A,
                                int64_t lda, int64_t r0, int64_t c0) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t c = blockIdx.y;
    if (i < rows) MXLU_AT(A, r0 + i, c0 + c, lda) = T[i + c * rows];
}

}  // namespace

namespace mxlu {

int swap_compose(const int32_t *ipiv, int64_t j0, int cnt, int64_t nrows, int *moves,
                 hipStream_t s) {
    if (cnt <= 0) return 0;
    if (cnt > kMaxSwaps || !moves || nrows - j0 > INT_MAX) {
        set_error_msg("laswp: too many interchanges, rows or no move buffer");
        return MXLU_E_NOMEM;
    }
    hipLaunchKernelGGL(swap_compose_kernel, dim3(1), dim3(256), 0, s, ipiv, j0, cnt, nrows,
                       moves);
    MXLU_LAUNCH_CHECK();
    return 0;
}

template <typename T>
int swap_apply(T *A, int64_t lda, int64_t j0, const int *moves, int64_t c_begin, int64_t ncols,
               int64_t skip_begin, int64_t skip_len, hipStream_t s) {
    if (ncols <= 0) return 0;
    const unsigned grid = (unsigned)((ncols + kSwapColsPerBlock - 1) / kSwapColsPerBlock);
    hipLaunchKernelGGL(swap_apply_kernel<T>, dim3(grid), dim3(256), 0, s, A, lda, j0, moves,
                       c_begin, ncols, skip_begin, skip_len);
    MXLU_LAUNCH_CHECK();
    return 0;
}
template int swap_apply<double>(double *, int64_t, int64_t, const int *, int64_t, int64_t,
                                int64_t, int64_t, hipStream_t);
template int swap_apply<float>(float *, int64_t, int64_t, const int *, int64_t, int64_t, int64_t,
                               int64_t, hipStream_t);
template int swap_apply<uint16_t>(uint16_t *, int64_t, int64_t, const int *, int64_t, int64_t,
                                  int64_t, int64_t, hipStream_t);

int laswp_f64(double *A, int64_t lda, int64_t nrows, const int32_t *ipiv, int64_t j0, int cnt,
              int64_t c_begin, int64_t ncols, int64_t skip_begin, int64_t skip_len,
              int *moves, hipStream_t s) {
    if (cnt <= 0 || ncols <= 0) return 0;
    MXLU_TRY(swap_compose(ipiv, j0, cnt, nrows, moves, s));
    return swap_apply<double>(A, lda, j0, moves, c_begin, ncols, skip_begin, skip_len, s);
}

int laswp_left_deferred_f64(double *A, int64_t lda, int64_t n, int64_t nb,
                            const int32_t *ipiv, int *moves, int32_t *q, int32_t *r, double *T,
                            hipStream_t s) {
    const int64_t K = (n + nb - 1) / nb;
    if (K < 2) return 0;
    const unsigned gn = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(perm_iota_kernel, dim3(gn), dim3(256), 0, s, n, q);
    MXLU_LAUNCH_CHECK();
    hipLaunchKernelGGL(perm_iota_kernel, dim3(gn), dim3(256), 0, s, n, r);
    MXLU_LAUNCH_CHECK();
    for (int64_t j = K - 2; j >= 0; --j) {
        const int64_t j1 = (j + 1) * nb, kb1 = std::min(nb, n - j1);
        // q <- r_{j+1} o q
        MXLU_TRY(swap_compose(ipiv, j1, (int)kb1, n, moves, s));
        hipLaunchKernelGGL(perm_moves_kernel, dim3(1), dim3(256), 0, s, moves, j1, r, 0);
        MXLU_LAUNCH_CHECK();
        const int64_t rows = n - j1;
        const unsigned gr = (unsigned)((rows + 255) / 256);
        hipLaunchKernelGGL(perm_compose_kernel, dim3(gr), dim3(256), 0, s, j1, n, r, q);
        MXLU_LAUNCH_CHECK();
        hipLaunchKernelGGL(perm_moves_kernel, dim3(1), dim3(256), 0, s, moves, j1, r, 1);
        MXLU_LAUNCH_CHECK();
        // panel j's columns, rows below it, gathered through q
        const int64_t c0 = j * nb, cols = nb;
        hipLaunchKernelGGL(gather_panel_rows_kernel, dim3(gr, (unsigned)cols), dim3(256), 0, s, A, lda,
                           j1, rows, c0, q, T);
        MXLU_LAUNCH_CHECK();
        hipLaunchKernelGGL(put_panel_rows_kernel, dim3(gr, (unsigned)cols), dim3(256), 0, s, T, rows, A,
                           lda, j1, c0);
        MXLU_LAUNCH_CHECK();
    }
    return 0;
}

}  // namespace mxlu
