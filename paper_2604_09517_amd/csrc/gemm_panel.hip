// C -= A B for the shapes inside a panel: many rows, few columns, short K
// (FP64 and FP32).
#include <hip/hip_runtime.h>

#include "common.h"
#include "kernels.h"
#include "matrix16.h"

namespace {

// A workgroup takes 64 rows and up to 64 columns of C, each wave 16 rows; K in
// chunks of 32.  The products are formed transposed (matrix rows: columns of C), so
// that the 16 lanes of a quarter wave are 16 consecutive rows of A and of C
// and both move as whole lines, A straight into the operand registers; only
// the chunk of B, which every wave needs, goes through LDS.
//
// These products are bound by the latency of a few dependent trips to memory
// and by how many CUs they reach (10 MFLOP and 4 MB at 5000 rows and 32
// columns): the loads of two chunks and of C are in flight at once, later
// chunks' two ahead, and tiles of 64 x 64 put 5000 rows on 79
// CUs, where 128 x 128 tiles reached 40 and spent three quarters of their
// matrix instructions on columns that are not there.
// Terms in ascending k, starting from C.
//
// us, by tiles of 128 x 128 in LDS (FP32: 64 x 64 without matrix instructions)
// and now: FP64, 4000 rows, N = K = 32 / 64 / 128: 17 / 17 / 18 -> 4.9 / 9 / 11;
// 20000 rows, 54 -> 18 / 25 / 42; 970 x 970, K = 64: 29 -> 10.5.  FP32, 2000
// rows, N = K = 64 / 128: 22 / 25 -> 7 / 8; 50000 rows, N = K = 256: 200 -> 165.
constexpr int kTile = 64, kChunk = 32;   // rows of a workgroup, k of a chunk
constexpr int kBst = 81;   // LDS row of a k: odd, and 4 rows apart in the banks

// NF: tiles of 16 columns per workgroup.
template <typename T, int NF>
__global__ __launch_bounds__(256) void gemm_panel_kernel(int64_t M, int64_t N, int64_t K,
                                                         const T *__restrict__ A, int64_t lda,
                                                         const T *__restrict__ B, int64_t ldb,
                                                         T *__restrict__ C, int64_t ldc, int tiles_n) {
    using V4 = typename Mat<T>::V4;
    constexpr int KS = kChunk / 4, NB = 2 * NF;   // steps of a chunk; values of B per thread
    __shared__ T Bs[2][kChunk][kBst];
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lq = lane >> 4;
    const int wave = tid >> 6;
    const int64_t tn = blockIdx.x % tiles_n, tm = blockIdx.x / tiles_n;
    const int64_t row = tm * kTile + 16 * wave + li, col0 = tn * (16 * NF);
    // rows and columns past the matrix: others' values, not stored; terms past
    // K: 0 times -0, which leaves even a sum of -0 as it is.  No load is under a
    // condition, so that all stay in flight together.
    const int64_t rowc = row < M ? row : M - 1;
    const T *Ar = A + rowc;
    const int bk = tid & 31, bc = tid >> 5;   // the thread's k and first column of a chunk of B
    auto load = [&](int64_t k0, T(&a)[KS], T(&b)[NB]) {
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) {
            const int64_t k = k0 + 4 * kk + lq;
            a[kk] = Ar[(size_t)(k < K ? k : K - 1) * lda];
        }
        const int64_t k = k0 + bk;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int64_t col = col0 + bc + 8 * q;
            b[q] = B[(size_t)(k < K ? k : K - 1) + (size_t)(col < N ? col : N - 1) * ldb];
        }
    };
    T a[2][KS], b[2][NB];
    load(0, a[0], b[0]);
    V4 acc[NF];
#pragma unroll
    for (int t = 0; t < NF; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int64_t col = col0 + 16 * t + Mat<T>::row(lq, r);
            acc[t][r] = C[(size_t)rowc + (size_t)(col < N ? col : N - 1) * ldc];
        }
    load(kChunk, a[1], b[1]);
    for (int64_t k1 = 0; k1 < K; k1 += 2 * kChunk) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int64_t k0 = k1 + h * kChunk;
            if (k0 >= K) break;   // uniform
#pragma unroll
            for (int q = 0; q < NB; ++q) Bs[h][bk][bc + 8 * q] = k0 + bk < K ? -b[h][q] : -(T)0;
            lds_barrier();   // (the chunk before last is consumed: one barrier a chunk is enough)
            if (k0 + kChunk > K)
#pragma unroll
                for (int kk = 0; kk < KS; ++kk) a[h][kk] = k0 + 4 * kk + lq < K ? a[h][kk] : (T)0;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk)
#pragma unroll
                for (int t = 0; t < NF; ++t)
                    acc[t] = Mat<T>::mul(Bs[h][4 * kk + lq][16 * t + li], a[h][kk], acc[t]);
            load(k0 + 2 * kChunk, a[h], b[h]);   // past the end: the last values again, not used
        }
    }
    if (row < M)
#pragma unroll
        for (int t = 0; t < NF; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t col = col0 + 16 * t + Mat<T>::row(lq, r);
                if (col < N) C[(size_t)row + (size_t)col * ldc] = acc[t][r];
            }
}

}  // namespace

namespace mxlu {

template <typename T>
int gemm_panel_sub(int64_t M, int64_t N, int64_t K, const T *A, int64_t lda, const T *B, int64_t ldb,
                   T *C, int64_t ldc, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    const int nf = N <= 16 ? 1 : N <= 32 ? 2 : 4;
    const int64_t tm = (M + kTile - 1) / kTile, tn = (N + 16 * nf - 1) / (16 * nf);
    if (tm > 0x7fffffff / tn) {
        set_error_msg("gemm_panel_sub: grid too large");
        return MXLU_E_NOMEM;
    }
    const dim3 grid((unsigned)(tm * tn));
    if (nf == 1)
        hipLaunchKernelGGL((gemm_panel_kernel<T, 1>), grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, C,
                           ldc, (int)tn);
    else if (nf == 2)
        hipLaunchKernelGGL((gemm_panel_kernel<T, 2>), grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, C,
                           ldc, (int)tn);
    else
        hipLaunchKernelGGL((gemm_panel_kernel<T, 4>), grid, dim3(256), 0, s, M, N, K, A, lda, B, ldb, C,
                           ldc, (int)tn);
    MXLU_LAUNCH_CHECK();
    return 0;
}
template int gemm_panel_sub<double>(int64_t, int64_t, int64_t, const double *, int64_t, const double *,
                                    int64_t, double *, int64_t, hipStream_t);
template int gemm_panel_sub<float>(int64_t, int64_t, int64_t, const float *, int64_t, const float *,
                                   int64_t, float *, int64_t, hipStream_t);

}  // namespace mxlu
