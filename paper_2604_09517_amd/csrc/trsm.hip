// B <- L^-1 B with L unit lower, up to 256 rows (FP64 and FP32): the row-panel
// solves of the factorizations.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"
#include "matrix16.h"
#include "quarter.h"

namespace {

// A workgroup takes 16 columns of B and all rows, in strips of 16 rows: wave v
// owns strips v, v + 8, each one 16 x 16 matrix-core accumulator.  A strip's
// owner solves it four rows a step, the waves of later strips apply its
// solution with the matrix cores, its next reader first.
//
// What bounds it is the chain of strips (16 for 256 rows), so a strip is kept
// short: the accumulator of quarter wave b holds rows 4 b .. 4 b + 3 of its
// lane's column, so that the four are solved within the lane (six multiply-
// adds, factor entries in registers), three lane permutes (a 4 x 4 transpose
// over the quarters) turn them into a matrix operand, and one matrix
// instruction takes them to the strip's rows still to come.  The factor's
// tiles are loaded a strip ahead.  Every element takes its terms in ascending
// order of k, one fused multiply-add each (a matrix instruction adds its four
// products one after the other, rounding each time).
// 512 threads hide what they can of it: two strips a wave at most, so that the
// next owner has little else to do.
//
// 32 / 64 / 128 / 256 rows against as many columns, us: FP64 4.6 / 4.7 / 7.4 /
// 16.3, FP32 5.0 / 5.4 / 7.9 / 13.4 (a launch that does nothing is about 3).
// With a thread per row, a barrier per row and 16 columns per workgroup the
// averages inside the factorizations were 18 us (n = 1024, 32 and 64 rows), 28
// (FP64, n = 5001, all four; now 6.3) and 32 (FP32, n = 3001; now 8).
constexpr int kStripRows = 16, kWaves = 8;

// Strip row that row i of the instruction stands for, so that lane (li, lq)
// accumulates strip rows 4 lq + r (FP64 accumulates rows lq + 4 r).
template <typename T>
__device__ __forceinline__ int strip_row(int i) {
    return sizeof(T) == 8 ? 4 * (i & 3) + (i >> 2) : i;
}

// NQ strips per wave: kb <= 128 NQ; min(8, strips) waves.  NT tiles of 16 columns.
template <typename T, int NQ, int NT>
__global__ __launch_bounds__(64 * kWaves) void trsm_llnu_kernel(int kb, int64_t ncols,
                                                                const T *__restrict__ L, int64_t ldl,
                                                                T *__restrict__ B, int64_t ldb) {
    using V4 = typename Mat<T>::V4;
    __shared__ T X[NQ * kWaves * kStripRows][16 * NT + 1];   // (odd: columns spread over the banks)
    __shared__ T D[NQ * kWaves][kStripRows][kStripRows];
    const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4;
    const int v = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int nstr = (kb + kStripRows - 1) / kStripRows;
    const int64_t c0 = (int64_t)blockIdx.x * (16 * NT);

    // rows past kb: others' values, used by nothing but rows past kb
    V4 acc[NQ][NT];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
            const int64_t col = c0 + 16 * c + li < ncols ? c0 + 16 * c + li : ncols - 1;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int row = min(kStripRows * (kWaves * q + v) + 4 * lq + r, kb - 1);
                acc[q][c][r] = B[(size_t)row + (size_t)col * ldb];
            }
        }
    // tile of strip t's rows and strip s's columns as a matrix operand
    auto tile = [&](int t, int s, T(&a)[4]) {
        const int row = min(kStripRows * t + strip_row<T>(li), kb - 1);
        const T *src = L + (size_t)row + (size_t)(kStripRows * s + lq) * ldl;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) a[kk] = src[(size_t)(4 * kk) * ldl];
    };
    // strip t's own tile waits in LDS (by columns); ahead of its turn, own
    // takes the 4 x 4 triangles (uniform), and the rows below each of them
    // against its four columns as a matrix operand
    auto stage = [&](int t) {
        const int row = min(kStripRows * t + li, kb - 1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            D[t][4 * kk + lq][li] =
                -L[(size_t)row + (size_t)min(kStripRows * t + 4 * kk + lq, kb - 1) * ldl];
    };
    T tri[4][6], below[4];
    auto own = [&](int t) {
#pragma unroll
        for (int b = 0; b < 4; ++b) {
#pragma unroll
            for (int i = 1, e = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < i; ++k, ++e) tri[b][e] = D[t][4 * b + k][4 * b + i];
            const int i = strip_row<T>(li);
            below[b] = i >= 4 * b + 4 ? D[t][4 * b + lq][i] : (T)0;
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {   // here, not where they are used
#pragma unroll
            for (int e = 0; e < 6; ++e) asm volatile("" : "+v"(tri[b][e]));
            asm volatile("" : "+v"(below[b]));
        }
    };
    auto solve = [&](V4(&c)[NT], int t) {
        auto step = [&](auto bq) {
            constexpr int b = decltype(bq)::value;
            T y[NT][4], x[NT];
#pragma unroll
            for (int h = 0; h < NT; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i) y[h][i] = c[h][i];
#pragma unroll
            for (int i = 1, e = 0; i < 4; ++i)
#pragma unroll
                for (int k = 0; k < i; ++k, ++e)
#pragma unroll
                    for (int h = 0; h < NT; ++h) y[h][i] = fma(tri[b][e], y[h][k], y[h][i]);
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                x[h] = spread<b>(y[h]);   // row 4 b + lq
                if (b < 3) c[h] = Mat<T>::mul(below[b], x[h], c[h]);
            }
#pragma unroll
            for (int h = 0; h < NT; ++h) X[kStripRows * t + 4 * b + lq][16 * h + li] = x[h];
        };
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
    };

    // a[j]: the tiles of strips s = j (mod 2), loaded when strip s - 2 has been
    // applied
    T a[2][NQ][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (kWaves * q + v > j && kWaves * q + v < nstr) tile(kWaves * q + v, j, a[j][q]);
#pragma unroll
    for (int q = 0; q < NQ; ++q) stage(kWaves * q + v);
    wave_sync_lds();   // the wave's own strips
    if (v < 2) own(v);
    if (v == 0) solve(acc[0], 0);
    auto strips = [&](auto qq) {   // strips 8 q .. 8 q + 7 as they are solved
        constexpr int q = decltype(qq)::value;
        for (int o2 = 0; o2 < kWaves; o2 += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int o = o2 + j, s = kWaves * q + o;
                if (s + 1 >= nstr) return;
                lds_barrier();
                T x[NT][4];
#pragma unroll
                for (int h = 0; h < NT; ++h)
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
                        x[h][kk] = -X[kStripRows * s + 4 * kk + lq][16 * h + li];
#pragma unroll
                for (int p = q; p < NQ; ++p) {
                    const int t = kWaves * p + v;
                    if (t <= s || t >= nstr) continue;
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                        for (int h = 0; h < NT; ++h)
                            acc[p][h] = Mat<T>::mul(a[j][p][kk], x[h][kk], acc[p][h]);
                    if (t > s + 2) tile(t, s + 2, a[j][p]);
                    if (t == s + 1) solve(acc[p], t);
                    if (t == s + 2) own(t);
                }
            }
        }
    };
    strips(std::integral_constant<int, 0>{});
    if constexpr (NQ > 1) strips(std::integral_constant<int, 1>{});
    lds_barrier();
    for (int c = v; c < 16 * NT && c0 + c < ncols; c += nw)
        for (int row = lane; row < kb; row += 64) B[(size_t)row + (size_t)(c0 + c) * ldb] = X[row][c];
}

}  // namespace

namespace mxlu {

template <typename T>
int trsm_llnu(int kb, int64_t ncols, const T *L, int64_t ldl, T *B, int64_t ldb, hipStream_t s) {
    if (kb <= 0 || ncols <= 0) return 0;
    if (kb > 256 || ncols > (int64_t)0x7fffffff * 16) {
        set_error_msg("trsm: diagonal block larger than 256 or too many columns");
        return MXLU_E_NOMEM;
    }
    const dim3 block(64 * std::min(kWaves, (kb + kStripRows - 1) / kStripRows));
    const dim3 narrow((unsigned)((ncols + 15) / 16)), wide((unsigned)((ncols + 31) / 32));
    // Two tiles of columns a workgroup (independent chains side by side, the
    // factor read once for both) when one would leave more workgroups than
    // run at once: one per CU in FP64, two in FP32.  256 rows: 4600 columns
    // FP64 33 -> 28 us, 24000 columns 130 -> 103; FP32 6000 columns 18 -> 21,
    // 12000 columns 30 -> 28, 49000 columns 246 -> 162.
    const bool two = ncols > (sizeof(T) == 8 ? 4096 : 8192);
    if (kb <= kWaves * kStripRows) {
        if (two)
            hipLaunchKernelGGL((trsm_llnu_kernel<T, 1, 2>), wide, block, 0, s, kb, ncols, L, ldl, B, ldb);
        else
            hipLaunchKernelGGL((trsm_llnu_kernel<T, 1, 1>), narrow, block, 0, s, kb, ncols, L, ldl, B, ldb);
    } else {
        if (two)
            hipLaunchKernelGGL((trsm_llnu_kernel<T, 2, 2>), wide, block, 0, s, kb, ncols, L, ldl, B, ldb);
        else
            hipLaunchKernelGGL((trsm_llnu_kernel<T, 2, 1>), narrow, block, 0, s, kb, ncols, L, ldl, B, ldb);
    }
    MXLU_LAUNCH_CHECK();
    return 0;
}
template int trsm_llnu<double>(int, int64_t, const double *, int64_t, double *, int64_t, hipStream_t);
template int trsm_llnu<float>(int, int64_t, const float *, int64_t, float *, int64_t, hipStream_t);

}  // namespace mxlu
