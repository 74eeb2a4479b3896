// Trailing-matrix update C -= A * B in FP64 on the matrix cores (gfx950).
//
// This is the DGEMM phase of the right-looking blocked LU (Sec. III-A.1: the
// update of the trailing submatrix, which carries almost all of the 2/3 N^3
// flops): A22 -= L21 * U12 with A = L21 (M x K), B = U12 (K x N), C = A22.
//
// Design (CDNA4):
//   * 256 threads = 4 waves in a 2 x 2 arrangement; a workgroup owns a
//     128 x 128 tile of C, each wave a 64 x 64 sub-tile held as 4 x 4
//     accumulators of v_mfma_f64_16x16x4_f64 (64 doubles per lane).
//   * The accumulators start from C and the MFMA consumes -A, so the tile is
//     read once and written once: C - sum_k a_ik b_kj in one pass.
//   * K is walked in steps of four k, operands loaded a few steps ahead;
//     chunks of B of 16 k go through LDS in the general kernel, through a
//     packed copy in the one for whole tiles.
//   * Tile order: consecutive workgroup ids are dealt round-robin over the 8
//     XCDs, so ids are remapped to give every XCD a contiguous run of tiles,
//     and tiles are ordered in groups of 8 tile-rows so that tiles that share
//     A rows run on the same XCD (shared L2).
//
// MFMA operand layout (16x16x4 f64, wave64; lane l, i = l % 16, q = l / 16),
// measured on gfx950: A operand A[i][q]; B operand B[q][i]; accumulator
// register r holds D[q + 4r][i].
#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 16;
constexpr int BST = BN + 4;   // LDS row of a k (padded: 16 k's of a column spread over the banks)
constexpr int GROUP_M = 8;

__device__ inline void tile_of(int g, int tiles_m, int tiles_n, int &tm, int &tn) {
    const int G = tiles_m * tiles_n;
    // XCD-contiguous remap: id g runs on XCD g % 8.
    const int per = G / 8, rem = G % 8;
    const int xcd = g % 8, local = g / 8;
    const int t = (xcd < rem) ? xcd * (per + 1) + local
                              : rem * (per + 1) + (xcd - rem) * per + local;
    // grouped order: GROUP_M tile-rows at a time, column-major inside a group
    const int in_group = GROUP_M * tiles_n;
    const int group = t / in_group;
    const int first_m = group * GROUP_M;
    const int gsize = min(tiles_m - first_m, GROUP_M);
    const int r = t - group * in_group;
    tm = first_m + r % gsize;
    tn = r / gsize;
}

// Any shape, alignment and leading dimension.  The product is formed
// transposed (matrix rows: columns of C), so that the 16 lanes of a quarter
// wave are 16 consecutive rows of A and of C: A goes straight into the operand
// registers, three steps of four k ahead, by 8-byte loads that need no alignment,
// and C moves as whole lines; the chunk of B, which all waves need, goes
// through two LDS buffers (one barrier a chunk).  No load is under a
// condition: rows and columns past the matrix read others' values and are not
// stored, terms past K are made zeros in the last chunk.
// 6100 x 7003, K = 300: 688 -> 590 us (43 TFLOP/s; a form that staged A too,
// by loads under a condition each, had 37); 4700 x 4700, K = 256: 288 -> 235.
// Bound by the matrix cores (330 us) and by C (683 MB, 157 us), which hardly
// overlap, and by the last round of tiles.
// TRANSB: B is given as its transpose (element (k, j) at B[j + k ldb]);
// ZEROC: C starts from zero instead of being read.
template <bool TRANSB, bool ZEROC>
__global__ __launch_bounds__(256, 2) void gemm_f64_sub_kernel(
    int64_t M, int64_t N, int64_t K, const double *__restrict__ A, int64_t lda,
    const double *__restrict__ B, int64_t ldb, double *__restrict__ C, int64_t ldc,
    int tiles_m, int tiles_n) {
    __shared__ double Bs[2][BK][BST];

    int tm, tn;
    tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lq = lane >> 4;
    const int64_t row0 = (int64_t)tm * BM + (wave & 1) * 64 + li;   // of the lane, tile 0
    const int64_t col0 = (int64_t)tn * BN;
    const int wn = (wave >> 1) * 64;

    // the lane's rows of A; a step of four k at a time, three steps ahead
    const double *Ar[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) Ar[i] = A + (row0 + 16 * i < M ? row0 + 16 * i : M - 1);
    auto load_a = [&](int64_t k, double (&a)[4]) {
        const size_t off = (size_t)(k + lq < K ? k + lq : K - 1) * (size_t)lda;
#pragma unroll
        for (int i = 0; i < 4; ++i) a[i] = Ar[i][off];
    };
    // the thread's part of a chunk of B: columns bc + 16 q of one k, or
    // (TRANSB) k's bk + 2 q of one column
    const int bk = TRANSB ? tid >> 7 : tid & 15, bc = TRANSB ? tid & 127 : tid >> 4;
    auto load_b = [&](int64_t k0, double (&b)[8]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t c = col0 + bc + (TRANSB ? 0 : 16 * q), cc = c < N ? c : N - 1;
            const int64_t k = k0 + bk + (TRANSB ? 2 * q : 0), kc = k < K ? k : K - 1;
            b[q] = TRANSB ? MXLU_AT(B, cc, kc, ldb) : MXLU_AT(B, kc, cc, ldb);
        }
    };
    auto put_b = [&](int64_t k0, int buf, const double (&b)[8]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = bk + (TRANSB ? 2 * q : 0);
            Bs[buf][k][bc + (TRANSB ? 0 : 16 * q)] = k0 + k < K ? -b[q] : -0.0;
        }
    };

    constexpr int D = BK / 4;   // steps of a chunk, sets of the ring
    double a[D][4], b[8];
    if (K > 0) {
        load_b(0, b);
#pragma unroll
        for (int u = 0; u < D - 1; ++u) load_a(4 * u, a[u]);
    }
    v4d acc[4][4];   // [tile of columns][tile of rows]: columns lq + 4 e, row li
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t r = row0 + 16 * i, c = col0 + wn + 16 * j + lq + 4 * e;
                acc[j][i][e] = ZEROC ? 0.0 : MXLU_AT(C, r < M ? r : M - 1, c < N ? c : N - 1, ldc);
            }
    if (K > 0) put_b(0, 0, b);
    retire_vector_loads();
    for (int64_t k0 = 0; k0 < K; k0 += BK) {
        const int h = (int)(k0 / BK) & 1;
        lds_barrier();   // this chunk of B is there, the one before is consumed
        load_b(k0 + BK, b);   // past the end: the last values again, not used
#pragma unroll
        for (int u = 0; u < D; ++u) {
            load_a(k0 + 4 * (u + D - 1), a[(u + D - 1) % D]);
            __builtin_amdgcn_sched_barrier(0);   // (left alone, the loads sink to their use)
            double av[4], bv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) av[i] = a[u][i];
            if (k0 + BK > K)
#pragma unroll
                for (int i = 0; i < 4; ++i) av[i] = k0 + 4 * u + lq < K ? av[i] : 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) bv[j] = Bs[h][4 * u + lq][wn + 16 * j + li];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[j][i] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv[j], av[i], acc[j][i], 0, 0, 0);
        }
        put_b(k0 + BK, h ^ 1, b);
    }
    const bool inside = (int64_t)(tm + 1) * BM <= M && col0 + BN <= N;   // uniform
    auto store = [&](auto all) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t r = row0 + 16 * i, c = col0 + wn + 16 * j + lq + 4 * e;
                    if (decltype(all)::value || (r < M && c < N)) MXLU_AT(C, r, c, ldc) = acc[j][i][e];
                }
    };
    if (inside) store(std::true_type{});
    else store(std::false_type{});
}

// Trailing update of the factorization, full tiles only: C -= A B with the
// same 128 x 128 tile and 2 x 2 wave arrangement as above, but with no LDS
// and no barrier: every wave loads its own operand fragments straight into
// registers with 16-byte loads, kDirectSets chunks of 4 k deep (three in
// flight while the MFMAs consume the fourth), so the four waves of a tile
// never wait for each other.  B is read from Bn, a packed copy of -B^T (row k
// holds -B[k][0 .. N), leading dimension ldbn), so the product needs no
// negation and a fragment of 2 adjacent columns is one 16-byte load.
//
// A 16-byte load gives a lane two adjacent rows of A (or columns of Bn), so
// the index i' of fragment pair p, half h stands for tile row 32 p + 2 i' + h
// of the wave's 64 (columns likewise): lane (li, lq) loads A rows wm*64 + 32p +
// 2li + {0, 1} and Bn columns wn*64 + 32p + 2li + {0, 1} at k = 4 kc + lq.  The
// product is formed transposed: MFMA (b, a) with a = 2 pa + ha, b = 2 pb + hb
// leaves in accumulator register r of lane (li, lq) the element at tile row
// wm*64 + 32 pa + 2 li + ha and tile column wn*64 + 32 pb + 2 (lq + 4 r) + hb,
// so that C moves as 16-byte pairs of rows, 256 bytes of a column at a time.
// Every element still takes its k terms in ascending groups of 4, starting
// from C, as in the LDS kernel.
// Bound by the matrix cores, and by C, whose loads and stores hardly overlap
// with them (all tiles of a round start together): n = 32768, K = 256: 60.5
// TFLOP/s with C by 64-byte pieces of a column, 64 by 256 bytes, 65.5 with C
// also past the caches, which keep the panels (a large library product: 73).
constexpr int kDirectSets = 4, kDirectK = 4 * kDirectSets;
typedef double v2d __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(256, 2) void gemm_f64_direct_kernel(
    int64_t M, int64_t N, int64_t K, const double *__restrict__ A, int64_t lda,
    const double *__restrict__ Bn, int64_t ldbn, double *__restrict__ C, int64_t ldc,
    int tiles_m, int tiles_n) {
    int tm, tn;
    tile_of(blockIdx.x, tiles_m, tiles_n, tm, tn);
    const int64_t row0 = (int64_t)tm * BM + ((threadIdx.x >> 6) & 1) * 64;
    const int64_t col0 = (int64_t)tn * BN + (threadIdx.x >> 7) * 64;
    const int lane = threadIdx.x & 63;
    const int li = lane & 15, lq = lane >> 4;

    // C columns 32 (b / 2) + 2 (lq + 4 r) + b % 2, rows 32 pa + 2 li + {0, 1}
    double *Cb = &MXLU_AT(C, row0 + 2 * li, col0 + 2 * lq, ldc);
    v4d acc[4][4];   // [b][a]
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int pa = 0; pa < 2; ++pa) {
                const v2d v = __builtin_nontemporal_load(
                    (const v2d *)&MXLU_AT(Cb, 32 * pa, 32 * (b >> 1) + 8 * r + (b & 1), ldc));
                acc[b][2 * pa][r] = v.x;
                acc[b][2 * pa + 1][r] = v.y;
            }

    const double *Ab = &MXLU_AT(A, row0 + 2 * li, lq, lda);
    const double *Bb = Bn + (size_t)lq * ldbn + col0 + 2 * li;
    const int nk = (int)(K / 4);
    v2d fa[kDirectSets][2], fb[kDirectSets][2];
    // chunks past the end reload the last one (never consumed), so that every
    // step issues the same loads and the wait before each step is the same
    auto load = [&](int kc, v2d (&xa)[2], v2d (&xb)[2]) {
        const int64_t k = (int64_t)4 * min(kc, nk - 1);
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            xa[p] = *(const v2d *)(Ab + 32 * p + k * lda);
            xb[p] = *(const v2d *)(Bb + 32 * p + k * ldbn);
        }
    };
#pragma unroll
    for (int st = 0; st < kDirectSets - 1; ++st) load(st, fa[st], fb[st]);
    // the scheduling barriers keep each prefetch where it is written: left
    // alone, the scheduler sinks the loads next to their use
    __builtin_amdgcn_sched_barrier(0);
    for (int kt0 = 0; kt0 < nk; kt0 += kDirectSets) {
#pragma unroll
        for (int u = 0; u < kDirectSets; ++u) {
            constexpr int D = kDirectSets;
            load(kt0 + u + D - 1, fa[(u + D - 1) % D], fb[(u + D - 1) % D]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const double av = (a & 1) ? fa[u][a >> 1].y : fa[u][a >> 1].x;
                    const double bv = (b & 1) ? fb[u][b >> 1].y : fb[u][b >> 1].x;
                    acc[b][a] = __builtin_amdgcn_mfma_f64_16x16x4f64(bv, av, acc[b][a], 0, 0, 0);
                }
        }
    }

#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int pa = 0; pa < 2; ++pa) {
                v2d v;
                v.x = acc[b][2 * pa][r];
                v.y = acc[b][2 * pa + 1][r];
                __builtin_nontemporal_store(v, (v2d *)&MXLU_AT(Cb, 32 * pa, 32 * (b >> 1) + 8 * r + (b & 1), ldc));
            }
}

// Bn[k][j] = -B[k][j] (B column-major K x N, Bn row-major with ldbn), through
// 32 x 32 LDS tiles so that reads and writes are both coalesced.
__global__ __launch_bounds__(256) void pack_neg_transpose_kernel(int64_t K, int64_t N,
                                                                 const double *__restrict__ B,
                                                                 int64_t ldb,
                                                                 double *__restrict__ Bn,
                                                                 int64_t ldbn, int tiles_k) {
    __shared__ double T[32][33];
    const int64_t k0 = (int64_t)(blockIdx.x % tiles_k) * 32;
    const int64_t j0 = (int64_t)(blockIdx.x / tiles_k) * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t k = k0 + tx, j = j0 + ty + 8 * q;
        T[ty + 8 * q][tx] = (k < K && j < N) ? -B[(size_t)k + (size_t)j * ldb] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t k = k0 + ty + 8 * q, j = j0 + tx;
        if (k < K && j < N) Bn[(size_t)k * ldbn + j] = T[tx][ty + 8 * q];
    }
}

}  // namespace

namespace mxlu {

int gemm_f64_sub(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                 const double *B, int64_t ldb, double *C, int64_t ldc, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    if (tiles_m * tiles_n > 0x7fffffff) {
        set_error_msg("gemm_f64_sub: grid too large");
        return MXLU_E_NOMEM;
    }
    // 64 x 64 tiles for fewer columns than a tile (N = K = 32, 4000 rows 17 -> 4.9
    // us), and where the large ones leave CUs idle: a round of 256 large tiles
    // takes as long as 3.7 of 256 small ones, so up to three of those (K = 512,
    // us, large / small: 1408 x 1408 89 / 54, 1664 x 1664 90 / 75, 1790 x 1790
    // 92 / 98, 256 x 14000 92 / 99; K = 64: 18.1 / 12.9, 18.4 / 17.3, 19.9 /
    // 23.2).
    const int64_t small = ((M + 63) / 64) * ((N + 63) / 64);
    if (N <= 128 || (tiles_m * tiles_n < 256 && small <= 768))
        return gemm_panel_sub<double>(M, N, K, A, lda, B, ldb, C, ldc, s);
    const dim3 grid((unsigned)(tiles_m * tiles_n));
    hipLaunchKernelGGL((gemm_f64_sub_kernel<false, false>), grid, dim3(256), 0, s, M, N, K, A, lda, B,
                       ldb, C, ldc, (int)tiles_m, (int)tiles_n);
    MXLU_LAUNCH_CHECK();
    return 0;
}

bool gemm_f64_update_ok(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda) {
    return M > 0 && N > 0 && K > 0 && M % BM == 0 && N % BN == 0 && K % kDirectK == 0 &&
           lda % 2 == 0 && ((uintptr_t)A % 16) == 0;
}

int pack_neg_transpose_f64(int64_t K, int64_t N, const double *B, int64_t ldb, double *Bn,
                           int64_t ldbn, hipStream_t s) {
    if (K <= 0 || N <= 0) return 0;
    const int64_t tiles_k = (K + 31) / 32, tiles_j = (N + 31) / 32;
    if (tiles_k * tiles_j > 0x7fffffff || ldbn < N) {
        set_error_msg("pack_neg_transpose_f64: bad shape");
        return MXLU_E_NOMEM;
    }
    hipLaunchKernelGGL(pack_neg_transpose_kernel, dim3((unsigned)(tiles_k * tiles_j)), dim3(256), 0,
                       s, K, N, B, ldb, Bn, ldbn, (int)tiles_k);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int gemm_f64_update(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                    const double *Bn, int64_t ldbn, double *C, int64_t ldc, hipStream_t s) {
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    if (!gemm_f64_update_ok(M, N, K, A, lda) || !Bn || ldbn < N || ldbn % 2 ||
        (uintptr_t)Bn % 16 || !C || ldc % 2 || (uintptr_t)C % 16) {
        set_error_msg("gemm_f64_update: shape, leading dimension or alignment not supported");
        return MXLU_E_NOMEM;
    }
    const int64_t tiles_m = M / BM, tiles_n = N / BN;
    if (tiles_m * tiles_n > 0x7fffffff) {
        set_error_msg("gemm_f64_update: grid too large");
        return MXLU_E_NOMEM;
    }
    hipLaunchKernelGGL(gemm_f64_direct_kernel, dim3((unsigned)(tiles_m * tiles_n)), dim3(256), 0,
                       s, M, N, K, A, lda, Bn, ldbn, C, ldc, (int)tiles_m, (int)tiles_n);
    MXLU_LAUNCH_CHECK();
    return 0;
}

int gemm_f64_nt_sub(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                    const double *B, int64_t ldb, double *C, int64_t ldc, bool accumulate,
                    hipStream_t s) {
    if (M <= 0 || N <= 0) return 0;
    const int64_t tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
    if (tiles_m * tiles_n > 0x7fffffff) {
        set_error_msg("gemm_f64_nt_sub: grid too large");
        return MXLU_E_NOMEM;
    }
    const dim3 grid((unsigned)(tiles_m * tiles_n));
    if (accumulate)
        hipLaunchKernelGGL((gemm_f64_sub_kernel<true, false>), grid, dim3(256), 0, s, M, N,
                           K, A, lda, B, ldb, C, ldc, (int)tiles_m, (int)tiles_n);
    else
        hipLaunchKernelGGL((gemm_f64_sub_kernel<true, true>), grid, dim3(256), 0, s, M, N,
                           K, A, lda, B, ldb, C, ldc, (int)tiles_m, (int)tiles_n);
    MXLU_LAUNCH_CHECK();
    return 0;
}

}  // namespace mxlu
