// Host-side launchers of the library's kernels (internal interface).
// Every launcher enqueues on stream `s` and returns 0 or an MXLU_E_* code.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <mutex>

namespace mxlu {

// C(M x N) -= A(M x K) * B(K x N), FP64, column-major.
int gemm_f64_sub(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                 const double *B, int64_t ldb, double *C, int64_t ldc, hipStream_t s);
// C(M x N) = (accumulate ? C : 0) - A(M x K) * B(N x K)^T.
// The trailing update A22 -= L21 U12 of the factorization with the
// register-direct kernel: full 128 x 128 tiles, K % 16 == 0, lda even and A
// 16-byte aligned (gemm_f64_update_ok; C must also be 16-byte aligned with
// ldc even); B comes as Bn = -U12^T, row-major with leading dimension
// ldbn >= N (even, 16-byte aligned), written by pack_neg_transpose_f64.
bool gemm_f64_update_ok(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda);
int pack_neg_transpose_f64(int64_t K, int64_t N, const double *B, int64_t ldb, double *Bn,
                           int64_t ldbn, hipStream_t s);
int gemm_f64_update(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                    const double *Bn, int64_t ldbn, double *C, int64_t ldc, hipStream_t s);
int gemm_f64_nt_sub(int64_t M, int64_t N, int64_t K, const double *A, int64_t lda,
                    const double *B, int64_t ldb, double *C, int64_t ldc, bool accumulate,
                    hipStream_t s);

// Exchange area of the multi-workgroup panel kernel (64-bit words, each a
// 32-bit payload tagged with a 32-bit column sequence number).
struct PanelExchange {
    uint64_t *slots;  // [2][kMaxGroups][4] candidates, then [2][kMaxGroups][kLeafW * 2] rows
    uint64_t *rowj;   // [2][kLeafW * 2] the current pivot row's old contents
    int *flags;       // [0]: first zero pivot (1-based), [1]: wait expired
    int group_cap;    // CUs a leaf may occupy (0: all); the LDS form puts one workgroup on each
    int spin_limit;   // looks after which a wait gives up (kSpinLimit; 0 by the test hook)
};
constexpr int kSpinLimit = 1 << 22;
constexpr int kLeafW = 32;        // columns factored by one leaf kernel
constexpr int kMaxGroups = 256;   // workgroups of one leaf kernel (<= CUs)

// Inputs of the leaf planner: the CUs the leaf may use (cap > 0: that many,
// else all `cus`), workgroups of the register form per CU (0: form not
// available), dynamic LDS per workgroup of the LDS form, element size.
struct LeafDevice {
    int cap, cus, occ_reg1, occ_reg2, elem_bytes;
    int64_t lds_budget;
};
enum { kLeafNone = 0, kLeafReg1 = 1, kLeafReg2 = 2, kLeafLds = 3 };
// Form (kLeaf*) and geometry (rows per group R, groups G) of an m-row leaf;
// host arithmetic only.
int leaf_plan(int64_t m, const LeafDevice &d, int64_t *R, int64_t *G);
// The current device's facts for the FP64 leaf with group cap `cap`.
int leaf_device_f64(int cap, LeafDevice *d);

// The leaf's wide form (panel_wide.h): up to 2048 rows on one workgroup, more
// on G = ceil(m / 1024).  *split: as of panel_leaf.
constexpr int kWideMaxGroups = 64;
template <typename T>
int panel_leaf_wide(int64_t m, int w, T *P, int64_t ldp, int64_t r0, int32_t *ipiv, int G,
                    const PanelExchange &ex, int *split, hipStream_t s);
// Interchanges of the leaf at column c0 (width w) of the m x kb panel P (whose
// column c0 is row and column rbase of the caller's numbering) on the panel's
// other columns, and those from column `split` on (split > 0) on the leaf's
// columns before it.
template <typename T>
int panel_leaf_swap(T *P, int64_t ldp, int64_t m, int64_t kb, int64_t c0, int w, int split,
                    const int32_t *ipiv, int64_t rbase, hipStream_t s);

// Factor the m x w (w <= kLeafW) leaf whose top-left element is P (leading
// dimension ldp) with partial pivoting.  r0 is the leaf's first row/column
// index within the caller's numbering: ipiv[r0 .. r0+w) receives r0 + the
// pivot row within the leaf; the column numbers r0 + j + 1 are the values of
// the workgroups' sequence flags, so they must grow from leaf to leaf.
// *split > 0: the leaf's columns before it still need the interchanges from
// column *split on (panel_leaf_swap).
template <typename T>
int panel_leaf(int64_t m, int w, T *P, int64_t ldp, int64_t r0, int32_t *ipiv,
               const PanelExchange &ex, int *split, hipStream_t s);

// Apply the interchanges ipiv[j0 .. j0+cnt) (rows >= j0 of a matrix with nrows
// rows, cnt <= 1024) to the columns c_begin + q (q < ncols, skipping
// [skip_begin, skip_begin + skip_len)).  An interchange row outside [j0 + t,
// nrows) counts as none.
template <typename T>
int swap_rows(T *A, int64_t lda, int64_t nrows, const int32_t *ipiv, int64_t j0, int cnt,
              int64_t c_begin, int64_t ncols, int64_t skip_begin, int64_t skip_len, hipStream_t s);
// The interchanges of every step applied to the columns left of its panel,
// deferred to after the factorization (each element moves once).  Scratch:
// maps of left_swap_map_ints ints, T of left_swap_rows x nb doubles.
int64_t left_swap_map_ints(int64_t n, int64_t nb);
int64_t left_swap_rows(int64_t n, int64_t nb);
int laswp_left_deferred_f64(double *A, int64_t lda, int64_t n, int64_t nb, const int32_t *ipiv,
                            int32_t *maps, double *T, hipStream_t s);

// C (M x N) -= A (M x K) B (K x N), tiles of 64 x 64 (gemm_panel.hip).
template <typename T>
int gemm_panel_sub(int64_t M, int64_t N, int64_t K, const T *A, int64_t lda, const T *B, int64_t ldb,
                   T *C, int64_t ldc, hipStream_t s);

// B(kb x ncols) = L^-1 B with L unit lower (kb x kb), kb <= 256.
template <typename T>
int trsm_llnu(int kb, int64_t ncols, const T *L, int64_t ldl, T *B, int64_t ldb, hipStream_t s);
class Scratch;
extern std::atomic<int> g_expire_waits;
// Zeroed exchange area of the panel kernels for a matrix of order n.
int alloc_panel_exchange(Scratch &scratch, int64_t n, PanelExchange *ex, hipStream_t s);
// GEPP of the m x kb panel P (recursive; leaves are panel_leaf<T>); element
// (0, 0) is row/column ibase of the caller's matrix, ipiv[ibase ..] receives
// caller-numbered rows; the interchanges are applied inside the panel only.
template <typename T>
int panel_factor(T *P, int64_t ldp, int64_t m, int64_t kb, int64_t ibase, int32_t *ipiv,
                 const PanelExchange &ex, hipStream_t s);

// perm[i] = original row at position i after the interchanges ipiv[0..n).
int perm_from_ipiv(int64_t n, const int32_t *ipiv, int32_t *perm, hipStream_t s);
// A chained solve with more workgroups than this, one for each XCD, hands its
// blocks out by tickets (see tri_chain_f64_kernel).
constexpr int kIdGroups = 8;

// State of a chained solve on the device, cleared by each launch for itself:
// blocks handed out, and whether a wait has expired.
struct TriSync {
    unsigned ticket, expired;
};
// A X = B (trans: A^T X = B) in place for nr <= 16 right-hand sides from the
// factors LU and the gather map perm of their interchanges; scratch: E, n x nr
// doubles (leading dimension lde), and *sync.
int tri_solve_f64(int64_t n, int nr, const double *LU, int64_t lda, const int32_t *perm, double *B,
                  int64_t ldb, int trans, double *E, int64_t lde, TriSync *sync, hipStream_t s);
// Solves of this kind on the current device whose waits have expired so far.
int tri_timeouts(int64_t *count);

// Streams of the mixed-precision factorization's look-ahead: `panel` factors
// the next panel while the rest of the trailing update runs on the caller's
// stream.  False at look-ahead depth 0 or when the streams are missing; on
// true the caller holds the process-wide look-ahead lock in *lk until its
// factorization has completed (the streams are shared by every call).
struct AheadStreams {
    hipStream_t panel = nullptr;
};
bool lp_ahead_streams(AheadStreams *out, std::unique_lock<std::mutex> *lk);

}  // namespace mxlu
