// Kernels of the block subspace iteration on n x b blocks (b <= 96, row-major, ld b), block.hip.
#pragma once

#include "common.hpp"

namespace dtrg {

// How an n x b block of nb instances is cut: the row kernels give each workgroup `rows` rows and leave one
// b x b partial product per workgroup (`chunks` of them); the Gram product cuts its inner index into
// `splits` parts of `kc` (splits = 1: it writes its output directly).
struct BlockCut {
    int n = 0, b = 0, nb = 1;
    int rows = 0, chunks = 0;
    int splits = 1, kc = 0;
    i64 vbs = 0;                 // instance stride of every n x b block
    i64 part_elems() const { return (i64)chunks * b * b; }
    i64 prod_elems() const { return splits > 1 ? (i64)splits * n * b : 1; }
};
BlockCut block_cut(int n, int b, int nb, i64 vbs);

// The shift of a new block X = Y + c V: c as given, or -f theta[b - 1] of the instance (theta not null).
struct BlockShift {
    double c = 0.0;
    const double* theta = nullptr;
    i64 th_bs = 0;
    double f = 0.5;
};

// Y = G V for the symmetric n x n matrices G (ld n): into Y, or (splits > 1) the parts of the sum into W
// (instance stride w_bs).
void block_product(const double* G, i64 g_bs, const double* V, double* Y, double* W, i64 w_bs, const BlockCut& q,
                   hipStream_t s);
// part = partial V^T Y; with parts of Y in W (not null) their sum is formed and written to Y.
void block_vty(const double* V, double* Y, const double* W, i64 w_bs, double* part, i64 p_bs, const BlockCut& q,
               hipStream_t s);
// Vo = V Z, Yo = Y Z (Z b x b); rpart[chunk][j] = partial sum of (Yo - theta_j Vo)^2 of column j; part (not
// null) = partial X^T X of the next block X = Yo + c Vo.
void block_rotate(const double* V, const double* Y, double* Vo, double* Yo, const double* Z, i64 z_bs,
                  const double* theta, i64 th_bs, const BlockShift& sh, double* rpart, i64 r_bs, double* part,
                  i64 p_bs, const BlockCut& q, hipStream_t s);
// res[j] = sqrt of the sum of rpart over the chunks, j < b
void block_residuals(const double* rpart, i64 r_bs, double* res, i64 res_bs, const BlockCut& q, hipStream_t s);
// part = partial X^T X.  V null: X is the block itself.  Otherwise X = Y + c V with Y in X (or, W not null, the
// parts of Y in W), written back to X.
void block_gram(double* X, const double* V, const double* W, i64 w_bs, const BlockShift& sh, double* part, i64 p_bs,
                const BlockCut& q, hipStream_t s);
// Out = X R (R b x b upper triangular); Out may be X.  V not null: X + c V in place of X.  Columns k with
// tiny[k] != 0 (tiny not null) are replaced by hash noise of unit scale before the product, and with drop those
// of Out that block_chol dropped after it.  part (not null):
// partial Out^T Out, not formed for instances with nogram[i] != 0.  Instances with skip[i] != 0 are left as
// they are.
void block_mult(const double* X, const double* V, const BlockShift& sh, const double* R, i64 r_bs, const int* tiny,
                i64 t_bs, bool drop, uint64_t seed, double* Out, double* part, i64 p_bs, const int* skip,
                const int* nogram, const BlockCut& q, hipStream_t s);
// Sum the chunks of part into the first where there are more than a consumer adds up itself; returns how many
// are left.  skip as in block_mult.
int block_reduce(double* part, i64 p_bs, const int* skip, const BlockCut& q, hipStream_t s);
// R^{-1} (b x b, upper triangular, zero below inside the diagonal tiles of 16) of the Cholesky factor of
// S + shift_rel tr(S) I, S the sum of np partials.  scaled: S is first scaled to a unit diagonal, D^{-1} S D^{-1},
// and D^{-1} R^{-1} returned; columns of norm at most 1e-30 of the largest count as absent (tiny[k] = 1, unit
// row and column in S).  near (not null): near[i] = 1 if S_i (scaled, and no column absent) is within near_tol of the
// identity in the Frobenius norm, and then there is no shift.  drop (not scaled): columns that depend on the ones
// before them (a pivot within rounding of zero) are left out and marked for block_mult.  flag |= 2 on such a pivot, or a
// non-positive one.  Instances with skip[i] != 0 are left as they are, with near[i] = 1.
void block_chol(const double* part, i64 p_bs, int np, int b, int nb, double shift_rel, bool scaled, double* Rinv,
                i64 r_bs, int* flag, const int* skip, int* near, double near_tol, int* tiny, i64 t_bs, bool drop,
                hipStream_t s);

// C = G V for the Gram in Kronecker form G[(a,c)][(b,d)] = sum_jk A[a][b][jk] B[c][d][jk] / s (kron.hip), V and C
// X^2 x w with ld w; W holds up to 16 partial sums of C.  Only sizes that kron_product_fits.
bool kron_product_fits(int X, int YY);
void kron_product(const double* A, i64 a_bs, const double* B, i64 b_bs, const double* V, i64 v_bs, double* W, i64 w_bs,
                  const double* s_dev, i64 s_bs, double* C, i64 c_bs, int X, int w, int nb, hipStream_t s);

// Full symmetric eigendecomposition of an n x n matrix (n <= kJacobiMax) that is positive semidefinite to
// rounding (a Gram or its Rayleigh-Ritz matrix), by one-sided Jacobi, one workgroup per instance (eig.hip):
// eigenvalues descending into lam_dev[0..n), to rounding of |A|_F, eigenvectors as the columns of V (ld ldv),
// orthonormal to rounding.  A is the sum of np partials, ap_bs apart.  flag_dev (nullable): flag_dev[i] |=
// flag_bit when instance i still rotated in its last allowed sweep.
void jacobi_psd(const double* A, int n, int lda, i64 a_bs, int np, i64 ap_bs, double* lam_dev, i64 lam_bs, double* V,
                int ldv, i64 v_bs, int nb, int max_sweeps, hipStream_t s, int* flag_dev = nullptr, int flag_bit = 0);

}  // namespace dtrg
