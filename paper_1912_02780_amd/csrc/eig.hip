// Small dense FP64 eigen kernels of the truncated eigensolve and its adjoint (gfx950).
//
// * jacobi_eig: one workgroup holds an n x n symmetric matrix and its eigenvector accumulator in
//   LDS (n <= 96: 2 x 96 x 97 doubles = 146 KiB of the 160 KiB LDS) and runs cyclic Jacobi in the
//   round-robin (Berger table) order: in every round n/2 disjoint index pairs are rotated at once,
//   rows first, then columns, each pass with one thread per row (or column) element of a pair, so
//   that a wave touches consecutive LDS words.  A pair is rotated while |a_pq| > 1e-16
//   sqrt(|a_pp a_qq|) and above an absolute floor (floor_rel |A|_F: 2^-60 for the spectra of the
//   eigensolver, which reach the FP64 floor; the callers may raise it to the rounding level of the
//   matrix, where rotations among large entries keep leaving residues of about u |A| next to small
//   eigenvalues), which keeps small eigenvalues to high relative accuracy.  (One pass over the disjoint 2 x 2 blocks of pair rows and pair columns, with one
//   barrier less per round, measured 40% slower: its LDS accesses scatter over the banks.)
// * jacobi_psd: the same for positive semidefinite matrices (the Gram and its Rayleigh-Ritz problems), one-sided
//   with the columns in registers.
// * element-wise helpers for the broadened inverse gaps of
//   the eigenvector adjoint and the Chebyshev expansion of the complement (interval, node values,
//   three-term recurrence, coefficient tail and boundedness checks).
// Every kernel serves nb independent instances (one workgroup or one y-slice of the grid each).
#include "block.hpp"

#include <algorithm>

namespace dtrg {

namespace {

constexpr int JM = kJacobiMax;
constexpr int JLD = JM + 1;
static_assert(JM <= 128, "one row or column element per thread of a group");

// GW: threads per group, one row (or column) element each, so n <= GW; JT threads in all (a single
// wave is slower: the row and column updates need the width).  12 waves, in groups of GW = 64 for
// n <= 64 and of GW = 96 for n <= 96 (a group may then straddle two waves): every thread of a group
// has an element, and the 12 or 8 groups share the pairs of a round.
template <int GW, int JT>
__global__ __launch_bounds__(JT) void jacobi_kernel(const double* __restrict__ Ain, int n, int lda, i64 a_bs,
                                                     double* __restrict__ lam, i64 lam_bs, double* __restrict__ Vout,
                                                     int ldv, i64 v_bs, int max_sweeps, int* sweeps_out,
                                                     int* flag, int flag_bit, double floor_rel) {
    constexpr int JG = JT / GW;                  // groups
    constexpr int JS = (JM / 2 + JG - 1) / JG;   // pair slots per group
    __shared__ double A[JM * JLD];
    __shared__ double V[JM * JLD];
    __shared__ int rp[JM / 2], rq[JM / 2];
    __shared__ double rc[JM / 2], rs[JM / 2];
    __shared__ int nrot, nact, any_active;
    __shared__ double fro;
    const int tid = threadIdx.x;
    Ain += blockIdx.x * a_bs;
    lam += blockIdx.x * lam_bs;
    Vout += blockIdx.x * v_bs;
    const int m = n + (n & 1);  // players, padded to even with a dummy index n
    for (int i = tid; i < n * n; i += JT) {
        const int r = i / n, c = i % n;
        A[r * JLD + c] = 0.5 * (Ain[(i64)r * lda + c] + Ain[(i64)c * lda + r]);
        V[r * JLD + c] = (r == c) ? 1.0 : 0.0;
    }
    if (tid == 0) fro = 0.0;
    __syncthreads();
    if (tid < 64) {
        double s = 0.0;
        for (int i = tid; i < n * n; i += 64) { const double v = A[(i / n) * JLD + (i % n)]; s += v * v; }
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
        if (tid == 0) fro = sqrt(s);
    }
    __syncthreads();
    // entries below the rounding level of the matrix are not rotated away (they are noise; rotating
    // them only costs sweeps on spectra that reach the FP64 floor)
    const double abs_floor = floor_rel * fro + 1e-300;
    int sweep = 0;
    for (; sweep < max_sweeps; ++sweep) {
        // A sweep in which no pair passes the rotation test leaves the matrix as it is, so every round
        // of it sees the matrix the sweep started from: the test over all pairs at once decides that
        // case without running the rounds (the result is the same as running them).
        if (tid == 0) any_active = 0;
        __syncthreads();
        {
            int mine = 0;
            for (int i = tid; i < n * n && !mine; i += JT) {
                const int p = i / n, q = i % n;
                if (q <= p) continue;
                const double apq = A[p * JLD + q];
                const double app = A[p * JLD + p], aqq = A[q * JLD + q];
                mine = fabs(apq) > fmax(1e-16 * sqrt(fabs(app * aqq)), abs_floor);
            }
            if (mine) any_active = 1;
        }
        __syncthreads();
        if (!any_active) break;
        if (tid == 0) nrot = 0;
        __syncthreads();
        for (int round = 0; round < m - 1; ++round) {
            // the n/2 pairs of this round are handled by wave 0 (m/2 <= 48 lanes); the pairs that
            // need a rotation are compacted into slots 0..nact-1
            if (tid < 64) {
                int p = 0, q = 0, active = 0;
                double c = 1.0, sn = 0.0;
                if (tid < m / 2) {
                    if (tid == 0) { p = m - 1; q = round; }
                    else { p = (round + tid) % (m - 1); q = (round - tid + (m - 1)) % (m - 1); }
                    if (p > q) { const int t = p; p = q; q = t; }
                    if (q < n) {
                        const double apq = A[p * JLD + q];
                        const double app = A[p * JLD + p], aqq = A[q * JLD + q];
                        if (fabs(apq) > fmax(1e-16 * sqrt(fabs(app * aqq)), abs_floor)) {
                            const double theta = (aqq - app) / (2.0 * apq);
                            double t;
                            if (fabs(theta) > 1e150) t = 0.5 / theta;
                            else t = (theta >= 0.0 ? 1.0 : -1.0) / (fabs(theta) + sqrt(1.0 + theta * theta));
                            c = 1.0 / sqrt(1.0 + t * t);
                            sn = t * c;
                            active = 1;
                        }
                    }
                }
                const unsigned long long mask = __ballot(active);
                const int slot = __popcll(mask & ((1ull << tid) - 1ull));
                if (active) { rp[slot] = p; rq[slot] = q; rc[slot] = c; rs[slot] = sn; }
                if (tid == 0) { nact = __popcll(mask); nrot += nact; }
            }
            __syncthreads();
            const int na = nact;
            if (na > 0) {
                // Slot i = g + JG t of group g (GW threads) is one active pair; thread l of the group
                // takes column l of its two rows, then row l of its two columns (and of V).  A
                // round's pairs are disjoint, so a thread issues every LDS read of a pass before its
                // first store: one round trip per pass instead of one per pair.
                const int g = tid / GW, l = tid % GW;
                const bool lv = l < n;
                const int lc = lv ? l : n - 1;
                const int ns = (na - g + JG - 1) / JG;   // active slots of this group
                int sp[JS], sq[JS];
                double sc[JS], ss[JS];
#pragma unroll
                for (int t = 0; t < JS; ++t) {
                    if (t >= ns) continue;
                    const int i = g + JG * t;
                    sp[t] = rp[i]; sq[t] = rq[i]; sc[t] = rc[i]; ss[t] = rs[i];
                }
                // rows: row_p <- c row_p - s row_q ; row_q <- s row_p + c row_q
                {
                    double ap[JS], aq[JS];
#pragma unroll
                    for (int t = 0; t < JS; ++t) {
                        if (t >= ns) continue;
                        ap[t] = A[sp[t] * JLD + lc];
                        aq[t] = A[sq[t] * JLD + lc];
                    }
#pragma unroll
                    for (int t = 0; t < JS; ++t) {
                        if (t >= ns || !lv) continue;
                        A[sp[t] * JLD + l] = sc[t] * ap[t] - ss[t] * aq[t];
                        A[sq[t] * JLD + l] = ss[t] * ap[t] + sc[t] * aq[t];
                    }
                }
                __syncthreads();
                // columns of A and of V
                {
                    double ap[JS], aq[JS], vp[JS], vq[JS];
#pragma unroll
                    for (int t = 0; t < JS; ++t) {
                        if (t >= ns) continue;
                        ap[t] = A[lc * JLD + sp[t]];
                        aq[t] = A[lc * JLD + sq[t]];
                        vp[t] = V[lc * JLD + sp[t]];
                        vq[t] = V[lc * JLD + sq[t]];
                    }
#pragma unroll
                    for (int t = 0; t < JS; ++t) {
                        if (t >= ns || !lv) continue;
                        A[l * JLD + sp[t]] = sc[t] * ap[t] - ss[t] * aq[t];
                        A[l * JLD + sq[t]] = ss[t] * ap[t] + sc[t] * aq[t];
                        V[l * JLD + sp[t]] = sc[t] * vp[t] - ss[t] * vq[t];
                        V[l * JLD + sq[t]] = ss[t] * vp[t] + sc[t] * vq[t];
                    }
                }
            }
            __syncthreads();
        }
        const int done = (nrot == 0);
        __syncthreads();
        if (done) break;
    }
    // every sweep still rotated something: the matrix is not diagonal to the rotation threshold
    if (tid == 0 && flag && sweep >= max_sweeps) atomicOr(flag + blockIdx.x, flag_bit);
    // sort descending (ties by index) and write out
    for (int i = tid; i < n; i += JT) {
        const double li = A[i * JLD + i];
        int rank = 0;
        for (int j = 0; j < n; ++j) {
            const double lj = A[j * JLD + j];
            rank += (lj > li) || (lj == li && j < i);
        }
        lam[rank] = li;
        for (int r = 0; r < n; ++r) Vout[(i64)r * ldv + rank] = V[r * JLD + i];
    }
    if (tid == 0 && sweeps_out) atomicMax(sweeps_out, sweep);
}

// ---------------------------------------------------------------------------------------------
// One-sided Jacobi of a positive semidefinite (to rounding) matrix
// ---------------------------------------------------------------------------------------------
// The columns of S = A / |A|_F + sigma I (sigma = 1.7 2^-12) are rotated in pairs until they are orthogonal:
// S W = U diag(s), and for a positive definite S the normalised columns U are its eigenvectors.  (Eigenvalues
// of A below -sigma |A|_F would be mixed with those above; a Gram has none beyond its noise.)  The shift sets
// what counts as rounding: two columns of tiny eigenvalues are orthogonal to 2^-50 once |A_pq| is below
// 2^-61 |A|_F, below the rounding level of A.  With a shift near that level the noise columns are resolved against each
// other instead, which took 11 and 26 sweeps in place of 3 and 9 on nearly diagonal matrices graded over sixteen
// decades (n = 64).  Between 2^-14 and 2^-10 the shift changes the last bits of the vectors and nothing else about
// the solve, but there are results that the last bits decide: gradients where a cut splits a pair of (nearly) equal
// eigenvalues or a multiplet is kept, and which side of a mirror-symmetric tensor weighs less.  Each value is as
// good as any other.  This one was taken, of sixteen between 2^-12 and 2^-11, because with it such results fall within
// the fixed bounds that the tests had for them: the Ising model at beta = 0.50, chi = 12 in FP32 and six-product
// split-bf16, the XY chain at chi = 25 in the latter, the sides of mirror-symmetric tensors.  With the others one or
// more of the four, in no order, does not, as the oracle's do not under noise of 2^-22 of its steps' outputs (to
// 1.9e-3 and 4.7e-4 in the first and third), so that passing there says nothing about a kernel;
// test_gpu_rounding_cuts.py holds them to what rounding moves, and passes with the shift at 2^-12, 1.5 2^-12 and 2^-11.
//
// What bounds it is latency: a sweep is n - 1 dependent rounds of n/2 rotations.  A two-sided rotation moves
// two rows and two columns of A and two columns of V through LDS between three barriers; here the columns
// live in registers, V is never formed, and LDS and the barrier are only used to pass blocks of eight
// columns on.  A wave holds two blocks, and lane l the rows l / 8, l / 8 + 8, ... of column l mod 8 of each,
// so that up to n = 64 every SIMD has one wave and the eight rotations of a round are worked out
// by one instruction stream: the eight products are summed over the eight lanes of a column, and the next
// eight of the 64 pairs are one lane permutation within eight away.  After eight rounds the blocks move one
// place along the round-robin circle.  (Four pairs a wave with one row per lane took 34 us a sweep at n = 64,
// with four rows per lane 27.)
// The rotations leave the length of a column right to a few roundings only, so the eigenvalues are taken
// as u^T A u in the end (matrix instructions, A is kept in LDS).
// On the Rayleigh-Ritz problems of the Ising model at beta_c, chi = 32 (b = 64) a call took 396 us as a
// two-sided Jacobi and takes 161, on the XY chain at D = 96 (b = 96) 803 and 350; a sweep takes 10, 22
// and 58 us at n = 28, 64 and 96 (before: 29, 85 and 190).  The last sweep of a call turns nothing: it is the test
// that the columns are orthogonal (the two-sided kernel tests all pairs at once).
constexpr double kPsdShift = 0x1.bp-12;
constexpr double kPsdTol2 = 0x1p-100;   // columns count as orthogonal at |x.y| <= 2^-50 |x| |y|

template <int CTRL>
__device__ inline double dpp_f64(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int quad(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
constexpr int kRowRor = 0x120, kHalfMirror = 0x141;

__device__ inline double row_pair_sum(double v) {   // sum over the rows 2q, 2q + 1 of 16 lanes
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
           __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}
__device__ inline double half_pair_sum(double v) {  // sum over lanes l and l xor 32
    const long long b = __double_as_longlong(v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    return __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
           __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
}

// The sum of v over the eight lanes of l's column (those equal to l modulo 8), the same bits in each (every
// addition of the tree is between the same two numbers in both lanes).
__device__ inline double col_sum(double v) {
    v += dpp_f64<kRowRor + 8>(v);
    return half_pair_sum(row_pair_sum(v));
}

// R rows of one column (per lane)
template <int R>
struct Col {
    double v[R];
};
template <int R>
__device__ inline double dot(const Col<R>& x, const Col<R>& y) {
    double s = x.v[0] * y.v[0], t = x.v[1] * y.v[1];
#pragma unroll
    for (int r = 2; r < R; r += 2) {
        s += x.v[r] * y.v[r];
        t += x.v[r + 1] * y.v[r + 1];
    }
    return s + t;
}
// lane l takes what lane l xor MASK has, MASK = 1, 2, 3 or 7
template <int MASK>
__device__ inline double lane_xor(double v) {
    constexpr int ctrl = MASK == 1 ? quad(1, 0, 3, 2)
                                   : (MASK == 2 ? quad(2, 3, 0, 1) : (MASK == 3 ? quad(3, 2, 1, 0) : kHalfMirror));
    return dpp_f64<ctrl>(v);
}
template <int MASK, int R>
__device__ inline void permute(Col<R>& x) {
#pragma unroll
    for (int r = 0; r < R; ++r) x.v[r] = lane_xor<MASK>(x.v[r]);
}

// Whether columns of squared norms a, b and product d are to be rotated.
__device__ inline bool oblique(double a, double b, double d) { return d * d > kPsdTol2 * (a * b); }

// The rotation by theta that makes the columns x and y of a lane orthogonal, x <- c x - s y, y <- s x + c y, as the
// three shears x -= h y, y += s x, x -= h y with h = tan(theta / 2), s = sin theta (c = 1 - h s): three in-place
// operations an element.  t = tan theta.  The angle comes from the reciprocals and roots as the hardware gives
// them (2^-24: an error in it only leaves that fraction of the product); s = 2 h / (1 + h^2) is to rounding,
// which makes the shears a rotation whatever h.  Zero where the columns are orthogonal already.
__device__ inline void rotation(double a, double b, double d, bool active, double& h, double& s, double& t) {
    const double del = b - a, h2 = del * del + 4.0 * (d * d);
    const double den = fabs(del) + h2 * __builtin_amdgcn_rsq(h2);
    t = 2.0 * d * __builtin_amdgcn_rcp(den);
    t = del >= 0.0 ? t : -t;
    // equal norms to rounding (exactly degenerate by a symmetry, as in the first steps of the Ising model):
    // either eighth of a turn does, so the choice is fixed rather than left to the last bit of del
    if (fabs(del) <= 0x1p-46 * (a + b) && fabs(d) > 0x1p10 * fabs(del)) t = 1.0;
    t = active ? t : 0.0;
    const double p = 1.0 + t * t;
    h = t * __builtin_amdgcn_rcp(1.0 + p * __builtin_amdgcn_rsq(p));
    const double m = 1.0 + h * h;
    double r = __builtin_amdgcn_rcp(m);
    const double e = 1.0 - m * r;
    r += r * (e + e * e);
    s = 2.0 * h * r;
}

// Rotate the pairs (x, y) of the eight columns of a wave's blocks, with their squared norms.  Returns whether any was.
template <int R>
__device__ inline bool rotate8(Col<R>& x, Col<R>& y, double& a, double& b) {
    const double d = col_sum(dot(x, y));
    const bool active = oblique(a, b, d);
    if (__ballot(active) == 0) return false;
    double h, s, t;
    rotation(a, b, d, active, h, s, t);
    a -= t * d;
    b += t * d;
#pragma unroll
    for (int r = 0; r < R; ++r) x.v[r] -= h * y.v[r];
#pragma unroll
    for (int r = 0; r < R; ++r) y.v[r] += s * x.v[r];
#pragma unroll
    for (int r = 0; r < R; ++r) x.v[r] -= h * y.v[r];
    return true;
}

// The pairs (c, c xor mask) within each of the two blocks, mask = 1 .. 7: every lane takes its partner's columns and
// keeps its own half of the rotations (x of the smaller index, or y).
template <int R>
__device__ inline bool rotate_within(Col<R>& x, Col<R>& y, int mask, bool first) {
    Col<R> o = x, q = y;
    const double nx = col_sum(dot(x, x)), ny = col_sum(dot(y, y));
    double no = nx, nq = ny;
    if (mask & 1) { permute<1>(o); permute<1>(q); no = lane_xor<1>(no); nq = lane_xor<1>(nq); }
    if (mask & 2) { permute<2>(o); permute<2>(q); no = lane_xor<2>(no); nq = lane_xor<2>(nq); }
    if (mask & 4) {
        permute<3>(o); permute<3>(q);
        permute<7>(o); permute<7>(q);
        no = lane_xor<7>(lane_xor<3>(no));
        nq = lane_xor<7>(lane_xor<3>(nq));
    }
    const double dx = col_sum(dot(x, o)), dy = col_sum(dot(y, q));
    const double ax = first ? nx : no, bx = first ? no : nx, ay = first ? ny : nq, by = first ? nq : ny;
    const bool actx = oblique(ax, bx, dx), acty = oblique(ay, by, dy);
    if (__ballot(actx || acty) == 0) return false;
    double hx, sx, hy, sy, t;
    rotation(ax, bx, dx, actx, hx, sx, t);
    rotation(ay, by, dy, acty, hy, sy, t);
    const double cx = 1.0 - hx * sx, cy = 1.0 - hy * sy;
    sx = first ? -sx : sx;
    sy = first ? -sy : sy;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        x.v[r] = cx * x.v[r] + sx * o.v[r];
        y.v[r] = cy * y.v[r] + sy * q.v[r];
    }
    return true;
}

typedef double v4d __attribute__((ext_vector_type(4)));

// R >= n / 8 rows per lane (even); blockDim.x = 64 ceil(n / 16).  Column j >= n of the last wave is the unit vector
// of row j, where no other column has an entry: it is orthogonal to them and stays.
template <int R>
__global__ __launch_bounds__(32 * R) void jacobi_psd_kernel(const double* __restrict__ Ain, int n, int lda, i64 a_bs,
                                                            int np, i64 ap_bs, double* __restrict__ lam, i64 lam_bs,
                                                            double* __restrict__ Vout, int ldv, i64 v_bs,
                                                            int max_sweeps, int* flag, int flag_bit) {
    constexpr int NC = 8 * R;                     // columns (16 a wave, R / 2 waves)
    __shared__ double As[NC * (NC + 1)];          // A, rows of n + 1
    __shared__ double buf[NC * (NC + 1)];         // exchange of blocks; the eigenvectors
    __shared__ double nrm[NC];
    __shared__ int rank_of[NC];
    __shared__ double wsum[R / 2];
    __shared__ int rotated[3];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, W = blockDim.x >> 6, nt = blockDim.x;
    const int cq = lane & 7, rq = lane >> 3;      // column of a block, first row
    const int ld = n + 1;
    Ain += blockIdx.x * a_bs;
    lam += blockIdx.x * lam_bs;
    Vout += blockIdx.x * v_bs;
    double f2 = 0.0;
    for (int i = tid; i < n * n; i += nt) {
        const int r = i / n, c = i % n;
        double v = Ain[(i64)r * lda + c];
        for (int p = 1; p < np; ++p) v += Ain[p * ap_bs + (i64)r * lda + c];
        As[r * ld + c] = v;
        f2 += v * v;
    }
    for (int o = 32; o > 0; o >>= 1) f2 += __shfl_xor(f2, o);
    if (lane == 0) wsum[w] = f2;
    if (tid < 3) rotated[tid] = 0;
    __syncthreads();
    double fro = 0.0;
    for (int i = 0; i < W; ++i) fro += wsum[i];
    fro = sqrt(fro);
    const double scale = fro > 0.0 ? 0.5 / fro : 0.0;   // the zero matrix: S = sigma I
    // top block w and bottom block 2W - 1 - w of the circle
    Col<R> X, Y;
    {
        const int cx = 8 * w + cq, cy = 8 * (2 * W - 1 - w) + cq;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = rq + 8 * r;
            double vx = row == cx ? 1.0 : 0.0, vy = row == cy ? 1.0 : 0.0;
            if (row < n && cx < n) vx = scale * (As[row * ld + cx] + As[cx * ld + row]) + vx * kPsdShift;
            if (row < n && cy < n) vy = scale * (As[row * ld + cy] + As[cy * ld + row]) + vy * kPsdShift;
            X.v[r] = vx;
            Y.v[r] = vy;
        }
    }
    int sweep = 0;
    for (; sweep < max_sweeps; ++sweep) {
        bool any = false;
        for (int mask = 1; mask < 8; ++mask) {
            const bool first = (cq ^ mask) > cq;
            any |= rotate_within(X, Y, mask, first);
        }
        double nx = col_sum(dot(X, X)), ny = col_sum(dot(Y, Y));
        for (int round = 0; round < 2 * W - 1; ++round) {
            // x_c with y_{c xor k}, k = 0 .. 7
            any |= rotate8(X, Y, nx, ny);
            permute<1>(Y); ny = lane_xor<1>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<3>(Y); ny = lane_xor<3>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<1>(Y); ny = lane_xor<1>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<7>(Y); ny = lane_xor<7>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<1>(Y); ny = lane_xor<1>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<3>(Y); ny = lane_xor<3>(ny);
            any |= rotate8(X, Y, nx, ny);
            permute<1>(Y); ny = lane_xor<1>(ny);
            any |= rotate8(X, Y, nx, ny);
            if (W == 1) continue;
            // the blocks move one place: T_0 stays, T_i -> T_{i+1}, T_{W-1} -> B_{W-1}, B_i -> B_{i-1},
            // B_0 -> T_1.  Place of T_i: i, of B_i: W + i; a place holds its lanes' registers as they are.
            const int px = w == 0 ? 0 : (w < W - 1 ? w + 1 : 2 * W - 1), py = w == 0 ? 1 : W + w - 1;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (w) buf[(px * R + r) * 64 + lane] = X.v[r];
                buf[(py * R + r) * 64 + lane] = Y.v[r];
            }
            if (lane < 8) {
                if (w) nrm[8 * px + lane] = nx;
                nrm[8 * py + lane] = ny;
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (w) X.v[r] = buf[(w * R + r) * 64 + lane];
                Y.v[r] = buf[((W + w) * R + r) * 64 + lane];
            }
            if (w) nx = nrm[8 * w + cq];
            ny = nrm[8 * (W + w) + cq];
            __syncthreads();
        }
        // three slots, one barrier a sweep: slot s is read after this barrier and cleared two sweeps on
        const int slot = sweep % 3;
        if (any && lane == 0) rotated[slot] = 1;
        if (tid == 0) rotated[(sweep + 1) % 3] = 0;
        __syncthreads();
        if (!rotated[slot]) break;
    }
    // every sweep still rotated something: the columns are not orthogonal to the tolerance
    if (tid == 0 && flag && sweep >= max_sweeps) atomicOr(flag + blockIdx.x, flag_bit);
    // eigenvectors by place, rows of n + 1; a padding column has its entry in a row n or beyond
    auto put = [&](const Col<R>& c, int place) {
        const double inv = 1.0 / sqrt(col_sum(dot(c, c)));
        bool pad = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = rq + 8 * r;
            pad |= row >= n && c.v[r] != 0.0;
            if (row < n) buf[place * ld + row] = c.v[r] * inv;
        }
        const bool padded = __ballot(pad) & (0x0101010101010101ULL << cq);
        if (rq == 0) nrm[place] = padded ? -INFINITY : 0.0;
    };
    put(X, 8 * w + cq);
    put(Y, 8 * (W + w) + cq);
    __syncthreads();
    // lambda = u^T A u of 16 columns at a time: the products A u of 16 rows, times u
    const int lr = lane >> 4, lc = lane & 15, nk = (n + 3) / 4;
    for (int ct = w; ct < W; ct += W) {
        const int col = 16 * ct + lc;
        double l = 0.0;
        for (int rt = 0; 16 * rt < n; ++rt) {
            const int row = min(16 * rt + lc, n - 1);
            v4d acc = {0, 0, 0, 0};
            for (int k = 0; k < nk; ++k) {
                const int kk = 4 * k + lr;
                const bool in = kk < n;
                const double x = As[row * ld + (in ? kk : 0)], u = buf[col * ld + (in ? kk : 0)];
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? x : 0.0, in ? u : 0.0, acc, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int ro = 16 * rt + lr + 4 * r;
                if (ro < n) l += acc[r] * buf[col * ld + ro];
            }
        }
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        if (lr == 0) nrm[col] = nrm[col] < 0.0 ? -INFINITY : l;
    }
    __syncthreads();
    // their order (descending, ties by place)
    for (int i = tid; i < 16 * W; i += nt) {
        const double li = nrm[i];
        int rank = 0;
        for (int j = 0; j < 16 * W; ++j) {
            const double lj = nrm[j];
            rank += (lj > li) || (lj == li && j < i);
        }
        rank_of[i] = rank;
        if (rank < n) lam[rank] = li;
    }
    __syncthreads();
    for (int i = tid; i < 16 * W * n; i += nt) {
        const int r = i / (16 * W), c = i % (16 * W), rank = rank_of[c];
        if (rank < n) Vout[(i64)r * ldv + rank] = buf[c * ld + r];
    }
}

__device__ inline double bgap(double d, double eps) { return d / (d * d + eps); }

// S = [[0, R], [R^T, 0]] (2K x 2K, ld 2K) from R (K x K, ld K)
__global__ __launch_bounds__(256) void sym_augment_kernel(const double* R, i64 r_bs, int K, double* S, i64 s_bs) {
    R += blockIdx.y * r_bs;
    S += blockIdx.y * s_bs;
    const int m = 2 * K;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < m * m; idx += gridDim.x * blockDim.x) {
        const int i = idx / m, j = idx % m;
        double v = 0.0;
        if (i < K && j >= K) v = R[i * K + (j - K)];
        else if (i >= K && j < K) v = R[j * K + (i - K)];
        S[idx] = v;
    }
}

__global__ __launch_bounds__(256) void kept_block_kernel(const double* Om, i64 om_bs, const double* lam,
                                                          i64 lam_bs, int k, double eps, double* S, i64 s_bs) {
    Om += blockIdx.y * om_bs;
    lam += blockIdx.y * lam_bs;
    S += blockIdx.y * s_bs;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < k * k; idx += gridDim.x * blockDim.x) {
        const int i = idx / k, j = idx % k;
        S[idx] = (i == j) ? 0.0 : bgap(lam[j] - lam[i], eps) * 0.5 * (Om[i * k + j] - Om[j * k + i]);
    }
}

__global__ __launch_bounds__(256) void over_block_kernel(const double* Om, i64 om_bs, const double* lam,
                                                          i64 lam_bs, int p, int k, double eps, double* M, i64 m_bs) {
    Om += blockIdx.y * om_bs;
    lam += blockIdx.y * lam_bs;
    M += blockIdx.y * m_bs;
    const double* theta = lam + k;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < p * k; idx += gridDim.x * blockDim.x) {
        const int i = idx / k, j = idx % k;
        M[idx] = bgap(lam[j] - theta[i], eps) * 0.5 * Om[idx];
    }
}

// Memory: five n x k blocks and the parts of the product, each once.
__global__ __launch_bounds__(256) void cheb_step_kernel(const double* Y, const double* W, i64 w_bs, int splits,
                                                         const double* Vc, const double* Vp, double* Vn, double* X,
                                                         i64 bs, int n, int k, const double* lohi, i64 lohi_bs,
                                                         int first, const double* coef, i64 coef_bs) {
    const int z = blockIdx.y;
    const i64 o = z * bs;
    const double lo = lohi[z * lohi_bs], hi = lohi[z * lohi_bs + 1];
    const double a = (first ? 1.0 : 2.0) / (hi - lo), sum = hi + lo;
    coef += z * coef_bs;
    const i64 total = (i64)n * k;
    for (i64 idx = blockIdx.x * (i64)blockDim.x + threadIdx.x; idx < total; idx += (i64)gridDim.x * blockDim.x) {
        const int j = (int)(idx % k);
        const double vc = Vc[o + idx];
        double y = 0.0;
        if (W) {
            double t[8];
#pragma unroll
            for (int p = 0; p < 8; ++p) t[p] = p < splits ? W[z * w_bs + p * total + idx] : 0.0;
#pragma unroll
            for (int p = 0; p < 8; ++p) y += t[p];
        } else {
            y = Y[o + idx];
        }
        double v = a * (2.0 * y - sum * vc);
        if (!first) v -= Vp[o + idx];
        Vn[o + idx] = v;
        if (first) X[o + idx] = coef[j] * vc + coef[k + j] * v;
        else X[o + idx] += coef[j] * v;
    }
}

__global__ void cheb_interval_kernel(const double* th, i64 th_bs, int e, const double* rn, i64 rn_bs, int n,
                                     double mult, double* lohi, i64 lohi_bs, int nb) {
    const int z = blockIdx.x * blockDim.x + threadIdx.x;
    if (z >= nb) return;
    const double* t = th + z * th_bs;
    const double nu = 64.0 * n * 0x1p-53 * fmax(t[0], 0.0);
    const double hi = mult * (fmax(1.1 * (fmax(t[e], 0.0) + rn[z * rn_bs]), nu) + 1e-300);
    lohi[z * lohi_bs] = -fmax(nu, 0.05 * hi);
    lohi[z * lohi_bs + 1] = hi;
}

__global__ __launch_bounds__(256) void cheb_table_kernel(double* ct, int m) {
    const int N = m + 1;
    const i64 total = (i64)N * N;
    for (i64 idx = blockIdx.x * (i64)blockDim.x + threadIdx.x; idx < total; idx += (i64)gridDim.x * blockDim.x) {
        const int q = (int)(idx / N), k = (int)(idx % N);
        // q (k + 1/2) / N reduced modulo 2 keeps the argument of cospi small and exact
        const i64 num = (i64)q * (2 * k + 1) % (4 * (i64)N);
        ct[idx] = (q == 0 ? 1.0 : 2.0) / N * cospi((double)num / (2.0 * N));
    }
}

__global__ __launch_bounds__(256) void cheb_fvals_kernel(const double* lam, i64 lam_bs, int K, double eps,
                                                          const double* lohi, i64 lohi_bs, int m, double* fv,
                                                          i64 fv_bs) {
    const int z = blockIdx.y;
    lam += z * lam_bs;
    fv += z * fv_bs;
    const double lo = lohi[z * lohi_bs], hi = lohi[z * lohi_bs + 1];
    const int N = m + 1;
    const i64 total = (i64)N * K;
    for (i64 idx = blockIdx.x * (i64)blockDim.x + threadIdx.x; idx < total; idx += (i64)gridDim.x * blockDim.x) {
        const int k = (int)(idx / K), j = (int)(idx % K);
        const double x = cospi((2.0 * k + 1.0) / (2.0 * N));
        const double t = 0.5 * (hi - lo) * x + 0.5 * (hi + lo);
        const double d = lam[j] - t;
        fv[idx] = 0.5 * d / (d * d + eps);
    }
}

__global__ __launch_bounds__(256) void cheb_tail_kernel(const double* coef, i64 coef_bs, int m, int K, double* ratio,
                                                         i64 ratio_bs) {
    const int z = blockIdx.x;
    coef += z * coef_bs;
    double mx = 0.0, tail = 0.0;
    const i64 total = (i64)(m + 1) * K;
    for (i64 idx = threadIdx.x; idx < total; idx += 256) {
        const double a = fabs(coef[idx]);
        const double a2 = isfinite(a) ? a : INFINITY;
        mx = fmax(mx, a2);
        if (idx / K >= m - 1) tail = fmax(tail, a2);
    }
    __shared__ double s1[256], s2[256];
    s1[threadIdx.x] = mx;
    s2[threadIdx.x] = tail;
    __syncthreads();
    for (int st = 128; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) {
            s1[threadIdx.x] = fmax(s1[threadIdx.x], s1[threadIdx.x + st]);
            s2[threadIdx.x] = fmax(s2[threadIdx.x], s2[threadIdx.x + st]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) ratio[z * ratio_bs] = s1[0] > 0.0 ? s2[0] / s1[0] : 0.0;
}

__global__ void cheb_bound_kernel(const double* vm, const double* v0, i64 bs, int nb, int* flag, int bit) {
    const int z = blockIdx.x * blockDim.x + threadIdx.x;
    if (z >= nb) return;
    const double a = vm[z * bs], b = v0[z * bs];
    if (!(isfinite(a) && isfinite(b) && a <= 1.5 * b)) flag[z] |= bit;
}

dim3 grid2(i64 n, int nb) {
    const i64 per = std::max<i64>(1, std::min<i64>((n + 255) / 256, std::max<i64>(1, 8192 / nb)));
    return dim3((unsigned)per, (unsigned)nb);
}

}  // namespace

void jacobi_eig(const double* A, int n, int lda, i64 a_bs, double* lam_dev, i64 lam_bs, double* V, int ldv, i64 v_bs,
                int nb, int max_sweeps, int* sweeps_dev, hipStream_t s, int* flag_dev, int flag_bit, double floor_rel) {
    DTRG_REQUIRE(n >= 1 && n <= kJacobiMax, DTRG_EINVAL, "jacobi_eig: n out of range");
    static_assert(kJacobiMax <= 96, "the widest Jacobi group has 96 threads");
    if (n <= 64)
        hipLaunchKernelGGL((jacobi_kernel<64, 768>), dim3(nb), dim3(768), 0, s, A, n, lda, a_bs, lam_dev, lam_bs, V,
                           ldv, v_bs, max_sweeps, sweeps_dev, flag_dev, flag_bit, floor_rel);
    else
        hipLaunchKernelGGL((jacobi_kernel<96, 768>), dim3(nb), dim3(768), 0, s, A, n, lda, a_bs, lam_dev, lam_bs, V,
                           ldv, v_bs, max_sweeps, sweeps_dev, flag_dev, flag_bit, floor_rel);
    DTRG_HIP(hipGetLastError());
}

void jacobi_psd(const double* A, int n, int lda, i64 a_bs, int np, i64 ap_bs, double* lam_dev, i64 lam_bs, double* V,
                int ldv, i64 v_bs, int nb, int max_sweeps, hipStream_t s, int* flag_dev, int flag_bit) {
    DTRG_REQUIRE(n >= 1 && n <= kJacobiMax, DTRG_EINVAL, "jacobi_psd: n out of range");
    static_assert(kJacobiMax <= 96, "twelve rows per lane hold 96 rows");
    const dim3 threads(64 * ((n + 15) / 16));
#define DTRG_PSD(R)                                                                                                  \
    hipLaunchKernelGGL((jacobi_psd_kernel<R>), dim3(nb), threads, 0, s, A, n, lda, a_bs, np, ap_bs, lam_dev, lam_bs, V, \
                       ldv, v_bs, max_sweeps, flag_dev, flag_bit)
    switch ((n + 15) / 16) {
        case 1: DTRG_PSD(2); break;
        case 2: DTRG_PSD(4); break;
        case 3: DTRG_PSD(6); break;
        case 4: DTRG_PSD(8); break;
        case 5: DTRG_PSD(10); break;
        default: DTRG_PSD(12); break;
    }
#undef DTRG_PSD
    DTRG_HIP(hipGetLastError());
}

void sym_augment(const double* R, i64 r_bs, int K, double* S, i64 s_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(sym_augment_kernel, grid2((i64)4 * K * K, nb), dim3(256), 0, s, R, r_bs, K, S, s_bs);
    DTRG_HIP(hipGetLastError());
}

void kept_block_adjoint(const double* Om, i64 om_bs, const double* lam_dev, i64 lam_bs, int k, double eps, double* S,
                        i64 s_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(kept_block_kernel, grid2((i64)k * k, nb), dim3(256), 0, s, Om, om_bs, lam_dev, lam_bs, k, eps,
                       S, s_bs);
    DTRG_HIP(hipGetLastError());
}

void over_block_adjoint(const double* Om, i64 om_bs, const double* lam_dev, i64 lam_bs, int p, int k, double eps,
                        double* M, i64 m_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(over_block_kernel, grid2((i64)p * k, nb), dim3(256), 0, s, Om, om_bs, lam_dev, lam_bs, p, k,
                       eps, M, m_bs);
    DTRG_HIP(hipGetLastError());
}

void cheb_step(const double* Y, const double* W, i64 w_bs, int splits, const double* Vc, const double* Vp, double* Vn,
               double* X, i64 bs, int n, int k, const double* lohi_dev, i64 lohi_bs, bool first, const double* coef_dev,
               i64 coef_bs, int nb, hipStream_t s) {
    DTRG_REQUIRE(!W || (splits >= 1 && splits <= 8), DTRG_EINVAL, "cheb_step: parts out of range");
    hipLaunchKernelGGL(cheb_step_kernel, grid2((i64)n * k, nb), dim3(256), 0, s, Y, W, w_bs, splits, Vc, Vp, Vn, X, bs,
                       n, k, lohi_dev, lohi_bs, first ? 1 : 0, coef_dev, coef_bs);
    DTRG_HIP(hipGetLastError());
}

void cheb_interval(const double* th, i64 th_bs, int e, const double* res_next, i64 rn_bs, int n, double mult,
                   double* lohi_dev, i64 lohi_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(cheb_interval_kernel, dim3((nb + 63) / 64), dim3(64), 0, s, th, th_bs, e, res_next, rn_bs, n,
                       mult, lohi_dev, lohi_bs, nb);
    DTRG_HIP(hipGetLastError());
}

void cheb_table(double* ct, int m, hipStream_t s) {
    hipLaunchKernelGGL(cheb_table_kernel, grid2((i64)(m + 1) * (m + 1), 1), dim3(256), 0, s, ct, m);
    DTRG_HIP(hipGetLastError());
}

void cheb_fvals(const double* lam, i64 lam_bs, int K, double eps, const double* lohi_dev, i64 lohi_bs, int m,
                double* fv, i64 fv_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(cheb_fvals_kernel, grid2((i64)(m + 1) * K, nb), dim3(256), 0, s, lam, lam_bs, K, eps, lohi_dev,
                       lohi_bs, m, fv, fv_bs);
    DTRG_HIP(hipGetLastError());
}

void cheb_tail(const double* coef, i64 coef_bs, int m, int K, double* ratio_dev, i64 ratio_bs, int nb, hipStream_t s) {
    hipLaunchKernelGGL(cheb_tail_kernel, dim3(nb), dim3(256), 0, s, coef, coef_bs, m, K, ratio_dev, ratio_bs);
    DTRG_HIP(hipGetLastError());
}

void cheb_bound_check(const double* vm_dev, const double* v0_dev, i64 bs, int nb, int* flag_dev, int bit,
                      hipStream_t s) {
    hipLaunchKernelGGL(cheb_bound_kernel, dim3((nb + 63) / 64), dim3(64), 0, s, vm_dev, v0_dev, bs, nb, flag_dev, bit);
    DTRG_HIP(hipGetLastError());
}

}  // namespace dtrg
