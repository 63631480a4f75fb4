// The block subspace iteration's own kernels (gfx950): products, Rayleigh-Ritz rotations and CholeskyQR of
// n x b blocks, b <= 96, FP64 matrix instructions.
//
// These products are small (an iteration at n = 1024, b = 64 is 0.2 GFLOP) and form one dependent chain, so
// launches, memory round trips and the few workgroups of a general contraction bound them, not its rate.
// Here one workgroup takes a strip of rows with one wave per 16 columns, and what follows in the chain is
// done on the strip while it is in registers: the accumulator of v_mfma_f64_16x16x4f64 (register r of lane
// l: row l / 16 + 4 r, column l mod 16) is also its operand layout for the r-th step of 4 rows, so the
// b x b product of a freshly computed strip with itself needs one exchange of the strip through LDS
// and no memory.  Each workgroup leaves a b x b partial that the next kernel (or block_reduce) adds up.
#include "block.hpp"

#include <algorithm>
#include <type_traits>
#include <utility>

namespace dtrg {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ inline v4d mma(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

constexpr int kMaxTiles = 6;          // b <= 96
constexpr int kConsumerParts = 8;     // partials a single workgroup adds up itself
constexpr int kMaxSplits = 8;         // parts of a product's inner index
constexpr double kDropped = -1.0;     // in place of a diagonal entry of R^{-1} (positive): noise for this column

__device__ inline double shift_of(const BlockShift& sh, int z, int b) {
    return sh.theta ? -sh.f * sh.theta[z * sh.th_bs + b - 1] : sh.c;
}

__device__ inline uint64_t mix64(uint64_t z) {
    z += 0x9e3779b97f4a7c15ULL;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ULL;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebULL;
    return z ^ (z >> 31);
}

// hash noise of element `at` of a block, uniform in (-unit, unit)
__device__ inline double noise_of(uint64_t seed, i64 at, double unit) {
    const uint64_t h = mix64(seed ^ mix64((uint64_t)at));
    return ((double)(h >> 11) * (2.0 / 9007199254740992.0) - 1.0) * unit;
}

// Where a lane sits: lr = lane / 16, lc = lane mod 16, column tile w.
struct Lane {
    int lane, w, lr, lc, col;
    bool ok;
    __device__ Lane(int b) {
        lane = threadIdx.x & 63;
        w = threadIdx.x >> 6;
        lr = lane >> 4;
        lc = lane & 15;
        col = 16 * w + lc;
        ok = col < b;
    }
};

// acc[i] += (tile i of the strip left in sh)^T (this wave's tile y): 16 rows
template <int T>
__device__ inline void strip_product(v4d* acc, const double (*sh)[4][64], const double* y, int lane) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int i = 0; i < T; ++i) acc[i] = mma(sh[i][r][lane], y[r], acc[i]);
}

template <int T>
__device__ inline void store_part(const v4d* acc, double* part, int chunk, int b, const Lane& L) {
    double* o = part + (i64)chunk * b * b;
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = 16 * i + L.lr + 4 * r;
            if (row < b && L.ok) o[row * b + L.col] = acc[i][r];
        }
}

// --- Y = G V -----------------------------------------------------------------------------------
// 32 rows a workgroup, inner index split over blockIdx.y.  G is symmetric: its rows are read as columns, so
// that a load of 4 inner indices x 16 rows is four whole 128-byte lines.  Eight steps of loads are in flight
// under the products of the eight before.
template <int T>
__global__ __launch_bounds__(64 * T) void block_product_kernel(const double* __restrict__ G, i64 g_bs,
                                                               const double* __restrict__ V, i64 vbs, double* Y,
                                                               double* W, i64 w_bs, int n, int b, int kc) {
    constexpr int U = 8;
    const Lane L(b);
    const int z = blockIdx.z, row0 = blockIdx.x * 32, k0 = blockIdx.y * kc, k1 = min(n, k0 + kc);
    G += z * g_bs;
    V += z * vbs;
    const int ra = min(row0 + L.lc, n - 1), rb = min(row0 + 16 + L.lc, n - 1);
    const int cv = L.ok ? L.col : 0;
    v4d acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
    double a0[U], a1[U], v[U];
    auto load = [&](int k) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kk = k + 4 * u + L.lr;
            const bool in = kk < k1;
            const i64 kr = in ? kk : 0;
            const double x0 = G[kr * n + ra], x1 = G[kr * n + rb], y = V[kr * b + cv];
            a0[u] = in ? x0 : 0.0;
            a1[u] = in ? x1 : 0.0;
            v[u] = in && L.ok ? y : 0.0;
        }
    };
    load(k0);
    for (int k = k0; k < k1; k += 4 * U) {
        double c0[U], c1[U], cw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { c0[u] = a0[u]; c1[u] = a1[u]; cw[u] = v[u]; }
        if (k + 4 * U < k1) load(k + 4 * U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            acc0 = mma(c0[u], cw[u], acc0);
            acc1 = mma(c1[u], cw[u], acc1);
        }
    }
    double* o = W ? W + z * w_bs + (i64)blockIdx.y * n * b : Y + z * vbs;
    if (!L.ok) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = row0 + L.lr + 4 * r;
        if (row < n) o[(i64)row * b + L.col] = acc0[r];
        if (row + 16 < n) o[(i64)(row + 16) * b + L.col] = acc1[r];
    }
}

// --- V^T Y, and X^T X of X = Y + c V --------------------------------------------------------------
// GRAM: the left operand is the block X itself.
template <int T, bool GRAM>
__global__ __launch_bounds__(64 * T) void block_vty_kernel(const double* V, double* Y, i64 vbs,
                                                           const double* __restrict__ W, i64 w_bs, int splits,
                                                           BlockShift shift, double* __restrict__ part, i64 p_bs,
                                                           int n, int b, int rows) {
    __shared__ double sh[2][T][4][64];
    const Lane L(b);
    const int z = blockIdx.y, r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
    if (V) V += z * vbs;
    Y += z * vbs;
    if (W) W += z * w_bs;
    const double c = GRAM && V ? shift_of(shift, z, b) : 0.0;
    const bool store = W || (GRAM && V);
    v4d acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = v4d{0, 0, 0, 0};
    double y[4], v[4];
    // What lies outside the strip or past the last part is read from inside and multiplied by zero: a select on a
    // loaded value would make each load wait for the one before (8 loads of the parts took four times their
    // latency).
    const double cm = L.ok ? 1.0 : 0.0;
    const int cc = L.ok ? L.col : 0;
    double pm[kMaxSplits];
    i64 po[kMaxSplits];
#pragma unroll
    for (int p = 0; p < kMaxSplits; ++p) {
        pm[p] = p < splits ? 1.0 : 0.0;
        po[p] = (i64)(p < splits ? p : 0) * n * b;
    }
    auto load = [&](int rb) {
        double m[4];
        i64 idx[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = rb + 4 * r + L.lr;
            m[r] = row < r1 ? cm : 0.0;
            idx[r] = (i64)min(row, r1 - 1) * b + cc;
        }
        if (W) {
            double t[4][kMaxSplits];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int p = 0; p < kMaxSplits; ++p) t[r][p] = W[po[p] + idx[r]];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double s = 0.0;
#pragma unroll
                for (int p = 0; p < kMaxSplits; ++p) s += t[r][p] * pm[p];
                y[r] = s;
            }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = Y[idx[r]];
        }
        if (V) {
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = V[idx[r]];
            if (GRAM)
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r] += c * v[r];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            y[r] *= m[r];
            v[r] = V ? v[r] * m[r] : 0.0;
        }
    };
    load(r0);
    int buf = 0;
    for (int rb = r0; rb < r1; rb += 16, buf ^= 1) {
        double cur[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            cur[r] = y[r];
            sh[buf][L.w][r][L.lane] = GRAM ? y[r] : v[r];
            const int row = rb + 4 * r + L.lr;
            if (store && row < r1 && L.ok) Y[(i64)row * b + L.col] = y[r];
        }
        __syncthreads();
        if (rb + 16 < r1) load(rb + 16);
        strip_product<T>(acc, sh[buf], cur, L.lane);
    }
    store_part<T>(acc, part + z * p_bs, blockIdx.x, b, L);
}

// --- V Z, Y Z, residuals, Gram of the next block --------------------------------------------------
template <int T>
__global__ __launch_bounds__(64 * T) void block_rotate_kernel(const double* __restrict__ V, const double* __restrict__ Y,
                                                              double* __restrict__ Vo, double* __restrict__ Yo, i64 vbs,
                                                              const double* __restrict__ Z, i64 z_bs,
                                                              const double* __restrict__ theta, i64 th_bs,
                                                              BlockShift shift, double* __restrict__ rpart, i64 r_bs,
                                                              double* __restrict__ part, i64 p_bs, int n, int b,
                                                              int rows) {
    __shared__ double sh[2][T][4][64];
    const Lane L(b);
    const int z = blockIdx.y, r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
    V += z * vbs; Y += z * vbs; Vo += z * vbs; Yo += z * vbs;
    Z += z * z_bs;
    const double c = part ? shift_of(shift, z, b) : 0.0;
    const double th = L.ok ? theta[z * th_bs + L.col] : 0.0;
    double zf[4 * T];
#pragma unroll
    for (int k = 0; k < 4 * T; ++k) {
        const int row = 4 * k + L.lr;
        const bool in = row < b && L.ok;
        const double x = Z[in ? row * b + L.col : 0];
        zf[k] = in ? x : 0.0;
    }
    v4d acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = v4d{0, 0, 0, 0};
    double rs = 0.0;
    int buf = 0;
    for (int rb = r0; rb < r1; rb += 16, buf ^= 1) {
        double av[4 * T], ay[4 * T];
        const int row = rb + L.lc;
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) {
            const int col = 4 * k + L.lr;
            const bool in = row < r1 && col < b;
            const i64 idx = in ? (i64)row * b + col : 0;
            const double x = V[idx], y = Y[idx];
            av[k] = in ? x : 0.0;
            ay[k] = in ? y : 0.0;
        }
        v4d pv = {0, 0, 0, 0}, py = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) {
            pv = mma(av[k], zf[k], pv);
            py = mma(ay[k], zf[k], py);
        }
        double x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ro = rb + L.lr + 4 * r;
            if (ro < r1 && L.ok) {
                Vo[(i64)ro * b + L.col] = pv[r];
                Yo[(i64)ro * b + L.col] = py[r];
            }
            const double e = py[r] - th * pv[r];
            rs += e * e;
            x[r] = py[r] + c * pv[r];
        }
        if (part) {
#pragma unroll
            for (int r = 0; r < 4; ++r) sh[buf][L.w][r][L.lane] = x[r];
            __syncthreads();
            strip_product<T>(acc, sh[buf], x, L.lane);
        }
    }
    rs += __shfl_xor(rs, 16);
    rs += __shfl_xor(rs, 32);
    if (L.lr == 0 && L.ok) rpart[z * r_bs + (i64)blockIdx.x * b + L.col] = rs;
    if (part) store_part<T>(acc, part + z * p_bs, blockIdx.x, b, L);
}

__global__ __launch_bounds__(128) void block_residual_kernel(const double* __restrict__ rpart, i64 r_bs, int chunks,
                                                             int b, double* __restrict__ res, i64 res_bs) {
    const int j = threadIdx.x, z = blockIdx.x;
    if (j >= b) return;
    const double* p = rpart + z * r_bs + j;
    double s = 0.0;
    for (int c = 0; c < chunks; c += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = c + u < chunks ? p[(i64)(c + u) * b] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += v[u];
    }
    res[z * res_bs + j] = sqrt(s);
}

// --- X R, Gram of the result ----------------------------------------------------------------------
// R is upper triangular: column tile w takes the first 16 (w + 1) columns of X.  Out may be X: every wave has
// the strip in registers before the barrier, and stores its tile after it.
template <int T>
__global__ __launch_bounds__(64 * T) void block_mult_kernel(const double* X, const double* V, i64 vbs,
                                                            BlockShift shift, const double* __restrict__ R, i64 r_bs,
                                                            const int* __restrict__ tiny, i64 t_bs, int drop,
                                                            uint64_t seed,
                                                            double* Out, double* __restrict__ part, i64 p_bs,
                                                            const int* __restrict__ skip,
                                                            const int* __restrict__ nogram, int n, int b, int rows) {
    __shared__ double sh[2][T][4][64];
    const Lane L(b);
    const int z = blockIdx.y, r0 = blockIdx.x * rows, r1 = min(n, r0 + rows);
    if (skip && skip[z]) return;
    const bool gram = part && !(nogram && nogram[z]);
    X += z * vbs;
    Out += z * vbs;
    if (V) V += z * vbs;
    R += z * r_bs;
    if (tiny) tiny += z * t_bs;
    if (z) seed = mix64(seed ^ (0x5bd1e995ULL + z));
    const double c = V ? shift_of(shift, z, b) : 0.0;
    const double unit = 1.0 / sqrt((double)n);
    double rf[4 * T];
#pragma unroll
    for (int k = 0; k < 4 * T; ++k) {
        const int row = 4 * k + L.lr;
        const bool in = k < 4 * (L.w + 1) && row < b && L.ok;
        const double x = R[in ? row * b + L.col : 0];
        rf[k] = in ? x : 0.0;
    }
    unsigned noise = 0;
    if (tiny) {
        int t[4 * T];
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) t[k] = tiny[min(4 * k + L.lr, b - 1)];
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) noise |= (unsigned)(t[k] != 0 && 4 * k + L.lr < b) << k;
    }
    const bool noisy = __ballot(noise != 0) != 0;
    // a dropped column: its mark is with the lane that has the diagonal entry (row 4 k + lr, lr = lc mod 4)
    bool fill = false;
    if (drop) {
        bool mark = false;
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) mark |= 4 * k + L.lr == L.col && rf[k] == kDropped;
        fill = (__ballot(mark) & (0x0001000100010001ULL << L.lc)) != 0;
    }
    v4d acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = v4d{0, 0, 0, 0};
    int buf = 0;
    for (int rb = r0; rb < r1; rb += 16, buf ^= 1) {
        // all columns, and clamped in place of selected (rows at or past r1 are not stored and get no part in
        // the Gram, columns at or past b meet zeros of R): the loads are all in flight together
        double a[4 * T];
        const int row = rb + L.lc;
        const double m = row < r1 ? 1.0 : 0.0;
        const i64 at = (i64)min(row, r1 - 1) * b;
#pragma unroll
        for (int k = 0; k < 4 * T; ++k) a[k] = X[at + min(4 * k + L.lr, b - 1)];
        if (V) {
#pragma unroll
            for (int k0 = 0; k0 < 4 * T; k0 += 8) {
                double y[8];
#pragma unroll
                for (int u = 0; u < 8 && k0 + u < 4 * T; ++u) y[u] = V[at + min(4 * (k0 + u) + L.lr, b - 1)];
#pragma unroll
                for (int u = 0; u < 8 && k0 + u < 4 * T; ++u) a[k0 + u] += c * y[u];
            }
        }
        if (noisy) {
#pragma unroll
            for (int k = 0; k < 4 * T; ++k)
                if (noise >> k & 1) {
                    a[k] = noise_of(seed, at + 4 * k + L.lr, unit);
                }
        }
        v4d p0 = {0, 0, 0, 0}, p1 = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < T; ++j) {
            if (j > L.w) continue;
#pragma unroll
            for (int k = 4 * j; k < 4 * j + 4; k += 2) {
                p0 = mma(a[k] * m, rf[k], p0);
                p1 = mma(a[k + 1] * m, rf[k + 1], p1);
            }
        }
        double x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            x[r] = p0[r] + p1[r];
            if (fill) {
                const int ro = rb + L.lr + 4 * r;
                x[r] = ro < r1 ? noise_of(seed, (i64)ro * b + L.col, unit) : 0.0;
            }
            if (gram) sh[buf][L.w][r][L.lane] = x[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int ro = rb + L.lr + 4 * r;
            if (ro < r1 && L.ok) Out[(i64)ro * b + L.col] = x[r];
        }
        if (gram) strip_product<T>(acc, sh[buf], x, L.lane);
    }
    if (gram) store_part<T>(acc, part + z * p_bs, blockIdx.x, b, L);
}

__global__ __launch_bounds__(256) void block_reduce_kernel(double* part, i64 p_bs, int chunks, int bb,
                                                           const int* __restrict__ skip) {
    if (skip && skip[blockIdx.y]) return;
    double* p = part + blockIdx.y * p_bs;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= bb) return;
    double s = 0.0;
    for (int c = 0; c < chunks; c += 16) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = c + u < chunks ? p[(i64)(c + u) * bb + i] : 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) s += v[u];
    }
    p[i] = s;
}

// --- Cholesky factor and its inverse -----------------------------------------------------------------
// Four waves, tiles of 16: the chain is what bounds it (with one barrier per column or pair of columns it
// is LDS round trip, barrier and reciprocal root, b times over).  A diagonal tile is factored and inverted
// by one wave without a barrier (a row of the tile per lane, the same in the four rows of 16 lanes; pivots
// and multipliers are broadcast within a row of lanes), and everything else is products with matrix
// instructions: L_ik = A_ik D_k^T and X_kj = D_k X_kj with D_k the inverse of the diagonal factor, then
// A_ij -= L_ik L_jk^T and X_ij -= L_ik X_kj, X = L^{-1} being built beside L.  The update of the next
// diagonal tile and its factorisation run on wave 0 under the other waves' updates.
// b = 28, 64, 96: 9, 17, 31 us a call, launch included (12, 28, 51 with two columns eliminated per barrier).
//
// A Gram of numerically low rank (the Ising model deep in a phase) gives blocks of fewer directions than columns.
// The shift carries the first pass over that; in the plain passes after it a column that depends on the ones
// before it has a pivot that is rounding only, of either sign, and its reciprocal root would fill the tiles
// after it with infinities.  Where the caller asks for it, such a column is dropped instead: its row of L^{-1} and
// its column of L are zero but for the mark kDropped on the diagonal, and block_mult puts hash noise in its place,
// which the next pass orthonormalises.  kDependent: that far below the column's squared norm the pivot is rounding (96
// columns: 2^-53 x 96 = 2^-46.4, and the explicit inverses of the tiles add to it).
constexpr double kDependent = 0x1p-42;

__device__ inline void wave_sync() {   // LDS stores of this wave's lanes before loads by others of them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline double rsqrt64(double d) {
    double r = __builtin_amdgcn_rsq(d);
    r *= 1.5 - 0.5 * d * r * r;
    r *= 1.5 - 0.5 * d * r * r;
    return r;
}

template <int J>
__device__ inline double row_bcast(double v) {   // the value of lane J of this row of 16 lanes
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, 0x150 + J, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), 0x150 + J, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// column K of a 16 x 16 tile: row i = lane mod 16 in a, columns 4 (lane / 16) + m of the inverse in x.  Bit K of bad:
// its pivot is not positive (DROP: above `least` of row K) or not finite.
template <bool DROP, int K, int... J>
__device__ inline void diag_column(double (&a)[16], double (&x)[4], int i, double least, unsigned& bad,
                                   std::integer_sequence<int, J...>) {
    double d = row_bcast<K>(a[K]);
    const bool no = !(d > (DROP ? row_bcast<K>(least) : 0.0)) || !isfinite(d);
    if (no) { bad |= 1u << K; d = 1e-300; }
    const double r = DROP && no ? 0.0 : rsqrt64(d);
    const double l = i > K ? a[K] * r : 0.0;
    ((a[K + 1 + J] -= l * row_bcast<K + 1 + J>(l)), ...);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const double xk = row_bcast<K>(x[m]) * r;
        x[m] = i == K ? xk : x[m] - l * xk;
    }
}
template <bool DROP, int... K>
__device__ inline void diag_columns(double (&a)[16], double (&x)[4], int i, double least, unsigned& bad,
                                    std::integer_sequence<int, K...>) {
    (diag_column<DROP, K>(a, x, i, least, bad, std::make_integer_sequence<int, 15 - K>()), ...);
}

// DROP: not scaled, and dependent columns are dropped
template <int T, bool DROP>
__global__ __launch_bounds__(256) void block_chol_kernel(const double* __restrict__ part, i64 p_bs, int np, int b,
                                                         double shift, int scaled, double* __restrict__ Rinv,
                                                         i64 r_bs, int* flag, const int* skip, int* near,
                                                         double near_tol, int* tiny, i64 t_bs) {
    // rows 4 modulo 32 doubles apart: the 16 rows x 4 columns of an operand read fall on different banks
    constexpr int N = 16 * T, LD = N <= 36 ? 36 : (N <= 68 ? 68 : 100);
    __shared__ double A[N * LD], X[N * LD];
    __shared__ double inv[N], dist[4];   // inv, DROP: the least pivots
    __shared__ unsigned gone_of[T];      // DROP: the dropped columns of each diagonal tile
    const int tid = threadIdx.x, z = blockIdx.x, lane = tid & 63, w = tid >> 6, lr = lane >> 4, lc = lane & 15;
    const int ty = tid >> 4, tx = tid & 15;
    if (skip && skip[z]) {
        if (near && tid == 0) near[z] = 1;
        return;
    }
    part += z * p_bs;
    Rinv += z * r_bs;
    if (tiny) tiny += z * t_bs;
    const int bb = b * b;
    auto sum = [&](int i) {
        double v[kConsumerParts], s = 0.0;
#pragma unroll
        for (int u = 0; u < kConsumerParts; ++u) v[u] = u < np ? part[(i64)u * bb + i] : 0.0;
#pragma unroll
        for (int u = 0; u < kConsumerParts; ++u) s += v[u];
        return s;
    };
    if (scaled) {
        // column norms, and what counts as an absent column (every wave has all of them for the largest)
        double mx = 0.0, mine = 1.0;
        for (int j = lane; j < b; j += 64) {
            const double d = sum(j * b + j);
            mx = fmax(mx, d);
            if (j == tid) mine = d;
        }
        for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
        if (tid < b) {
            const double d = sqrt(mine);
            const bool gone = !(d > 1e-200 + 1e-30 * sqrt(mx));
            inv[tid] = gone ? 0.0 : 1.0 / d;
            if (tiny) tiny[tid] = gone;
        }
        __syncthreads();
    }
    // the lower triangle (the partials are symmetric: both halves are the same products in the same order)
    double far = 0.0;   // squared distance from the identity, of the lower triangle
#pragma unroll
    for (int p = 0; p < T; ++p)
#pragma unroll
        for (int q = 0; q <= p; ++q) {
            const int r = 16 * p + ty, c = 16 * q + tx;
            const bool in = r < b && c < b;
            double v = r == c ? 1.0 : 0.0;
            if (in) {
                const double f = scaled ? inv[r] * inv[c] : 1.0, g = sum(r * b + c);
                if (f != 0.0) v = r == c && scaled ? 1.0 : g * f;
                else far = INFINITY;   // an absent column
            }
            const double e = v - (r == c ? 1.0 : 0.0);
            far += e * e;
            if (DROP && r == c) inv[r] = kDependent * v;
            A[r * LD + c] = v;
            X[r * LD + c] = 0.0;
        }
    for (int o = 32; o > 0; o >>= 1) far += __shfl_xor(far, o);
    if (lane == 0) dist[w] = far;
    __syncthreads();
    const bool close = 2.0 * (dist[0] + dist[1] + dist[2] + dist[3]) <= near_tol * near_tol;
    if (near && tid == 0) near[z] = close;
    if (close) shift = 0.0;
    bool bad = false;
    // the diagonal tile kb: its inverse factor into X
    auto diagonal = [&](int kb) {
        double a[16], x[4];
        unsigned no = 0;
        const double least = DROP ? inv[16 * kb + lc] : 0.0;
#pragma unroll
        for (int j = 0; j < 16; ++j) a[j] = A[(16 * kb + lc) * LD + 16 * kb + j] + (j == lc ? shift : 0.0);
#pragma unroll
        for (int m = 0; m < 4; ++m) x[m] = 4 * lr + m == lc ? 1.0 : 0.0;
        diag_columns<DROP>(a, x, lc, least, no, std::make_integer_sequence<int, 16>());
        bad = bad || no;
        if (DROP && lane == 0) gone_of[kb] = no;
#pragma unroll
        for (int m = 0; m < 4; ++m) X[(16 * kb + lc) * LD + 16 * kb + 4 * lr + m] = x[m];
    };
    // P (tile i, k) times Q (tile j, l), transposed or not, added to acc
    auto product = [&](const double* P, int i, int k, const double* Q, int j, int l, bool transposed, double sign,
                       v4d acc) {
        double p[4], q[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            p[r] = sign * P[(16 * i + lc) * LD + 16 * k + 4 * r + lr];
            q[r] = transposed ? Q[(16 * j + lc) * LD + 16 * l + 4 * r + lr] : Q[(16 * j + 4 * r + lr) * LD + 16 * l + lc];
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = mma(p[r], q[r], acc);
        return acc;
    };
    auto tile = [&](const double* P, int i, int j) {
        v4d t;
#pragma unroll
        for (int r = 0; r < 4; ++r) t[r] = P[(16 * i + lr + 4 * r) * LD + 16 * j + lc];
        return t;
    };
    auto put = [&](double* P, int i, int j, v4d t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) P[(16 * i + lr + 4 * r) * LD + 16 * j + lc] = t[r];
    };
    if (w == 0) diagonal(0);
    __syncthreads();
    for (int kb = 0; kb < T; ++kb) {
        // row kb of X, column kb of L
        const v4d zero = {0, 0, 0, 0};
        for (int t = w; t < T - 1; t += 4) {
            if (t < kb) put(X, kb, t, product(X, kb, kb, X, kb, t, false, 1.0, zero));
            else put(A, t + 1, kb, product(A, t + 1, kb, X, kb, kb, true, 1.0, zero));
        }
        __syncthreads();
        if (kb + 1 == T) break;
        if (w == 0) {
            put(A, kb + 1, kb + 1, product(A, kb + 1, kb, A, kb + 1, kb, true, -1.0, tile(A, kb + 1, kb + 1)));
            wave_sync();   // its lanes read what others of them have just stored
            diagonal(kb + 1);
        } else {
            int turn = 0;
            for (int i = kb + 1; i < T; ++i) {
                for (int j = kb + 1; j <= i; ++j) {
                    if (i == kb + 1 && j == kb + 1) continue;
                    if (turn++ % 3 == w - 1) put(A, i, j, product(A, i, kb, A, j, kb, true, -1.0, tile(A, i, j)));
                }
                for (int j = 0; j <= kb; ++j)
                    if (turn++ % 3 == w - 1) put(X, i, j, product(A, i, kb, X, kb, j, false, -1.0, tile(X, i, j)));
            }
        }
        __syncthreads();
    }
    if (bad && tid == 0) flag[z] |= 2;
    __syncthreads();
    // R^{-1}[r][c] = X[c][r] / D_r (tiles below the diagonal are not read)
#pragma unroll
    for (int p = 0; p < T; ++p)
#pragma unroll
        for (int q = p; q < T; ++q) {
            const int r = 16 * p + ty, c = 16 * q + tx;
            if (r >= b || c >= b) continue;
            const double f = scaled ? inv[r] : 1.0;
            const bool dropped = DROP && r == c && (gone_of[q] >> tx & 1);
            Rinv[r * b + c] = dropped ? kDropped : X[c * LD + r] * (f != 0.0 ? f : 1.0);
        }
}

// calls f with the number of 16-column tiles as a compile-time constant
template <class F>
void with_tiles(int b, F f) {
    switch ((b + 15) / 16) {
        case 1: f(std::integral_constant<int, 1>()); break;
        case 2: f(std::integral_constant<int, 2>()); break;
        case 3: f(std::integral_constant<int, 3>()); break;
        case 4: f(std::integral_constant<int, 4>()); break;
        case 5: f(std::integral_constant<int, 5>()); break;
        default: f(std::integral_constant<int, 6>()); break;
    }
}

void check_cut(const BlockCut& q) {
    DTRG_REQUIRE(q.b >= 1 && q.b <= 16 * kMaxTiles && q.n >= 1 && q.nb >= 1 && q.nb < 65536 && q.rows % 16 == 0 &&
                     (i64)q.rows * q.chunks >= q.n && (i64)q.kc * q.splits >= q.n,
                 DTRG_EINVAL, "block kernel: bad sizes");
}

}  // namespace

BlockCut block_cut(int n, int b, int nb, i64 vbs) {
    BlockCut q;
    q.n = n; q.b = b; q.nb = nb; q.vbs = vbs;
    // One strip a workgroup, as long as that leaves no more than 144 partials: at n = 1024, b = 64 the product
    // and its Gram take 7.0, 10.3, 17.1 us with 16, 32 and 64 rows and adding up the partials 4.4, 3.3, 3.3; at
    // n = 9216, b = 96 they take 41, 41 and 34 us, and adding up 30, 12 and 7.
    q.rows = 16 * ((n + 16 * 144 - 1) / (16 * 144));
    q.chunks = (n + q.rows - 1) / q.rows;
    // the product: 32 rows a workgroup, the inner index split to give every compute unit one, in parts of
    // at least 64
    const i64 wg = (i64)((n + 31) / 32) * nb;
    q.splits = (int)std::max<i64>(1, std::min<i64>({kMaxSplits, n / 64, 512 / wg}));
    q.kc = ((n + q.splits - 1) / q.splits + 31) / 32 * 32;
    q.splits = (n + q.kc - 1) / q.kc;
    return q;
}

void block_product(const double* G, i64 g_bs, const double* V, double* Y, double* W, i64 w_bs, const BlockCut& q,
                   hipStream_t s) {
    check_cut(q);
    const dim3 grid((q.n + 31) / 32, q.splits, q.nb);
    with_tiles(q.b, [&](auto T) {
        hipLaunchKernelGGL((block_product_kernel<T()>), grid, dim3(64 * T()), 0, s, G, g_bs, V, q.vbs, Y,
                           q.splits > 1 ? W : nullptr, w_bs, q.n, q.b, q.kc);
    });
    DTRG_HIP(hipGetLastError());
}

void block_vty(const double* V, double* Y, const double* W, i64 w_bs, double* part, i64 p_bs, const BlockCut& q,
               hipStream_t s) {
    check_cut(q);
    with_tiles(q.b, [&](auto T) {
        hipLaunchKernelGGL((block_vty_kernel<T(), false>), dim3(q.chunks, q.nb), dim3(64 * T()), 0, s, V, Y, q.vbs, W,
                           w_bs, q.splits, BlockShift{}, part, p_bs, q.n, q.b, q.rows);
    });
    DTRG_HIP(hipGetLastError());
}

void block_gram(double* X, const double* V, const double* W, i64 w_bs, const BlockShift& sh, double* part, i64 p_bs,
                const BlockCut& q, hipStream_t s) {
    check_cut(q);
    with_tiles(q.b, [&](auto T) {
        hipLaunchKernelGGL((block_vty_kernel<T(), true>), dim3(q.chunks, q.nb), dim3(64 * T()), 0, s, V, X, q.vbs, W,
                           w_bs, q.splits, sh, part, p_bs, q.n, q.b, q.rows);
    });
    DTRG_HIP(hipGetLastError());
}

void block_rotate(const double* V, const double* Y, double* Vo, double* Yo, const double* Z, i64 z_bs,
                  const double* theta, i64 th_bs, const BlockShift& sh, double* rpart, i64 r_bs, double* part,
                  i64 p_bs, const BlockCut& q, hipStream_t s) {
    check_cut(q);
    with_tiles(q.b, [&](auto T) {
        hipLaunchKernelGGL((block_rotate_kernel<T()>), dim3(q.chunks, q.nb), dim3(64 * T()), 0, s, V, Y, Vo, Yo, q.vbs,
                           Z, z_bs, theta, th_bs, sh, rpart, r_bs, part, p_bs, q.n, q.b, q.rows);
    });
    DTRG_HIP(hipGetLastError());
}

void block_residuals(const double* rpart, i64 r_bs, double* res, i64 res_bs, const BlockCut& q, hipStream_t s) {
    hipLaunchKernelGGL(block_residual_kernel, dim3(q.nb), dim3(128), 0, s, rpart, r_bs, q.chunks, q.b, res, res_bs);
    DTRG_HIP(hipGetLastError());
}

void block_mult(const double* X, const double* V, const BlockShift& sh, const double* R, i64 r_bs, const int* tiny,
                i64 t_bs, bool drop, uint64_t seed, double* Out, double* part, i64 p_bs, const int* skip,
                const int* nogram, const BlockCut& q, hipStream_t s) {
    check_cut(q);
    with_tiles(q.b, [&](auto T) {
        hipLaunchKernelGGL((block_mult_kernel<T()>), dim3(q.chunks, q.nb), dim3(64 * T()), 0, s, X, V, q.vbs, sh, R,
                           r_bs, tiny, t_bs, drop ? 1 : 0, seed, Out, part, p_bs, skip, nogram, q.n, q.b, q.rows);
    });
    DTRG_HIP(hipGetLastError());
}

int block_reduce(double* part, i64 p_bs, const int* skip, const BlockCut& q, hipStream_t s) {
    if (q.chunks <= kConsumerParts) return q.chunks;
    const int bb = q.b * q.b;
    hipLaunchKernelGGL(block_reduce_kernel, dim3((bb + 255) / 256, q.nb), dim3(256), 0, s, part, p_bs, q.chunks, bb,
                       skip);
    DTRG_HIP(hipGetLastError());
    return 1;
}

void block_chol(const double* part, i64 p_bs, int np, int b, int nb, double shift_rel, bool scaled, double* Rinv,
                i64 r_bs, int* flag, const int* skip, int* near, double near_tol, int* tiny, i64 t_bs, bool drop,
                hipStream_t s) {
    DTRG_REQUIRE(b >= 1 && b <= 16 * kMaxTiles && np >= 1 && np <= kConsumerParts, DTRG_EINVAL,
                 "block_chol: bad sizes");
    DTRG_REQUIRE(scaled ? !drop : shift_rel == 0.0 && !tiny, DTRG_EINVAL,
                 "block_chol: a shift and absent columns need a scaled Gram, dropped ones a plain one");
    const double shift = shift_rel * b;   // the trace of a unit diagonal
    with_tiles(b, [&](auto T) {
        auto go = [&](auto DROP) {
            hipLaunchKernelGGL((block_chol_kernel<T(), DROP()>), dim3(nb), dim3(256), 0, s, part, p_bs, np, b, shift,
                               scaled ? 1 : 0, Rinv, r_bs, flag, skip, near, near_tol, tiny, t_bs);
        };
        if (drop) go(std::true_type());
        else go(std::false_type());
    });
    DTRG_HIP(hipGetLastError());
}

}  // namespace dtrg
