// Products with a Gram in Kronecker form (gfx950), FP64 matrix instructions:
//   C[(a,c)][alpha] = (1/s) sum_d sum_jk B[c][d][jk] (sum_b A[a][b][jk] V[(b,d)][alpha])
// for A, B [X][X][16] (a squared physical dimension of 16) and X <= 128.
//
// As two contractions the intermediate, 16 times the size of V, is written and read once, in scattered pieces:
// at X = 96 with 96 columns (2 x 2.7 GFLOP, 113 MB) they took 101 and 87 us, and the permutation of A before
// and the scaling after them 10.  Here the intermediate stays in registers: for one a and d, the 16 x 16 tile of
// jk and alpha that v_mfma_f64_16x16x4f64 accumulates (register r of lane l: jk = l / 16 + 4 r, alpha = l mod 16)
// is the operand of the r-th step of 4 of the sum over jk.  A wave takes one a and 16 columns, holds A[a] in
// registers and runs over d; four waves share the rows of V and B of each d through LDS (one d ahead).  The range of
// d is split to give every compute unit about four workgroups, and a second kernel adds the parts up.
// Measured there: 110 us and 10 for the sum, 49 TFLOP/s (148 with selects on the loaded values, which made each
// load wait for the one before).
// Y^2 = 16 only: the tile is jk x alpha, and 4 or 9 values of jk would leave three quarters or half of its rows empty
// (or want several a in it, another layout of A and of the sums).  Above X = 128 A[a] and the sums do not fit the
// registers.  Those sizes keep the two contractions; up to X = 2 Y^2 = 32 the Gram is formed.
#include <algorithm>
#include <type_traits>

#include "block.hpp"

namespace dtrg {

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ inline v4d mma(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

constexpr int kMaxParts = 16;

// T = ceil(X / 16)
template <int T>
__global__ __launch_bounds__(256) void kron_product_kernel(const double* __restrict__ A, i64 a_bs,
                                                           const double* __restrict__ B, i64 b_bs,
                                                           const double* __restrict__ V, i64 v_bs,
                                                           double* __restrict__ W, i64 w_bs, int X, int w, int parts,
                                                           int per) {
    constexpr int NX = 16 * T, LB = 17;   // rows of 17: the 16 rows of an operand of B fall on different banks
    __shared__ double Vs[2][NX * 16];     // [b][alpha]
    __shared__ double Bs[2][NX * LB];     // [c][jk]
    const int tid = threadIdx.x, lane = tid & 63, lr = lane >> 4, lc = lane & 15;
    const int z = blockIdx.z / parts, part = blockIdx.z % parts;
    const int al0 = 16 * blockIdx.x, a = 4 * blockIdx.y + (tid >> 6), d0 = part * per, d1 = min(X, d0 + per);
    A += z * a_bs;
    B += z * b_bs;
    V += z * v_bs;
    double av[4 * T];
#pragma unroll
    for (int k = 0; k < 4 * T; ++k) {
        const int b = 4 * k + lr;
        const bool in = a < X && b < X;
        const double x = A[in ? ((i64)a * X + b) * 16 + lc : 0];
        av[k] = in ? x : 0.0;
    }
    // Rows at or past X are row X - 1 again: those of V meet zeros of A, those of B and columns at or past w are
    // not stored.  (No select on a loaded value: it would wait for each load.)
    const int row = tid >> 4, col = tid & 15;
    const double* vp = V + min(al0 + col, w - 1);
    const double* bp = B + col;
    double vr[T], br[T];
    auto load = [&](int d) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const i64 rd = (i64)min(row + 16 * i, X - 1) * X + d;
            vr[i] = vp[rd * w];
            br[i] = bp[rd * 16];
        }
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int r = row + 16 * i;
            Vs[buf][r * 16 + col] = vr[i];
            Bs[buf][r * LB + col] = br[i];
        }
    };
    v4d acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = v4d{0, 0, 0, 0};
    load(d0);
    store(0);
    __syncthreads();
    int buf = 0;
    for (int d = d0; d < d1; ++d, buf ^= 1) {
        if (d + 1 < d1) load(d + 1);
        v4d p0 = {0, 0, 0, 0}, p1 = {0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < 4 * T; k += 2) {
            p0 = mma(av[k], Vs[buf][(4 * k + lr) * 16 + lc], p0);
            p1 = mma(av[k + 1], Vs[buf][(4 * k + 4 + lr) * 16 + lc], p1);
        }
        const v4d p = p0 + p1;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < T; ++i) acc[i] = mma(Bs[buf][(16 * i + lc) * LB + lr + 4 * r], p[r], acc[i]);
        if (d + 1 < d1) store(buf ^ 1);
        __syncthreads();
    }
    if (a >= X || al0 + lc >= w) return;
    double* o = W + z * w_bs + ((i64)part * X + a) * X * w + al0 + lc;
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = 16 * i + lr + 4 * r;
            if (c < X) o[(i64)c * w] = acc[i][r];
        }
}

__global__ __launch_bounds__(256) void kron_sum_kernel(const double* __restrict__ W, i64 w_bs, int parts, i64 total,
                                                       const double* __restrict__ s, i64 s_bs, double* __restrict__ C,
                                                       i64 c_bs) {
    const int z = blockIdx.y;
    const double f = 1.0 / s[z * s_bs];
    W += z * w_bs;
    C += z * c_bs;
    for (i64 i = blockIdx.x * (i64)256 + threadIdx.x; i < total; i += (i64)gridDim.x * 256) {
        double t[kMaxParts], sum = 0.0;
#pragma unroll
        for (int p = 0; p < kMaxParts; ++p) t[p] = p < parts ? W[p * total + i] : 0.0;
#pragma unroll
        for (int p = 0; p < kMaxParts; ++p) sum += t[p];
        C[i] = sum * f;
    }
}

}  // namespace

bool kron_product_fits(int X, int YY) { return YY == 16 && X > 32 && X <= 128; }

void kron_product(const double* A, i64 a_bs, const double* B, i64 b_bs, const double* V, i64 v_bs, double* W, i64 w_bs,
                  const double* s_dev, i64 s_bs, double* C, i64 c_bs, int X, int w, int nb, hipStream_t s) {
    DTRG_REQUIRE(kron_product_fits(X, 16) && w >= 1 && nb >= 1, DTRG_EINVAL, "kron_product: bad sizes");
    const i64 total = (i64)X * X * w;
    const int tiles = (w + 15) / 16, groups = (X + 3) / 4;
    int parts = (int)std::max<i64>(1, std::min<i64>({kMaxParts, X / 4, 1024 / ((i64)tiles * groups * nb)}));
    const int per = (X + parts - 1) / parts;
    parts = (X + per - 1) / per;
    DTRG_REQUIRE(parts * total <= w_bs && (i64)nb * parts < 65536 && groups < 65536, DTRG_EINVAL,
                 "kron_product: the workspace does not hold the parts");
    const dim3 grid(tiles, groups, nb * parts);
    auto go = [&](auto T) {
        hipLaunchKernelGGL((kron_product_kernel<T()>), grid, dim3(256), 0, s, A, a_bs, B, b_bs, V, v_bs, W, w_bs, X, w,
                           parts, per);
    };
    switch ((X + 15) / 16) {
        case 3: go(std::integral_constant<int, 3>()); break;
        case 4: go(std::integral_constant<int, 4>()); break;
        case 5: go(std::integral_constant<int, 5>()); break;
        case 6: go(std::integral_constant<int, 6>()); break;
        case 7: go(std::integral_constant<int, 7>()); break;
        default: go(std::integral_constant<int, 8>()); break;
    }
    DTRG_HIP(hipGetLastError());
    const unsigned blocks = (unsigned)std::max<i64>(1, std::min<i64>((total + 255) / 256, 4096));
    hipLaunchKernelGGL(kron_sum_kernel, dim3(blocks, nb), dim3(256), 0, s, W, w_bs, parts, total, s_dev, s_bs, C, c_bs);
    DTRG_HIP(hipGetLastError());
}

}  // namespace dtrg
