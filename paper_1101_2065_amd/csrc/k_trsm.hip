// Substitution inside a 256-row block of the blocked LU and solves (complex
// FP64): X <- L^{-1} X or U^{-1} X for the block's triangle, whose 64 x 64
// diagonal blocks come inverted (Section 2 eq. Coulombscreening, the dense
// solve of W).
//
// Panel by panel, X_p <- T_pp^{-1} X_p, then X_q -= T_qp X_p for the panels q
// still to come.  As separate products these were bound by HBM: each K = 64
// update reads and writes all the rows below it (44-55 TF in 8MNK).  Here a
// workgroup keeps a strip of 32 columns of all 256 rows in registers, so X is
// read and written once and the products run from LDS: wave w holds rows
// 16 w .. 16 w + 15 of every panel, which gives the four waves equal shares of
// every step.  X_p goes through LDS as the matrix-core operand B (the register
// layout of a result is already that order: one conflict-free 16-byte store per
// value); the operand A comes from the factors in L2, four steps ahead.  The
// arithmetic, and its order, is that of the separate products.
// 256 rows, 2000 columns, 120 matrices: 1.07 ms, 74 TF in 8MNK (62 TF for 8
// matrices, whose 504 strips just fill the chip); bound by the matrix cores (103
// TF in this count) and, at two waves per SIMD, the latency around the barriers
// of its ten steps.  A launch for seven: 39 solves of n = 1100 take 25 ms instead
// of 38.  Strips of 32 columns: 64 would leave one wave per SIMD (registers).
#include "gw_internal.h"
#include "gw_prof.h"
#include "k_mfma.h"

#include <hip/hip_runtime.h>

namespace gwk {

namespace {

constexpr int TNB = 64;  // panel

typedef double td2 __attribute__((ext_vector_type(2)));
typedef double td2u __attribute__((ext_vector_type(2), aligned(8)));
typedef Mfma<double>::v4 tv4;

// acc += A B over 64 k for this wave's 16 rows and 32 columns, as three real
// products (ac, bd, (a + b)(c + d)); ap: the lane's value of A at k = lane / 16,
// already holding the first four steps in a; kmax: the last k with data.
struct Acc {
    tv4 r[2], i[2], s[2];
};
template <typename G2>
__device__ __forceinline__ void load4(td2 (&a)[4], const G2 *row, int k0, int lk, int kmax) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = row[min(k0 + 4 * q + lk, kmax)];
}
template <typename G2>
__device__ __forceinline__ void mul64(Acc &c, td2 (&a)[4], const G2 *row, int lk, int lane, int kmax, const td2 *b) {
#pragma unroll
    for (int j = 0; j < 2; ++j) c.r[j] = c.i[j] = c.s[j] = tv4{0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        td2 n[4];
        if (h < 3) load4(n, row, 16 * (h + 1), lk, kmax);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const td2 b0 = b[(2 * (4 * h + q)) * 64 + lane], b1 = b[(2 * (4 * h + q) + 1) * 64 + lane];
            const double sa = a[q].x + a[q].y, s0 = b0.x + b0.y, s1 = b1.x + b1.y;
            c.r[0] = Mfma<double>::op(a[q].x, b0.x, c.r[0]);
            c.r[1] = Mfma<double>::op(a[q].x, b1.x, c.r[1]);
            c.i[0] = Mfma<double>::op(a[q].y, b0.y, c.i[0]);
            c.i[1] = Mfma<double>::op(a[q].y, b1.y, c.i[1]);
            c.s[0] = Mfma<double>::op(sa, s0, c.s[0]);
            c.s[1] = Mfma<double>::op(sa, s1, c.s[1]);
        }
        if (h < 3) {
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = n[q];
        }
    }
}

// T: the block's corner in the factors (wo x wo of it, wo <= 256), leading
// dimension ldt; inv: its inverted diagonal blocks, 64 x 64 each, zero past wo;
// X: wo x n, leading dimension ldx; c0: the strip's first column.  tri >= 0
// (upper only): the block's first row's index among X's columns; panel p is
// then needed in columns below tri + 64 (p + 1) alone (a symmetric result, its
// lower triangle).
template <bool UPPER, typename G2>
__device__ __forceinline__ void solve_strip(int wo, int n, const G2 *T, int64_t ldt, const G2 *inv, G2 *X, int64_t ldx,
                                            int tri, int c0) {
    __shared__ td2 xb[32 * 64], yb[32 * 64];  // X_p before and after its diagonal block
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int np = (wo + TNB - 1) / TNB;
    // panels in order of solution: step s is panel s, or np - 1 - s
    const int first = tri >= 0 ? max(0, (c0 - tri) / TNB) : 0;  // upper: panels below it are not needed
    td2 x[4][2][4];  // [panel][column half][e]: row 64 p + 16 wave + lk + 4 e, column c0 + 16 h + lr
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = TNB * p + 16 * wave + lk + 4 * e, col = c0 + 16 * h + lr;
                x[p][h][e] = td2{0, 0};
                if (p >= first && row < wo && col < n) x[p][h][e] = X[(int64_t)row * ldx + col];
            }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        // (the panel index has to be static, so an upper solve of fewer panels
        // skips the first steps)
        constexpr int last = 3;
        const int p = UPPER ? last - s : s;
        if (p >= np || p < first) continue;  // uniform
        const G2 *di = inv + (int64_t)p * TNB * TNB + (16 * wave + lr) * TNB;
        td2 a[4];
        load4(a, di, 0, lk, TNB - 1);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) xb[(2 * (4 * wave + e) + h) * 64 + lane] = x[p][h][e];
        __syncthreads();
        Acc c;
        mul64(c, a, di, lk, lane, TNB - 1, xb);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const td2 y{c.r[h][e] - c.i[h][e], c.s[h][e] - c.r[h][e] - c.i[h][e]};
                yb[(2 * (4 * wave + e) + h) * 64 + lane] = y;
                const int row = TNB * p + 16 * wave + lk + 4 * e, col = c0 + 16 * h + lr;
                if (row < wo && col < n) X[(int64_t)row * ldx + col] = y;
            }
        // the panels still to come
        const int kmax = min(TNB, wo - TNB * p) - 1;
        auto row_of = [&](int q) {
            return T + (int64_t)min(TNB * q + 16 * wave + lr, wo - 1) * ldt + TNB * p;
        };
        bool have = false;
#pragma unroll
        for (int d = 1; d < 4; ++d) {
            const int q = UPPER ? p - d : p + d;
            if (q < 0 || q > 3) continue;
            if (q >= np || q < first) continue;  // uniform
            const G2 *row = row_of(q);
            load4(a, row, 0, lk, kmax);
            if (!have) __syncthreads();  // yb is complete
            have = true;
            mul64(c, a, row, lk, lane, kmax, yb);
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[q][h][e].x = -(c.r[h][e] - c.i[h][e]) + x[q][h][e].x;
                    x[q][h][e].y = -(c.s[h][e] - c.r[h][e] - c.i[h][e]) + x[q][h][e].y;
                }
        }
        // (no reader of xb or yb is left behind: the next step writes xb after
        // this step's first barrier and yb after its own)
    }
}

template <bool UPPER>
__global__ __launch_bounds__(256, 2) void k_block_solve(int wo, int n, const double *T_, int64_t ldt, int64_t sT,
                                                        const double *inv_, int64_t sI, double *X_, int64_t ldx,
                                                        int64_t sX, int tri) {
    typedef dglobal<td2u> G2;
    const int64_t nt = (int64_t)gridDim.x * gridDim.y, l = blockIdx.x + (int64_t)gridDim.x * blockIdx.y;
    const int64_t n8 = nt / 8, t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;  // one matrix's strips on one XCD
    const int64_t b = t / gridDim.x;
    solve_strip<UPPER, G2>(wo, n, (const G2 *)T_ + b * sT, ldt, (const G2 *)inv_ + b * sI, (G2 *)X_ + b * sX, ldx, tri,
                           (int)(t % gridDim.x) * 32);
}

// Many batched block solves in one launch, a strip per workgroup, in the order
// of k_block_solve.
template <bool UPPER>
__global__ __launch_bounds__(256, 2) void k_block_solve_group(const GemmItem *__restrict__ items, int n_items,
                                                              int64_t n_tiles) {
    typedef dglobal<td2u> G2;
    const int64_t l = blockIdx.x, n8 = n_tiles / 8;
    const int64_t t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;
    int a = 0, b = n_items - 1;
    while (a < b) {
        const int m = (a + b + 1) >> 1;
        if (items[m].t0 <= t) a = m;
        else b = m - 1;
    }
    const GemmItem g = items[a];
    const int64_t r = t - g.t0, bz = r / g.tx;
    solve_strip<UPPER, G2>(g.M, g.N, (const G2 *)g.A + bz * g.sA, g.lda, (const G2 *)g.B + bz * g.sB,
                           (G2 *)g.C + bz * g.sC, g.ldc, g.K, (int)(r - bz * g.tx) * 32);
}

}  // namespace

hipError_t launch_block_solve(hipStream_t st, bool upper, int wo, int n, const zdbl *T, int64_t ldt, int64_t sT,
                              const zdbl *inv, int64_t sI, zdbl *X, int64_t ldx, int64_t sX, int batch, int tri) {
    if (wo <= 0 || n <= 0 || batch <= 0) return hipSuccess;
    if (wo > 4 * TNB || batch > 65535) return hipErrorInvalidValue;
    if (!upper) tri = -1;
    // the triangle with its diagonal blocks' other halves
    const double flops = 8.0 * 0.5 * wo * (wo + TNB) * n * batch;
    if (OpRecorder *rec = g_rec) {
        RecOp o;
        o.kind = RecOp::GEMM;
        o.key = QK_SOLVE * 4 + (upper ? 1 : 0);
        o.g = GemmItem{T, inv, X, ldt, 0, ldx, sT, sI, sX, 0.0, 0.0, wo, n, tri, batch, 0, 0, 0};
        o.flops = flops;
        rec->ops.push_back(std::move(o));
        return hipSuccess;
    }
    ProfScope ps(st, "block_solve", flops, 32.0 * wo * (double)n * batch);
    const dim3 grid((unsigned)((n + 31) / 32), (unsigned)batch);
    if (upper)
        hipLaunchKernelGGL((k_block_solve<true>), grid, dim3(256), 0, st, wo, n, (const double *)T, ldt, sT,
                           (const double *)inv, sI, (double *)X, ldx, sX, tri);
    else
        hipLaunchKernelGGL((k_block_solve<false>), grid, dim3(256), 0, st, wo, n, (const double *)T, ldt, sT,
                           (const double *)inv, sI, (double *)X, ldx, sX, tri);
    return hipGetLastError();
}

hipError_t launch_block_solve_group(hipStream_t st, bool upper, const GemmItem *items, int n_items, int64_t n_tiles) {
    if (n_tiles > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)n_tiles), blk(256);
    if (upper) hipLaunchKernelGGL((k_block_solve_group<true>), grid, blk, 0, st, items, n_items, n_tiles);
    else hipLaunchKernelGGL((k_block_solve_group<false>), grid, blk, 0, st, items, n_items, n_tiles);
    return hipGetLastError();
}
int block_solve_occupancy(bool upper) {
    int occ = 0;
    const hipError_t e =
        upper ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_block_solve_group<true>, 256, 0)
              : hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_block_solve_group<false>, 256, 0);
    return e == hipSuccess && occ > 0 ? occ : 2;
}

}  // namespace gwk
