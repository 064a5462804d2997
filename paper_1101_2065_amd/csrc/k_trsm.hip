// Substitution inside a 256-row block of the blocked LU and solves (complex
// FP64 and FP32): X <- L^{-1} X or U^{-1} X for the block's triangle, whose 64 x 64
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
// value); the operand A comes from the factors in L2, four steps ahead.
// 256 rows, 2000 columns, 120 matrices: 1.07 ms, 74 TF in 8MNK (62 TF for 8
// matrices, whose 504 strips just fill the chip); bound by the matrix cores (103
// TF in this count) and, at two waves per SIMD, the latency around the barriers
// of its ten steps.  n = 1100: 25 ms of launches where the products took 32.
// Wider strips would leave one wave per SIMD (registers).
//
// FP32 has the same products in FP64 and rounds once per panel: the error of the
// 32-bit forms after refinement is a power of their first solution's.  With the
// sums in FP32, 128 roundings a panel, the split-BF16 form's error at 655 rows
// (tolerance 1e-10, 14 chains) was 9.3e-12, against 5.4e-12 by separate
// split-BF16 products and 4.4e-12 so.  It costs matrix-core time: 517 and 655
// rows, 128 frequencies, three solves, 5.1 and 7.4 ms of launches for 4.3 and
// 5.9; the separate products took 6.5 (FP32) and 7.2 (split BF16).
#include "gw_internal.h"
#include "gw_prof.h"
#include "k_mfma.h"

#include <hip/hip_runtime.h>

namespace gwk {

namespace {

constexpr int TNB = 64;  // panel

// v2: a complex value in registers and LDS; G2: in global memory, where it lies
// on its real type's boundaries.  (Functions take T and name G2 themselves: a
// type given as a template argument loses its alignment.)
template <typename T>
struct Tv;
template <>
struct Tv<double> {
    typedef double v2 __attribute__((ext_vector_type(2)));
    typedef double v2u __attribute__((ext_vector_type(2), aligned(8)));
    typedef dglobal<v2u> G2;
};
template <>
struct Tv<float> {
    typedef float v2 __attribute__((ext_vector_type(2)));
    typedef float v2u __attribute__((ext_vector_type(2), aligned(4)));
    typedef dglobal<v2u> G2;
};
typedef Tv<double>::v2 zd2;
typedef Mfma<double>::v4 v4;
constexpr int NH = 2;  // sixteens of columns in a strip

// c = A B over 64 k for this wave's 16 rows and the strip's columns, as three
// real FP64 products (ac, bd, (a + b)(c + d)).  row: the lane's row of A; a
// already holds its first four steps (k = lane / 16 + 4 q).
struct Acc {
    v4 r[NH], i[NH], s[NH];
    __device__ __forceinline__ double re(int h, int e) const { return r[h][e] - i[h][e]; }
    __device__ __forceinline__ double im(int h, int e) const { return s[h][e] - r[h][e] - i[h][e]; }
};
template <typename T>
__device__ __forceinline__ void load4(typename Tv<T>::v2 (&a)[4], const typename Tv<T>::G2 *row, int k0, int lk,
                                      int kmax) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = row[min(k0 + 4 * q + lk, kmax)];
}
template <typename T>
__device__ __forceinline__ void mul64(Acc &c, typename Tv<T>::v2 (&a)[4], const typename Tv<T>::G2 *row, int lk,
                                      int lane, int kmax, const zd2 *b) {
#pragma unroll
    for (int j = 0; j < NH; ++j) c.r[j] = c.i[j] = c.s[j] = v4{0, 0, 0, 0};
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        typename Tv<T>::v2 n[4];
        if (h < 3) load4<T>(n, row, 16 * (h + 1), lk, kmax);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            zd2 bv[NH];
#pragma unroll
            for (int j = 0; j < NH; ++j) bv[j] = b[(NH * (4 * h + q) + j) * 64 + lane];
            const double ax = a[q].x, ay = a[q].y, sa = ax + ay;
#pragma unroll
            for (int j = 0; j < NH; ++j) c.r[j] = Mfma<double>::op(ax, bv[j].x, c.r[j]);
#pragma unroll
            for (int j = 0; j < NH; ++j) c.i[j] = Mfma<double>::op(ay, bv[j].y, c.i[j]);
#pragma unroll
            for (int j = 0; j < NH; ++j) c.s[j] = Mfma<double>::op(sa, bv[j].x + bv[j].y, c.s[j]);
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
template <typename T, bool UPPER>
__device__ __forceinline__ void solve_strip(int wo, int n, const typename Tv<T>::G2 *Tm, int64_t ldt,
                                            const typename Tv<T>::G2 *inv, typename Tv<T>::G2 *X, int64_t ldx, int tri,
                                            int c0) {
    typedef typename Tv<T>::v2 V2;
    typedef typename Tv<T>::G2 G2;
    __shared__ zd2 xb[NH * TNB * 16], yb[NH * TNB * 16];  // X_p before and after its diagonal block
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 15, lk = lane >> 4;
    const int np = (wo + TNB - 1) / TNB;
    // where a result's row goes as operand B: step k / 4, lanes 16 (k % 4) ..
    auto slot = [&](int h, int e) {
        const int k = Mfma<double>::row(lane, e);
        return (NH * (4 * wave + (k >> 2)) + h) * 64 + 16 * (k & 3) + lr;
    };
    // panels in order of solution: step s is panel s, or np - 1 - s
    const int first = tri >= 0 ? max(0, (c0 - tri) / TNB) : 0;  // upper: panels below it are not needed
    V2 x[4][NH][4];  // [panel][sixteen of columns][e]: row 64 p + 16 wave + Mfma row e, column c0 + 16 h + lr
#pragma unroll
    for (int p = 0; p < 4; ++p)
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = TNB * p + 16 * wave + Mfma<double>::row(lane, e), col = c0 + 16 * h + lr;
                x[p][h][e] = V2{0, 0};
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
        V2 a[4];
        load4<T>(a, di, 0, lk, TNB - 1);
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) xb[slot(h, e)] = zd2{(double)x[p][h][e].x, (double)x[p][h][e].y};
        __syncthreads();
        Acc c;
        mul64<T>(c, a, di, lk, lane, TNB - 1, xb);
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const V2 y{(T)c.re(h, e), (T)c.im(h, e)};
                yb[slot(h, e)] = zd2{(double)y.x, (double)y.y};
                const int row = TNB * p + 16 * wave + Mfma<double>::row(lane, e), col = c0 + 16 * h + lr;
                if (row < wo && col < n) X[(int64_t)row * ldx + col] = y;
            }
        // the panels still to come
        const int kmax = min(TNB, wo - TNB * p) - 1;
        auto row_of = [&](int q) {
            return Tm + (int64_t)min(TNB * q + 16 * wave + lr, wo - 1) * ldt + TNB * p;
        };
        bool have = false;
#pragma unroll
        for (int d = 1; d < 4; ++d) {
            const int q = UPPER ? p - d : p + d;
            if (q < 0 || q > 3) continue;
            if (q >= np || q < first) continue;  // uniform
            const G2 *row = row_of(q);
            load4<T>(a, row, 0, lk, kmax);
            if (!have) __syncthreads();  // yb is complete
            have = true;
            mul64<T>(c, a, row, lk, lane, kmax, yb);
#pragma unroll
            for (int h = 0; h < NH; ++h)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[q][h][e].x = (T)(x[q][h][e].x - c.re(h, e));
                    x[q][h][e].y = (T)(x[q][h][e].y - c.im(h, e));
                }
        }
        // (no reader of xb or yb is left behind: the next step writes xb after
        // this step's first barrier and yb after its own)
    }
}

template <typename T, bool UPPER>
__global__ __launch_bounds__(256, 2) void k_block_solve(int wo, int n, const T *T_, int64_t ldt, int64_t sT,
                                                        const T *inv_, int64_t sI, T *X_, int64_t ldx,
                                                        int64_t sX, int tri) {
    typedef typename Tv<T>::G2 G2;
    const int64_t nt = (int64_t)gridDim.x * gridDim.y, l = blockIdx.x + (int64_t)gridDim.x * blockIdx.y;
    const int64_t n8 = nt / 8, t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;  // one matrix's strips on one XCD
    const int64_t b = t / gridDim.x;
    solve_strip<T, UPPER>(wo, n, (const G2 *)T_ + b * sT, ldt, (const G2 *)inv_ + b * sI, (G2 *)X_ + b * sX, ldx,
                              tri, (int)(t % gridDim.x) * 16 * NH);
}

// Many batched block solves in one launch, a strip per workgroup, in the order
// of k_block_solve.
template <typename T, bool UPPER>
__global__ __launch_bounds__(256, 2) void k_block_solve_group(const GemmItem *__restrict__ items, int n_items,
                                                              int64_t n_tiles) {
    typedef typename Tv<T>::G2 G2;
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
    solve_strip<T, UPPER>(g.M, g.N, (const G2 *)g.A + bz * g.sA, g.lda, (const G2 *)g.B + bz * g.sB,
                              (G2 *)g.C + bz * g.sC, g.ldc, g.K, (int)(r - bz * g.tx) * 16 * NH);
}

template <typename T, typename Z>
hipError_t block_solve(hipStream_t st, bool upper, int wo, int n, const Z *Tm, int64_t ldt, int64_t sT, const Z *inv,
                       int64_t sI, Z *X, int64_t ldx, int64_t sX, int batch, int tri) {
    if (wo <= 0 || n <= 0 || batch <= 0) return hipSuccess;
    if (wo > 4 * TNB || batch > 65535) return hipErrorInvalidValue;
    if (!upper) tri = -1;
    // the triangle with its diagonal blocks' other halves
    const double flops = 8.0 * 0.5 * wo * (wo + TNB) * n * batch;
    if (OpRecorder *rec = g_rec) {
        RecOp o;
        o.kind = RecOp::GEMM;
        o.key = QK_SOLVE * 4 + (sizeof(T) == 4 ? 2 : 0) + (upper ? 1 : 0);
        o.g = GemmItem{Tm, inv, X, ldt, 0, ldx, sT, sI, sX, 0.0, 0.0, wo, n, tri, batch, 0, 0, 0};
        o.flops = flops;
        rec->ops.push_back(std::move(o));
        return hipSuccess;
    }
    ProfScope ps(st, sizeof(T) == 4 ? "block_solve_c" : "block_solve", flops, 4.0 * sizeof(T) * wo * (double)n * batch);
    const int cols = 16 * NH;
    const dim3 grid((unsigned)((n + cols - 1) / cols), (unsigned)batch);
    if (upper)
        hipLaunchKernelGGL((k_block_solve<T, true>), grid, dim3(256), 0, st, wo, n, (const T *)Tm, ldt, sT,
                           (const T *)inv, sI, (T *)X, ldx, sX, tri);
    else
        hipLaunchKernelGGL((k_block_solve<T, false>), grid, dim3(256), 0, st, wo, n, (const T *)Tm, ldt, sT,
                           (const T *)inv, sI, (T *)X, ldx, sX, tri);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_block_solve(hipStream_t st, bool upper, int wo, int n, const zdbl *T, int64_t ldt, int64_t sT,
                              const zdbl *inv, int64_t sI, zdbl *X, int64_t ldx, int64_t sX, int batch, int tri) {
    return block_solve<double>(st, upper, wo, n, T, ldt, sT, inv, sI, X, ldx, sX, batch, tri);
}
hipError_t launch_block_solve(hipStream_t st, bool upper, int wo, int n, const zflt *T, int64_t ldt, int64_t sT,
                              const zflt *inv, int64_t sI, zflt *X, int64_t ldx, int64_t sX, int batch, int tri) {
    return block_solve<float>(st, upper, wo, n, T, ldt, sT, inv, sI, X, ldx, sX, batch, tri);
}

#define GW_SOLVE(OP)                             \
    do {                                         \
        if (variant == 0) OP(double, false);     \
        else if (variant == 1) OP(double, true); \
        else if (variant == 2) OP(float, false); \
        else OP(float, true);                    \
    } while (0)

hipError_t launch_block_solve_group(hipStream_t st, int variant, const GemmItem *items, int n_items, int64_t n_tiles) {
    if (n_tiles > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)n_tiles), blk(256);
#define GW_RUN(T, UP) hipLaunchKernelGGL((k_block_solve_group<T, UP>), grid, blk, 0, st, items, n_items, n_tiles)
    GW_SOLVE(GW_RUN);
#undef GW_RUN
    return hipGetLastError();
}
int block_solve_occupancy(int variant) {
    int occ = 0;
    hipError_t e = hipErrorInvalidValue;
#define GW_OCC(T, UP) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_block_solve_group<T, UP>, 256, 0)
    GW_SOLVE(GW_OCC);
#undef GW_OCC
    return e == hipSuccess && occ > 0 ? occ : 2;
}
int block_solve_columns() { return 16 * NH; }

}  // namespace gwk
