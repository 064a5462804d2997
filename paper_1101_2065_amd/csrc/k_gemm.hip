// Dense products on the CDNA4 matrix cores (MFMA), for the W solve:
// forming A = 1 - v chi0, the trailing updates of the blocked LU, the
// triangular block products of the solve, and the FP64 refinement residual
// (Section 2 eq. Coulombscreening, Section 3 eq. tensorform-scr-inter).
//
// Complex numbers are interleaved {re, im}.  The products of the FP64 LU and
// solves use three real MFMA products per complex product, ac, bd and
// (a + b)(c + d) (a quarter less matrix-core work, normwise as accurate); the
// FP64 refinement residual and the FP32 products use four.
// Tiles: 256-thread workgroups, four 64-wide waves in 2x2.  The FP64 products,
// complex (zgemm_tile), real and real-times-complex (rgemm_tile), copy their
// operands from global memory straight into LDS in matrix-core order and keep
// almost nothing but MFMA instructions in the K loop.  The FP32 products
// (gemm_tile) stage them through registers, 64x64 (K steps of 16), 128x64 and
// narrower (K steps of 8), as do at 64x64 the real and real-times-complex ones
// whose rows rgemm_tile cannot copy 16 bytes at a time.  The tiles are dealt to
// the XCDs in contiguous ranges (each XCD has its own L2).
#include "gw_internal.h"
#include "gw_prof.h"
#include "k_mfma.h"

#include <hip/hip_runtime.h>

#include <algorithm>

namespace gwk {

namespace {

// C = alpha * A * B + beta * C (+ identity on the real diagonal if add_eye).
// AC/BC: A/B complex (else real).  C is complex unless both are real.
// Optional C32: a complex-float copy of the result (same ld).
// Workgroup = 256 threads = 2x2 waves; a wave owns WM x WN MFMA blocks of
// 16x16, so the workgroup tile is (32 WM) x (32 WN); K advances BK per
// LDS stage.
// One (32 WM) x (32 WN) tile of C with its top-left corner at (m0, n0); A, B,
// C (and C32) point at the tile's batch entry.
template <typename T, bool AC, bool BC, int WM, int WN, int BK, typename GT = T>
__device__ __forceinline__ void gemm_tile(int M, int N, int K, T alpha, const GT *__restrict__ A, int64_t lda,
                                          const GT *B, int64_t ldb, T beta, GT *C, int64_t ldc, int add_eye,
                                          float *C32, int m0, int n0) {
    static_assert(!(AC && BC) || sizeof(T) == 4, "complex FP64 products take zgemm_tile");
    constexpr int BM = 32 * WM, BN = 32 * WN;
    constexpr bool CC = AC || BC;
    constexpr int ea = AC ? 2 : 1, eb = BC ? 2 : 1, ec = CC ? 2 : 1;
    constexpr int EA = BM * BK / 256, TPRA = BK / EA;  // elements per thread, threads per row (A)
    constexpr int EB = BK * BN / 256, TPRB = BN / EB;  // (B)
    static_assert(EA >= 1 && EB >= 1 && TPRA >= 1 && TPRB >= 1 && BK % 8 == 0, "tile too small");
    typedef typename Mfma<T>::v4 v4;
    // the 64x64 tile gives each thread B columns TPRB apart
    constexpr int SB = (BK == 16) ? TPRB : 1;
    // complex operands are staged interleaved {re, im}: one 16-byte LDS read
    // per operand value instead of two 8-byte ones
    typedef T T2 __attribute__((ext_vector_type(2)));
    __shared__ T Ar[2][AC ? 1 : BK][AC ? 1 : BM];
    __shared__ T2 Ac[2][AC ? BK : 1][AC ? BM : 1];
    __shared__ T Br[2][BC ? 1 : BK][BC ? 1 : BN];
    __shared__ T2 Bc[2][BC ? BK : 1][BC ? BN : 1];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    v4 accr[WM][WN], acci[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            accr[i][j] = v4{0, 0, 0, 0};
            acci[i][j] = v4{0, 0, 0, 0};
        }

    const int a_row = tid / TPRA, a_k = (tid % TPRA) * EA;
    const int b_row = tid / TPRB, b_col = (SB == 1) ? (tid % TPRB) * EB : tid % TPRB;
    T ra_r[EA], ra_i[EA], rb_r[EB], rb_i[EB];
    // interior tiles take an unpredicated path
    const bool rows_in = m0 + BM <= M;
    const bool cols_in = n0 + BN <= N;
    auto gload = [&](int k0) {
        const int gr = m0 + a_row;
        if (rows_in && k0 + BK <= K) {
            const GT *p = A + ((int64_t)gr * lda + k0 + a_k) * ea;
#pragma unroll
            for (int c = 0; c < EA; ++c) {
                ra_r[c] = p[c * ea];
                if constexpr (AC) ra_i[c] = p[c * ea + 1];
                else ra_i[c] = T(0);
            }
        } else {
#pragma unroll
            for (int c = 0; c < EA; ++c) {
                const int gk = k0 + a_k + c;
                if (gr < M && gk < K) {
                    const GT *p = A + ((int64_t)gr * lda + gk) * ea;
                    ra_r[c] = p[0];
                    if constexpr (AC) ra_i[c] = p[1];
                    else ra_i[c] = T(0);
                } else {
                    ra_r[c] = T(0);
                    ra_i[c] = T(0);
                }
            }
        }
        const int gk = k0 + b_row;
        if (cols_in && gk < K) {
            const GT *p = B + ((int64_t)gk * ldb + n0 + b_col) * eb;
#pragma unroll
            for (int c = 0; c < EB; ++c) {
                rb_r[c] = p[c * SB * eb];
                if constexpr (BC) rb_i[c] = p[c * SB * eb + 1];
                else rb_i[c] = T(0);
            }
        } else {
#pragma unroll
            for (int c = 0; c < EB; ++c) {
                const int gc = n0 + b_col + c * SB;
                if (gk < K && gc < N) {
                    const GT *p = B + ((int64_t)gk * ldb + gc) * eb;
                    rb_r[c] = p[0];
                    if constexpr (BC) rb_i[c] = p[1];
                    else rb_i[c] = T(0);
                } else {
                    rb_r[c] = T(0);
                    rb_i[c] = T(0);
                }
            }
        }
    };
    auto lstore = [&](int b) {
#pragma unroll
        for (int c = 0; c < EA; ++c) {
            if constexpr (AC) Ac[b][a_k + c][a_row] = T2{ra_r[c], ra_i[c]};
            else Ar[b][a_k + c][a_row] = ra_r[c];
        }
#pragma unroll
        for (int c = 0; c < EB; ++c) {
            if constexpr (BC) Bc[b][b_row][b_col + c * SB] = T2{rb_r[c], rb_i[c]};
            else Br[b][b_row][b_col + c * SB] = rb_r[c];
        }
    };
    // LDS double buffer: compute on one buffer while the next K step is
    // written into the other; one barrier per K step.
    gload(0);
    lstore(0);
    __syncthreads();
    int cur = 0;
    for (int k0 = 0; k0 < K; k0 += BK) {
        const bool more = k0 + BK < K;
        if (more) gload(k0 + BK);
#pragma unroll
        for (int kk = 0; kk < BK; kk += 4) {
            // a real A: k = 0 2 4 6, then 1 3 5 7 of each 8, as in rgemm_tile, so
            // that a product's bits do not tell which of the two formed it
            const int kl = AC ? kk + (lane >> 4) : (kk & ~7) + 2 * (lane >> 4) + ((kk >> 2) & 1);
            T ar[WM], ai[WM], br[WN], bi[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int r = wm * 16 * WM + i * 16 + (lane & 15);
                if constexpr (AC) {
                    const T2 a2 = Ac[cur][kl][r];
                    ar[i] = a2.x;
                    ai[i] = a2.y;
                } else {
                    ar[i] = Ar[cur][kl][r];
                    ai[i] = T(0);
                }
            }
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                const int c = wn * 16 * WN + j * 16 + (lane & 15);
                if constexpr (BC) {
                    const T2 b2 = Bc[cur][kl][c];
                    br[j] = b2.x;
                    bi[j] = b2.y;
                } else {
                    br[j] = Br[cur][kl][c];
                    bi[j] = T(0);
                }
            }
            // two passes so that no MFMA waits on the one issued just before it
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) {
                    accr[i][j] = Mfma<T>::op(ar[i], br[j], accr[i][j]);
                    if constexpr (BC) acci[i][j] = Mfma<T>::op(ar[i], bi[j], acci[i][j]);
                    else if constexpr (AC) acci[i][j] = Mfma<T>::op(ai[i], br[j], acci[i][j]);
                }
            if constexpr (AC && BC) {
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        accr[i][j] = Mfma<T>::op(-ai[i], bi[j], accr[i][j]);
                        acci[i][j] = Mfma<T>::op(ai[i], br[j], acci[i][j]);
                    }
            }
        }
        if (more) lstore(cur ^ 1);
        __syncthreads();
        cur ^= 1;
    }
    // epilogue: element e of a lane is row Mfma<T>::row(lane, e), column lane % 16
    // of its 16x16 block (operands: A[lane % 16][lane / 16], B[lane / 16][lane % 16])
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + wm * 16 * WM + i * 16 + Mfma<T>::row(lane, e);
                const int col = n0 + wn * 16 * WN + j * 16 + (lane & 15);
                if (row < M && col < N) {
                    GT *pc = C + ((int64_t)row * ldc + col) * ec;
                    T vr = alpha * accr[i][j][e], vi = alpha * acci[i][j][e];
                    if (beta != T(0)) {
                        vr += beta * pc[0];
                        if constexpr (CC) vi += beta * pc[1];
                    }
                    if (add_eye && row == col) vr += T(1);
                    pc[0] = vr;
                    if constexpr (CC) pc[1] = vi;
                    if (C32) {
                        float *q = C32 + ((int64_t)row * ldc + col) * 2;
                        q[0] = (float)vr;
                        q[1] = (float)vi;
                    }
                }
            }
}

// ------------------------------------------------------------------ complex FP64 products
// C = alpha A B + beta C, one 32 WM x 32 WN tile at (m0, n0).
//
// What bounds it: an FP64 MFMA 16x16x4 holds its SIMD for 64 cycles, and every
// other vector instruction of any wave on that SIMD takes cycles from it
// rather than hiding behind it (measured: an integer operation about 2, an
// FP64 addition 3.6, a 16-byte LDS read 7).  So the loop issues as little else
// as it can: the operands go from global memory to LDS by 16-byte direct
// copies (no staging registers, no LDS stores), already in the order the
// matrix cores take them, so that a fragment is one conflict-free 16-byte LDS
// read per value at a constant offset, and the tile is as large as the
// registers allow (each fragment then feeds more MFMAs).
//
// LDS holds "chunks" of 64 values (1 KB), one per 16 rows (columns) x 4 k:
// B's in lane order (lane l: k = l / 16, column l % 16), A's with the four k of
// a row side by side, so that four lanes of the copy read 64 contiguous bytes,
// and permuted within each row by (row / 4) % 4, which spreads the 16 lanes of
// a fragment read over all banks.  Two K steps of 8 are kept: one is computed
// while the next is copied; one barrier per step.
//
// M3: three real products per complex product,
// (a + ib)(c + id) = ac - bd + i[(a + b)(c + d) - ac - bd], instead of four:
// a quarter fewer matrix-core operations.  Normwise as accurate (the imaginary
// part of an entry loses relative accuracy only where it is small against
// |a||c| + |b||d|); the LU and the solves use it, the FP64 refinement residual
// does not.
//
// Measured (three products, in 8MNK): 1744 x 1744 x 256, 32 frequencies: 128x64
// 82.0 TF, 64x64 80.7, 64x32 76.7, against 67.3 for the 64x32 tile staged
// through registers; 256 x 2000 x 1744: 89.1, 83.6, 75.4 against 71.6; the
// K = 64 products of the 256-wide blocks 44-55 (HBM-bound on C).
//
// DMA = false (a pointer that is not 16-byte aligned, which the direct copies
// would need) loads through registers instead.
typedef double zd2 __attribute__((ext_vector_type(2)));
typedef double zd2u __attribute__((ext_vector_type(2), aligned(8)));
constexpr int ZBK = 8;  // K step

// Waits for this wave's direct copies and LDS reads, then for the other waves.
__device__ __forceinline__ void copies_done_barrier() {
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int WM, int WN, bool M3, bool DMA>
__device__ __forceinline__ void zgemm_tile(int M, int N, int K, double alpha, const dglobal<double> *A_, int64_t lda,
                                           const dglobal<double> *B_, int64_t ldb, double beta, dglobal<double> *C_,
                                           int64_t ldc, int m0, int n0) {
    typedef Mfma<double>::v4 v4;
    typedef dglobal<zd2u> G2;
    constexpr int BM = 32 * WM, BN = 32 * WN, KC = ZBK / 4;
    constexpr int CA = BM / 16 * KC, CB = BN / 16 * KC;  // chunks per stage
    constexpr int NA = CA / 4, NB4 = CB / 4;             // copied by each wave
    static_assert(CA % 4 == 0 && CB % 4 == 0, "whole chunks per wave");
    __shared__ zd2 lds[2][(CA + CB) * 64];
    const G2 *A = (const G2 *)A_, *B = (const G2 *)B_;
    G2 *C = (G2 *)C_;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // this lane's value of each chunk its wave copies; rows and columns past
    // the edge repeat the last one (their results are not stored)
    const int ar = lane >> 2, ak = (lane & 3) ^ ((lane >> 4) & 3);
    const int bk = lane >> 4, bn = lane & 15;
    const G2 *pa[NA], *pb[NB4];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int c = wave * NA + i;
        pa[i] = A + (int64_t)min(m0 + (c / KC) * 16 + ar, M - 1) * lda + (c % KC) * 4 + ak;
    }
#pragma unroll
    for (int i = 0; i < NB4; ++i) {
        const int c = wave * NB4 + i;
        pb[i] = B + (int64_t)((c / (BN / 16)) * 4 + bk) * ldb + min(n0 + (c % (BN / 16)) * 16 + bn, N - 1);
    }
    // M3: accr = sum a c, acci = sum b d, accs = sum (a + b)(c + d)
    v4 accr[WM][WN], acci[WM][WN], accs[M3 ? WM : 1][M3 ? WN : 1];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            accr[i][j] = v4{0, 0, 0, 0};
            acci[i][j] = v4{0, 0, 0, 0};
            if constexpr (M3) accs[i][j] = v4{0, 0, 0, 0};
        }
    auto copy = [&](const G2 *g, zd2 *l) {
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (DMA) {
            __builtin_amdgcn_global_load_lds((const dglobal<uint32_t> *)g,
                                             (__attribute__((address_space(3))) uint32_t *)l, 16, 0, 0);
        } else {
            l[lane] = *g;
        }
#else
        l[lane] = *g;
#endif
    };
    auto stage = [&](int s) {
        zd2 *base = lds[s];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            copy(pa[i], base + (wave * NA + i) * 64);
            pa[i] += ZBK;
        }
#pragma unroll
        for (int i = 0; i < NB4; ++i) {
            copy(pb[i], base + (CA + wave * NB4 + i) * 64);
            pb[i] += ZBK * ldb;
        }
    };
    const int fa = 4 * (lane & 15) + ((lane >> 4) ^ ((lane >> 2) & 3));
    auto compute = [&](int s) {
        const zd2 *base = lds[s];
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            zd2 a[WM], b[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) a[i] = base[((wm * WM + i) * KC + q) * 64 + fa];
#pragma unroll
            for (int j = 0; j < WN; ++j) b[j] = base[(CA + q * (BN / 16) + wn * WN + j) * 64 + lane];
            if constexpr (M3) {
                // three passes, each over every block, so that no MFMA waits
                // on the one issued just before it
                double sa[WM], sb[WN];
#pragma unroll
                for (int i = 0; i < WM; ++i) sa[i] = a[i].x + a[i].y;
#pragma unroll
                for (int j = 0; j < WN; ++j) sb[j] = b[j].x + b[j].y;
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) accr[i][j] = Mfma<double>::op(a[i].x, b[j].x, accr[i][j]);
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) acci[i][j] = Mfma<double>::op(a[i].y, b[j].y, acci[i][j]);
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) accs[i][j] = Mfma<double>::op(sa[i], sb[j], accs[i][j]);
            } else {
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        accr[i][j] = Mfma<double>::op(a[i].x, b[j].x, accr[i][j]);
                        acci[i][j] = Mfma<double>::op(a[i].x, b[j].y, acci[i][j]);
                    }
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j) {
                        accr[i][j] = Mfma<double>::op(-a[i].y, b[j].y, accr[i][j]);
                        acci[i][j] = Mfma<double>::op(a[i].y, b[j].x, acci[i][j]);
                    }
            }
        }
    };
    const int nfull = K / ZBK;
    if (nfull > 0) stage(0);
    int cur = 0;
    for (int k = 0; k < nfull; ++k) {
        copies_done_barrier();
        if (k + 1 < nfull) stage(cur ^ 1);
        compute(cur);
        cur ^= 1;
    }
    if (nfull * ZBK < K) {
        // the last, partial step: zeros past K, into the buffer nobody reads
        const int k0 = nfull * ZBK;
        zd2 *base = lds[cur];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int c = wave * NA + i, k = k0 + (c % KC) * 4 + ak;
            zd2 x{0, 0};
            if (k < K) x = *pa[i];
            base[c * 64 + lane] = x;
        }
#pragma unroll
        for (int i = 0; i < NB4; ++i) {
            const int c = wave * NB4 + i, k = k0 + (c / (BN / 16)) * 4 + bk;
            zd2 x{0, 0};
            if (k < K) x = *pb[i];
            base[(CA + c) * 64 + lane] = x;
        }
        copies_done_barrier();
        compute(cur);
    }
    // every read of B is done before C, which may be B, is written
    copies_done_barrier();
    // element e of a lane is row lane / 16 + 4 e, column lane % 16 of its
    // 16x16 block (operands: A[lane % 16][lane / 16], B[lane / 16][lane % 16])
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + (wm * WM + i) * 16 + Mfma<double>::row(lane, e);
                const int col = n0 + (wn * WN + j) * 16 + (lane & 15);
                if (row < M && col < N) {
                    G2 *pc = C + (int64_t)row * ldc + col;
                    double vr, vi;
                    if constexpr (M3) {
                        vr = alpha * (accr[i][j][e] - acci[i][j][e]);
                        vi = alpha * (accs[i][j][e] - accr[i][j][e] - acci[i][j][e]);
                    } else {
                        vr = alpha * accr[i][j][e];
                        vi = alpha * acci[i][j][e];
                    }
                    if (beta != 0.0) {
                        const zd2 c = *pc;
                        vr += beta * c.x;
                        vi += beta * c.y;
                    }
                    *pc = zd2{vr, vi};
                }
            }
}

// Workgroup l of a launch (dealt to XCD l mod 8) takes tile
// (l mod 8) n / 8 + l / 8: each XCD works through a contiguous run of tiles,
// consecutive tiles sharing an A row band in that XCD's L2.
template <int WM, int WN, int OCC, bool M3, bool DMA>
__global__ __launch_bounds__(256, OCC) void k_zgemm(int M, int N, int K, double alpha, const double *A, int64_t lda,
                                                    int64_t sA, const double *B, int64_t ldb, int64_t sB, double beta,
                                                    double *C, int64_t ldc, int64_t sC) {
    const int gx = gridDim.x, gy = gridDim.y;
    const int64_t nt = (int64_t)gx * gy * gridDim.z;
    const int64_t l = blockIdx.x + (int64_t)gx * (blockIdx.y + (int64_t)gy * blockIdx.z);
    const int64_t n8 = nt / 8, t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;
    const int64_t bz = t / ((int64_t)gx * gy);
    zgemm_tile<WM, WN, M3, DMA>(M, N, K, alpha, (const dglobal<double> *)A + bz * sA * 2, lda,
                                (const dglobal<double> *)B + bz * sB * 2, ldb, beta,
                                (dglobal<double> *)C + bz * sC * 2, ldc, (int)((t / gx) % gy) * 32 * WM,
                                (int)(t % gx) * 32 * WN);
}

// ------------------------------------------------------------------ real FP64 products
// The same scheme for a real B, whose 16-byte copies carry two neighbouring
// columns (the MFMA's 16 columns are then every second one of 32), and
//   AC = false: a real A, whose copies carry two neighbouring k.  K advances 16
//     (8 for 128x128); within each 8 the matrix cores take k = 0 2 4 6, then
//     1 3 5 7.  A complex B is a real one with twice the columns.
//   AC = true: a complex A as in zgemm_tile, K advances 8.
// The copies need 16-byte aligned rows: even leading dimensions, and for an odd
// N a row of B that can be read one value past it (ldb > N).  MIR: row r >= 1
// of C is also written, conjugated, r rows before C's first row (C(-omega) =
// C(omega)* for a C whose rows are omega_r on a symmetric mesh starting at
// omega = 0).
//
// Measured against the tile staged through registers (gemm_tile), real A:
// 2000^3 x 24: 128x128 68.0 TF, 128x64 65.9, 64x64 60.3, staged 54.9;
// 1104 x 2208 x 1104 x 24: 61.7, 64.5, 61.6, staged 54.2.  The Cauchy product
// (512 x 4e6 x 192) gains little, 33.4 -> 32.4 ms: it writes 65 GB.
template <bool AC, int WM, int WN, int BK, bool MIR>
__device__ __forceinline__ void rgemm_tile(int M, int N, int K, double alpha, const dglobal<double> *A, int64_t lda,
                                           const dglobal<double> *B, int64_t ldb, double beta, dglobal<double> *C,
                                           int64_t ldc, int add_eye, float *C32, int m0, int n0) {
    typedef Mfma<double>::v4 v4;
    typedef dglobal<zd2u> G2;
    typedef dglobal<double> GD;
    constexpr int BM = 32 * WM, BN = 32 * WN, WP = WN / 2;
    constexpr int KA = AC ? 4 : 8;               // k per chunk of A
    constexpr int CA = BM / 16 * (BK / KA);      // chunks of 64 16-byte values per stage
    constexpr int CB = BN / 32 * (BK / 4);       // (B: 4 k x 32 columns)
    constexpr int NA = CA / 4, NB4 = CB / 4;     // copied by each wave
    constexpr int NP = AC ? 2 : 1;               // real and imaginary part of C
    static_assert(WN % 2 == 0 && CA % 4 == 0 && CB % 4 == 0, "whole chunks per wave");
    __shared__ zd2 lds[2][(CA + CB) * 64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // this lane's value of a chunk of A (rows as in zgemm_tile) ...
    const int ar = lane >> 2, aq = (lane & 3) ^ ((lane >> 4) & 3);
    auto a_at = [&](int c, int &row, int &k) {
        row = m0 + (c / (BK / KA)) * 16 + ar;
        k = (c % (BK / KA)) * KA + (AC ? aq : 2 * aq);
    };
    // ... and of B: chunk c holds the k of step c / (BN / 32): for a real A the
    // even or the odd k of an 8
    auto b_at = [&](int c, int &k, int &col) {
        const int st = c / (BN / 32);
        k = AC ? 4 * st + (lane >> 4) : 8 * (st >> 1) + 2 * (lane >> 4) + (st & 1);
        col = n0 + (c % (BN / 32)) * 32 + 2 * (lane & 15);
    };
    const GD *pa[NA], *pb[NB4];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        int row, k;
        a_at(wave * NA + i, row, k);
        pa[i] = A + ((int64_t)min(row, M - 1) * lda + k) * (AC ? 2 : 1);
    }
#pragma unroll
    for (int i = 0; i < NB4; ++i) {
        int k, col;
        b_at(wave * NB4 + i, k, col);
        pb[i] = B + (int64_t)k * ldb + min(col, (N - 1) & ~1);
    }
    v4 acc[NP][WM][WN];
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int j = 0; j < WN; ++j) acc[p][i][j] = v4{0, 0, 0, 0};
    auto stage = [&](int s) {
        zd2 *base = lds[s];
#if defined(__HIP_DEVICE_COMPILE__)
        typedef __attribute__((address_space(3))) uint32_t L;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            __builtin_amdgcn_global_load_lds((const dglobal<uint32_t> *)pa[i], (L *)(base + (wave * NA + i) * 64), 16,
                                             0, 0);
            pa[i] += BK * (AC ? 2 : 1);
        }
#pragma unroll
        for (int i = 0; i < NB4; ++i) {
            __builtin_amdgcn_global_load_lds((const dglobal<uint32_t> *)pb[i], (L *)(base + (CA + wave * NB4 + i) * 64),
                                             16, 0, 0);
            pb[i] += BK * ldb;
        }
#endif
    };
    const int fa = 4 * (lane & 15) + ((lane >> 4) ^ ((lane >> 2) & 3));
    auto compute = [&](int s) {
        const zd2 *base = lds[s];
#pragma unroll
        for (int q = 0; q < BK / KA; ++q) {
            zd2 a[WM];
#pragma unroll
            for (int i = 0; i < WM; ++i) a[i] = base[((wm * WM + i) * (BK / KA) + q) * 64 + fa];
#pragma unroll
            for (int t = 0; t < KA / 4; ++t) {
                zd2 b[WP];
#pragma unroll
                for (int j = 0; j < WP; ++j)
                    b[j] = base[(CA + (q * (KA / 4) + t) * (BN / 32) + wn * WP + j) * 64 + lane];
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int i = 0; i < WM; ++i) {
                        const double x = (AC ? p : t) ? a[i].y : a[i].x;
#pragma unroll
                        for (int j = 0; j < WP; ++j) {
                            acc[p][i][2 * j] = Mfma<double>::op(x, b[j].x, acc[p][i][2 * j]);
                            acc[p][i][2 * j + 1] = Mfma<double>::op(x, b[j].y, acc[p][i][2 * j + 1]);
                        }
                    }
            }
        }
    };
    const int nfull = K / BK;
    if (nfull > 0) stage(0);
    int cur = 0;
    for (int k = 0; k < nfull; ++k) {
        copies_done_barrier();
        if (k + 1 < nfull) stage(cur ^ 1);
        compute(cur);
        cur ^= 1;
    }
    if (nfull * BK < K) {
        // the last, partial step: zeros past K, into the buffer nobody reads
        const int left = K - nfull * BK;
        zd2 *base = lds[cur];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            int row, k;
            a_at(wave * NA + i, row, k);
            zd2 x{0, 0};
            if (k < left) {
                x.x = pa[i][0];
                if (AC || k + 1 < left) x.y = pa[i][1];
            }
            base[(wave * NA + i) * 64 + lane] = x;
        }
#pragma unroll
        for (int i = 0; i < NB4; ++i) {
            int k, col;
            b_at(wave * NB4 + i, k, col);
            zd2 x{0, 0};
            if (k < left) {
                x.x = pb[i][0];
                if (col + 1 < N) x.y = pb[i][1];
            }
            base[(CA + wave * NB4 + i) * 64 + lane] = x;
        }
        copies_done_barrier();
        compute(cur);
    }
    // every read of A and B is done before C, which may be one of them, is written
    copies_done_barrier();
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WP; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + (wm * WM + i) * 16 + Mfma<double>::row(lane, e);
                const int col = n0 + (wn * WP + j) * 32 + 2 * (lane & 15);
                if (row >= M || col >= N) continue;
                if constexpr (AC) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (col + h >= N) continue;
                        G2 *pc = (G2 *)C + (int64_t)row * ldc + col + h;
                        zd2 v{alpha * acc[0][i][2 * j + h][e], alpha * acc[NP - 1][i][2 * j + h][e]};
                        if (beta != 0.0) {
                            const zd2 c = *pc;
                            v.x += beta * c.x;
                            v.y += beta * c.y;
                        }
                        *pc = v;
                        if (MIR && row >= 1) *((G2 *)C + (col + h - (int64_t)row * ldc)) = zd2{v.x, -v.y};
                    }
                } else {
                    GD *pc = C + (int64_t)row * ldc + col;
                    zd2 v{alpha * acc[0][i][2 * j][e], alpha * acc[0][i][2 * j + 1][e]};
                    const bool two = col + 1 < N;
                    if (beta != 0.0) {
                        v.x += beta * pc[0];
                        if (two) v.y += beta * pc[1];
                    }
                    if (add_eye && col == 2 * row) v.x += 1.0;  // complex C: its real diagonal
                    if (two) *(G2 *)pc = v;
                    else pc[0] = v.x;
                    if (C32) {
                        float *q = C32 + (int64_t)row * ldc + col;
                        q[0] = (float)v.x;
                        if (two) q[1] = (float)v.y;
                    }
                }
            }
}

// BYCOL: tiles column band by column band (for a B much larger than A: each
// slice of B is read from HBM once), else row band by row band.
template <bool AC, int WM, int WN, int BK, int OCC, bool BYCOL, bool MIR>
__global__ __launch_bounds__(256, OCC) void k_rgemm(int M, int N, int K, double alpha, const double *A, int64_t lda,
                                                    int64_t sA, const double *B, int64_t ldb, int64_t sB, double beta,
                                                    double *C, int64_t ldc, int64_t sC, int add_eye, float *C32,
                                                    int64_t sC32) {
    const int gx = gridDim.x, gy = gridDim.y;
    const int64_t nt = (int64_t)gx * gy * gridDim.z;
    const int64_t l = blockIdx.x + (int64_t)gx * (blockIdx.y + (int64_t)gy * blockIdx.z);
    const int64_t n8 = nt / 8, t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;
    const int64_t bz = t / ((int64_t)gx * gy);
    const int by = (int)(BYCOL ? t % gy : (t / gx) % gy), bx = (int)(BYCOL ? (t / gy) % gx : t % gx);
    constexpr int e = AC ? 2 : 1;
    rgemm_tile<AC, WM, WN, BK, MIR>(M, N, K, alpha, (const dglobal<double> *)A + bz * sA * e, lda,
                                    (const dglobal<double> *)B + bz * sB, ldb, beta,
                                    (dglobal<double> *)C + bz * sC * e, ldc, add_eye, C32 ? C32 + bz * sC32 : nullptr,
                                    by * 32 * WM, bx * 32 * WN);
}

// Whether rgemm_tile can take these operands (see there).
bool rgemm_ok(int N, const void *A, int64_t lda, int64_t sA, bool ac, const void *B, int64_t ldb, int64_t sB) {
    const bool a_even = ac || ((lda | sA) & 1) == 0;
    return (((uintptr_t)A | (uintptr_t)B) & 15) == 0 && a_even && ((ldb | sB) & 1) == 0 && ((N & 1) == 0 || ldb > N);
}

// XR: workgroups are dealt to the eight XCDs in turn, each with its own L2, so
// each XCD gets a contiguous range of tiles, row band by row band (tiles sharing
// an A row band share that XCD's L2); else the tiles as launched.
template <typename T, bool AC, bool BC, int WM, int WN, int BK, int OCC, bool XR>
__global__ __launch_bounds__(256, OCC) void k_gemm(int M, int N, int K, T alpha, const T *__restrict__ A, int64_t lda,
                                                 int64_t sA, const T *B, int64_t ldb, int64_t sB, T beta,
                                                 T *C, int64_t ldc, int64_t sC, int add_eye, float *C32,
                                                 int64_t sC32) {
    constexpr int ea = AC ? 2 : 1, eb = BC ? 2 : 1, ec = (AC || BC) ? 2 : 1;
    int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    if constexpr (XR) {
        const int gx = gridDim.x, gy = gridDim.y;
        const int64_t nt = (int64_t)gx * gy * gridDim.z, l = bx + (int64_t)gx * (by + (int64_t)gy * bz);
        const int64_t n8 = nt / 8, t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;
        bx = (int)(t % gx);
        by = (int)((t / gx) % gy);
        bz = (int)(t / ((int64_t)gx * gy));
    }
    A += (int64_t)bz * sA * ea;
    B += (int64_t)bz * sB * eb;
    C += (int64_t)bz * sC * ec;
    if (C32) C32 += (int64_t)bz * sC32 * 2;
    gemm_tile<T, AC, BC, WM, WN, BK>(M, N, K, alpha, A, lda, B, ldb, beta, C, ldc, add_eye, C32, by * 32 * WM,
                                     bx * 32 * WN);
}

// Tile t of a multi-product launch: its item (searched from item a up; the
// items are ordered by their first tile) and the tile within it.
template <typename T, int WM, int WN, int BK, bool M3>
__device__ __forceinline__ void item_tile(const GemmItem *__restrict__ items, int n_items, int64_t t, int &a) {
    int b = n_items - 1;
    while (a < b) {
        const int m = (a + b + 1) >> 1;
        if (items[m].t0 <= t) a = m;
        else b = m - 1;
    }
    const GemmItem g = items[a];
    const int64_t r = t - g.t0, per = (int64_t)g.tx * g.ty;
    const int bz = (int)(r / per);
    const int64_t rr = r - bz * per;
    const int by = (int)(rr / g.tx), bx = (int)(rr % g.tx);
    // operands through global-address-space pointers (see dglobal)
    typedef dglobal<T> GT;
    const GT *Ap = (const GT *)g.A + (int64_t)bz * g.sA * 2;
    const GT *Bp = (const GT *)g.B + (int64_t)bz * g.sB * 2;
    GT *Cp = (GT *)g.C + (int64_t)bz * g.sC * 2;
    if constexpr (sizeof(T) == 8)
        zgemm_tile<WM, WN, M3, true>(g.M, g.N, g.K, g.alpha, Ap, g.lda, Bp, g.ldb, g.beta, Cp, g.ldc, by * 32 * WM,
                                     bx * 32 * WN);
    else
        gemm_tile<T, true, true, WM, WN, BK, GT>(g.M, g.N, g.K, (T)g.alpha, Ap, g.lda, Bp, g.ldb, (T)g.beta, Cp, g.ldc,
                                                 0, nullptr, by * 32 * WM, bx * 32 * WN);
}

// Many products in one launch, one tile per workgroup, the hardware
// dispatcher handing out the tiles: workgroup l (dealt to XCD l mod 8) takes
// tile (l mod 8) n/8 + l/8, so each XCD works through a contiguous run of
// tiles (consecutive tiles share an A row band, in that XCD's L2).
template <typename T, int WM, int WN, int BK, int OCC, bool M3>
__global__ __launch_bounds__(256, OCC) void k_gemm_group(const GemmItem *__restrict__ items, int n_items,
                                                       int64_t n_tiles) {
    const int64_t l = blockIdx.x, n8 = n_tiles / 8;
    const int64_t t = l < 8 * n8 ? (l % 8) * n8 + l / 8 : l;
    int a = 0;
    item_tile<T, WM, WN, BK, M3>(items, n_items, t, a);
}

// Workgroup barrier that orders LDS accesses only: unlike __syncthreads it
// does not wait for outstanding global stores (a tile's results) to land.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
}

// Persistent form of the same: the tiles are handed out by eight work queues,
// queue q owning the tiles [q n / 8, (q + 1) n / 8) in order.  A workgroup
// pulls from the queue of its XCD (workgroups are dealt to the XCDs in turn),
// then from the others; it leaves when all eight are empty, so every
// workgroup ends.  queue: eight counters, zero at launch.  On the LU's
// products it runs about a tenth slower than k_gemm_group, most likely
// because a wave's memory operations complete in order: the first loads of a
// workgroup's next tile wait for its previous tile's result stores to drain,
// which a newly dispatched workgroup does not.
template <typename T, int WM, int WN, int BK, int OCC, bool M3>
__global__ __launch_bounds__(256, OCC) void k_gemm_queue(const GemmItem *__restrict__ items, int n_items,
                                                       int64_t n_tiles, unsigned *__restrict__ queue) {
    __shared__ int64_t s_t;
    const int home = blockIdx.x & 7;
    for (int k = 0; k < 8; ++k) {
        const int q = (home + k) & 7;
        const int64_t lo = n_tiles * q / 8, hi = n_tiles * (q + 1) / 8;
        __syncthreads();  // everyone has read s_t
        if (threadIdx.x == 0) s_t = lo + (int64_t)atomicAdd(&queue[q], 1u);
        __syncthreads();
        int a = 0;  // item of the previous tile: one workgroup's tiles of a queue only grow
        for (;;) {
            // uniform over the workgroup: keep the tile index, the item
            // search and the item's fields in scalar registers
            const int64_t tv = s_t;
            const int64_t t = ((int64_t)__builtin_amdgcn_readfirstlane((int)(tv >> 32)) << 32) |
                              (unsigned)__builtin_amdgcn_readfirstlane((int)tv);
            if (t >= hi) break;
            // the next pull goes out now; its latency hides behind this
            // tile's first loads
            unsigned nxt = 0;
            if (threadIdx.x == 0) nxt = atomicAdd(&queue[q], 1u);
            item_tile<T, WM, WN, BK, M3>(items, n_items, t, a);
            lds_barrier();  // everyone has read s_t; the tile is done with LDS
            if (threadIdx.x == 0) s_t = lo + (int64_t)nxt;
            lds_barrier();
        }
    }
}

// ------------------------------------------------------------------ split-BF16 complex GEMM
// C = alpha A B + beta C for complex float, on v_mfma_f32_16x16x32_bf16: every
// float x is split into three bf16 terms x = h + m + l (round to nearest even
// at each step, so each remainder is exact in float), and the six products
// with h h, h m, m h, h l, m m, l h are accumulated in float.  The neglected
// terms are below 2^-24 relative, so the result is as accurate as an FP32
// product while running on the BF16 matrix rate.  Operand layout (measured on
// gfx950): lane l holds A[l % 16][8 (l / 16) + i] and B[8 (l / 16) + i][l % 16],
// i = 0..7; result element r of lane l is D[4 (l / 16) + r][l % 16].
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int XK = 32;  // complex k per stage

// What bounds it: per stage a wave has 96 products of 16 cycles, and beside them
// the splitting of 32 values per thread, which the matrix cores do not hide.  So
// the terms are rounded two at a time (v_cvt_pk_bf16_f32), the operands come in
// 16-byte loads where they lie inside the matrix, and a row's four 16-byte runs
// of k are kept in the order run ^ (row / 4) % 4, which spreads sixteen rows'
// reads (and B's writes) over all banks; two workgroups per CU, so that no
// accumulator is moved to the other half of the register file.  655 products,
// 128 frequencies: 105 us a launch (108.5 with single roundings, element loads
// and unswizzled rows).
__global__ __launch_bounds__(256, 2) void k_cgemm_bf16x(int M, int N, int K, float alpha, const float *__restrict__ A,
                                                        int64_t lda, int64_t sA, const float *B, int64_t ldb,
                                                        int64_t sB, float beta, float *C, int64_t ldc, int64_t sC) {
    // planes [term 0..2][part re/im][row or col 0..63][k 0..31] of bf16
    __shared__ __align__(16) unsigned short As[3][2][64][XK];
    __shared__ __align__(16) unsigned short Bs[3][2][64][XK];
    const int bz = blockIdx.z;
    A += (int64_t)bz * sA * 2;
    B += (int64_t)bz * sB * 2;
    C += (int64_t)bz * sC * 2;
    const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    f32x4 arr[2][2], aii[2][2], ari[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) arr[i][j] = aii[i][j] = ari[i][j] = f32x4{0, 0, 0, 0};
    // staging: A thread (row = tid / 4, k = (tid % 4) * 8 .. +8); B thread (col = tid % 64, k = (tid / 64) * 8 .. +8)
    const int a_row = tid >> 2, a_k = (tid & 3) * 8;
    const int b_col = tid & 63, b_k = (tid >> 6) * 8;
    float ar[8], ai[8], br[8], bi[8];
    typedef float f4u __attribute__((ext_vector_type(4), aligned(8)));
    auto gload = [&](int k0) {
        const int gr = m0 + a_row, gc = n0 + b_col;
        if (gr < M && k0 + a_k + 8 <= K) {
            const f4u *p = (const f4u *)(A + ((int64_t)gr * lda + k0 + a_k) * 2);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f4u v = p[c];
                ar[2 * c] = v.x;
                ai[2 * c] = v.y;
                ar[2 * c + 1] = v.z;
                ai[2 * c + 1] = v.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int gk = k0 + a_k + c;
                ar[c] = ai[c] = 0.f;
                if (gr < M && gk < K) {
                    const float *p = A + ((int64_t)gr * lda + gk) * 2;
                    ar[c] = p[0];
                    ai[c] = p[1];
                }
            }
        }
        if (k0 + XK <= K) {  // (a column past N: the last one's values, not stored)
            const float *p = B + ((int64_t)(k0 + b_k) * ldb + min(gc, N - 1)) * 2;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                br[c] = p[2 * c * ldb];
                bi[c] = p[2 * c * ldb + 1];
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int gk = k0 + b_k + c;
                br[c] = bi[c] = 0.f;
                if (gc < N && gk < K) {
                    const float *p = B + ((int64_t)gk * ldb + gc) * 2;
                    br[c] = p[0];
                    bi[c] = p[1];
                }
            }
        }
    };
    // eight k of one row or column: x = h + m + l, term by term
    auto split_store = [&](unsigned short (*P)[2][64][XK], int part, int rc, int k, const float *x) {
        bf16x8 t[3];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            t[0][c] = (__bf16)x[c];
            const float r1 = x[c] - (float)t[0][c];
            t[1][c] = (__bf16)r1;
            t[2][c] = (__bf16)(r1 - (float)t[1][c]);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x8 *>(&P[q][part][rc][k ^ (8 * ((rc >> 2) & 3))]) = t[q];
    };
    const int fk = 8 * ((lane >> 4) ^ ((lane >> 2) & 3));  // where a fragment row's run of k lies
    gload(0);
    for (int k0 = 0; k0 < K; k0 += XK) {
        __syncthreads();
        split_store(As, 0, a_row, a_k, ar);
        split_store(As, 1, a_row, a_k, ai);
        split_store(Bs, 0, b_col, b_k, br);
        split_store(Bs, 1, b_col, b_k, bi);
        __syncthreads();
        if (k0 + XK < K) gload(k0 + XK);
        // B fragments of all three terms for both column blocks
        bf16x8 fb[3][2][2];  // [term][part][block j]
#pragma unroll
        for (int t = 0; t < 3; ++t)
#pragma unroll
            for (int part = 0; part < 2; ++part)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    fb[t][part][j] = *reinterpret_cast<const bf16x8 *>(
                        &Bs[t][part][wn * 32 + j * 16 + (lane & 15)][fk]);
        // A term t pairs with B terms q, t + q <= 2
#pragma unroll
        for (int t = 0; t < 3; ++t) {
            bf16x8 fa[2][2];  // [part][block i]
#pragma unroll
            for (int part = 0; part < 2; ++part)
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    fa[part][i] = *reinterpret_cast<const bf16x8 *>(
                        &As[t][part][wm * 32 + i * 16 + (lane & 15)][fk]);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                if (t + q > 2) continue;
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        arr[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][i], fb[q][0][j], arr[i][j], 0, 0, 0);
                        aii[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[1][i], fb[q][1][j], aii[i][j], 0, 0, 0);
                        ari[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[0][i], fb[q][1][j], ari[i][j], 0, 0, 0);
                        ari[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[1][i], fb[q][0][j], ari[i][j], 0, 0, 0);
                    }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int row = m0 + wm * 32 + i * 16 + 4 * (lane >> 4) + e;
                const int col = n0 + wn * 32 + j * 16 + (lane & 15);
                if (row < M && col < N) {
                    float *pc = C + ((int64_t)row * ldc + col) * 2;
                    float vr = alpha * (arr[i][j][e] - aii[i][j][e]);
                    float vi = alpha * ari[i][j][e];
                    if (beta != 0.f) {
                        vr += beta * pc[0];
                        vi += beta * pc[1];
                    }
                    pc[0] = vr;
                    pc[1] = vi;
                }
            }
}

// A = 1 - diag(lam) chi0 (compressed metric), optional complex-float copy.
// Grid: x = 256-column blocks, y = rows, z = batch entries (grid strides).
__global__ void k_formA_diag(int n, int batch, const double *__restrict__ lam, const zdbl *__restrict__ chi0,
                             int64_t s_chi, zdbl *__restrict__ A, int64_t s_A, zflt *A32, int64_t s_A32) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= n) return;
    for (int b = blockIdx.z; b < batch; b += gridDim.z)
        for (int i = blockIdx.y; i < n; i += gridDim.y) {
            const int64_t idx = (int64_t)i * n + j;
            const zdbl c = chi0[b * s_chi + idx];
            zdbl a{-lam[i] * c.re, -lam[i] * c.im};
            if (i == j) a.re += 1.0;
            A[b * s_A + idx] = a;
            if (A32) A32[b * s_A32 + idx] = zflt{(float)a.re, (float)a.im};
        }
}

// Tile of the long complex products (M >= 256, K >= 128): < 0 the default.
// FP64: 0: 64x64, 1: 128x64, 2: 64x32, 3: 32x32 (K steps of 8); FP32: 0: 64x64
// K16, 1: 128x64 K8, 2: 64x32 K8, 3: 128x32 K8.  Per host thread, so the
// batched driver can record each molecule with its tuned tile.
thread_local int g_gemm_tile = -1;

const char *const kZgemmName[4] = {"zgemm_64x64", "zgemm_128x64", "zgemm_64x32", "zgemm_32x32"};
const char *const kCgemmName[4] = {"cgemm_64x64", "cgemm_128x64", "cgemm_64x32", "cgemm_128x32"};
const char *const kZgemm3Name[4] = {"zgemm3m_64x64", "zgemm3m_128x64", "zgemm3m_64x32", "zgemm3m_32x32"};
constexpr int kZRows[4] = {64, 128, 64, 32}, kZCols[4] = {64, 64, 32, 32};

// The tile of a complex FP64 product: the least padded area over the tile's
// rate.  Rates relative to 64x64 (84 TF on long products): 128x64 gains from
// K = 512 on (88 TF at 256 x 2000 x 1024 against 85; its longer fill and drain
// lose below), 64x32 and 32x32 run at 0.95 and 0.87 of it and win where they
// pad less (76 x 1100 x 1024: 57 TF by 32x32, 52 by 64x64) or, for 64x32, at
// M, K <= 64 (47 against 44 TF).  A launch that 64x64 tiles cannot spread over
// the 256 CUs (the lone frequency) takes 32x32.  in_place: C is B, so one tile
// must hold every row.
int ztile(int M, int N, int K, int batch, bool in_place) {
    const double rate[4] = {1.0, K >= 512 ? 1.04 : 0.96, M <= 64 && K <= 64 ? 1.04 : 0.95, 0.87};
    auto tiles = [&](int t) {
        return (double)((M + kZRows[t] - 1) / kZRows[t]) * ((N + kZCols[t] - 1) / kZCols[t]) * batch;
    };
    if (!in_place && tiles(0) < 256) return 3;
    int best = -1;
    double cost = 0;
    for (int t = 0; t < 4; ++t) {
        if (in_place && kZRows[t] < M) continue;
        if (t == 1 && tiles(1) < 1024) continue;  // two workgroups per CU: at least two rounds
        const double c = tiles(t) * kZRows[t] * kZCols[t] / rate[t];
        if (best < 0 || c < cost) {
            best = t;
            cost = c;
        }
    }
    return best;
}

// A real-B product by rgemm_tile (rgemm_ok): the tile of the least padded area
// over its rate (see there; the 128-wide ones need two rounds of two workgroups
// per CU to show theirs).
template <bool AC>
hipError_t launch_rgemm(hipStream_t st, int M, int N, int K, double alpha, const double *A, int64_t lda, int64_t sA,
                        const double *B, int64_t ldb, int64_t sB, double beta, double *C, int64_t ldc, int64_t sC,
                        int batch, int add_eye, float *C32, int64_t sC32) {
    const int bm[3] = {64, 128, 128}, bn[3] = {64, 64, 128};
    const double rate[3] = {1.0, 1.05, AC ? 0.0 : 1.08};
    int tile = 0;
    double cost = 0;
    for (int t = 0; t < 3; ++t) {
        if (rate[t] == 0) continue;
        const double tiles = (double)((M + bm[t] - 1) / bm[t]) * ((N + bn[t] - 1) / bn[t]) * batch;
        const double c = tiles * bm[t] * bn[t] / rate[t];
        if (t == 0 || (c < cost && tiles >= 1024)) {
            tile = t;
            cost = c;
        }
    }
#define GW_RGEMM(WM, WN, BK, OCC)                                                                                 \
    hipLaunchKernelGGL((k_rgemm<AC, WM, WN, BK, OCC, false, false>), dim3((N + 32 * WN - 1) / (32 * WN),          \
                       (M + 32 * WM - 1) / (32 * WM), batch), dim3(256), 0, st, M, N, K, alpha, A, lda, sA, B, ldb, \
                       sB, beta, C, ldc, sC, add_eye, C32, sC32)
    if constexpr (AC) {
        if (tile == 1) GW_RGEMM(4, 2, 8, 2);
        else GW_RGEMM(2, 2, 8, 3);
    } else {
        if (tile == 2) GW_RGEMM(4, 4, 8, 2);
        else if (tile == 1) GW_RGEMM(4, 2, 16, 2);
        else GW_RGEMM(2, 2, 16, 3);
    }
#undef GW_RGEMM
    return hipGetLastError();
}

// (in place: at most 128 rows, so that some tile holds them all)
template <bool M3>
hipError_t launch_zgemm_tile(hipStream_t st, int tile, bool dma, int M, int N, int K, double alpha, const double *A,
                             int64_t lda, int64_t sA, const double *B, int64_t ldb, int64_t sB, double beta, double *C,
                             int64_t ldc, int64_t sC, int batch) {
#define GW_ZGEMM(WM, WN, OCC, DMA)                                                                                    \
    hipLaunchKernelGGL((k_zgemm<WM, WN, OCC, M3, DMA>), dim3((N + 32 * WN - 1) / (32 * WN),                           \
                       (M + 32 * WM - 1) / (32 * WM), batch), dim3(256), 0, st, M, N, K, alpha, A, lda, sA, B, ldb, sB, \
                       beta, C, ldc, sC)
    if (!dma) GW_ZGEMM(4, 2, 2, false);
    else if (tile == 0) GW_ZGEMM(2, 2, 3, true);
    else if (tile == 1) GW_ZGEMM(4, 2, 2, true);
    else if (tile == 2) GW_ZGEMM(2, 1, 5, true);
    else GW_ZGEMM(1, 1, 8, true);
#undef GW_ZGEMM
    return hipGetLastError();
}

template <typename T, bool AC, bool BC, bool M3 = false>
hipError_t launch_gemm_t(hipStream_t st, int M, int N, int K, T alpha, const T *A, int64_t lda, int64_t sA,
                         const T *B, int64_t ldb, int64_t sB, T beta, T *C, int64_t ldc, int64_t sC, int batch,
                         int add_eye = 0, float *C32 = nullptr, int64_t sC32 = 0) {
    if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
    constexpr bool Z64 = AC && BC && sizeof(T) == 8;
    constexpr bool CF32 = AC && BC && sizeof(T) == 4;
    const bool tuned = g_gemm_tile >= 0 && g_gemm_tile <= 3;
    int tile;
    bool dma = false;
    if constexpr (Z64) {
        const bool big = M >= 256 && K >= 128;
        const bool in_place = (const void *)B == (const void *)C;
        if (in_place && M > 128) return hipErrorInvalidValue;
        tile = big && tuned ? g_gemm_tile : ztile(M, N, K, batch, in_place);
        dma = (((uintptr_t)A | (uintptr_t)B | (uintptr_t)C) & 15) == 0;
    } else if constexpr (CF32) {
        const bool big = M >= 256 && K >= 128;
        tile = big && tuned ? g_gemm_tile : (M >= 128 && K >= 64) ? 1 : 0;
    } else {
        tile = 0;
    }
    if (OpRecorder *rec = g_rec) {
        // lock-step recording: complex products become work-queue items, the
        // rest run as they are when their lock step comes
        if constexpr (Z64 || CF32) {
            RecOp o;
            o.kind = RecOp::GEMM;
            o.key = (Z64 ? (M3 ? QK_Z3M : QK_Z4M) : QK_C) * 4 + tile;
            o.g.A = A;
            o.g.B = B;
            o.g.C = C;
            o.g.lda = lda;
            o.g.ldb = ldb;
            o.g.ldc = ldc;
            o.g.sA = sA;
            o.g.sB = sB;
            o.g.sC = sC;
            o.g.alpha = (double)alpha;
            o.g.beta = (double)beta;
            o.g.M = M;
            o.g.N = N;
            o.g.K = K;
            o.g.batch = batch;
            o.flops = 8.0 * M * N * (double)K * batch;
            if (!add_eye && !C32 && (dma || !Z64)) {
                rec->ops.push_back(std::move(o));
                return hipSuccess;
            }
        }
        rec->other([=](hipStream_t s2) {
            return launch_gemm_t<T, AC, BC, M3>(s2, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch,
                                                add_eye, C32, sC32);
        });
        return hipSuccess;
    }
    ProfSink *prof = g_prof;
    const char *cls = nullptr;
    double flops = 0, bytes = 0;
    if (prof) {
        const bool dbl = sizeof(T) == 8;
        if (AC && BC) cls = dbl ? (M3 ? kZgemm3Name[tile] : kZgemmName[tile]) : kCgemmName[tile];
        else if (BC) cls = add_eye ? "formA" : "dzgemm";
        else if (AC) cls = "zdgemm";
        else cls = "dgemm";
        const double ea = sizeof(T) * (AC ? 2 : 1), eb = sizeof(T) * (BC ? 2 : 1), ec = sizeof(T) * ((AC || BC) ? 2 : 1);
        flops = (AC && BC ? 8.0 : (AC || BC) ? 4.0 : 2.0) * M * N * (double)K * batch;
        bytes = (double)M * K * ea * (sA ? batch : 1) + (double)K * N * eb * (sB ? batch : 1) +
                (double)M * N * ec * batch * (beta != T(0) ? 2 : 1);
    }
    ProfScope ps(st, cls ? cls : "", flops, bytes);
#define GW_GEMM(WM, WN, BK, OCC, XR)                                                                               \
    hipLaunchKernelGGL((k_gemm<T, AC, BC, WM, WN, BK, OCC, XR>), dim3((N + 32 * WN - 1) / (32 * WN),               \
                       (M + 32 * WM - 1) / (32 * WM), batch), dim3(256), 0, st, M, N, K, alpha, A, lda, sA, B, ldb, \
                       sB, beta, C, ldc, sC, add_eye, C32, sC32)
    if constexpr (Z64) {
        return launch_zgemm_tile<M3>(st, tile, dma, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch);
    } else if constexpr (CF32) {
        if (tile == 3) GW_GEMM(4, 1, 8, 4, true);
        else if (tile == 2) GW_GEMM(2, 1, 8, 4, true);
        else if (tile == 1) GW_GEMM(4, 2, 8, 2, false);
        else GW_GEMM(2, 2, 16, 2, false);
    } else {
        static_assert(sizeof(T) == 8, "real operands in FP64 only");
        // real A, complex B: a real product with twice the columns
        constexpr int eb = BC ? 2 : 1;
        if (rgemm_ok(N * eb, A, lda, sA, AC, B, ldb * eb, sB * eb))
            return launch_rgemm<AC>(st, M, N * eb, K, alpha, A, lda, sA, B, ldb * eb, sB * eb, beta, C, ldc * eb,
                                    sC * eb, batch, add_eye, C32, sC32 * 2);
        GW_GEMM(2, 2, 16, 2, false);
    }
#undef GW_GEMM
    return hipGetLastError();
}

}  // namespace

hipError_t launch_zgemm(hipStream_t st, int M, int N, int K, double alpha, const zdbl *A, int64_t lda, int64_t sA,
                        const zdbl *B, int64_t ldb, int64_t sB, double beta, zdbl *C, int64_t ldc, int64_t sC,
                        int batch) {
    return launch_gemm_t<double, true, true>(st, M, N, K, alpha, (const double *)A, lda, sA, (const double *)B, ldb,
                                             sB, beta, (double *)C, ldc, sC, batch);
}

// The products of the FP64 LU and solves: the three-product form.
hipError_t launch_zgemm_lu(hipStream_t st, int M, int N, int K, double alpha, const zdbl *A, int64_t lda,
                           int64_t sA, const zdbl *B, int64_t ldb, int64_t sB, double beta, zdbl *C, int64_t ldc,
                           int64_t sC, int batch) {
    return launch_gemm_t<double, true, true, true>(st, M, N, K, alpha, (const double *)A, lda, sA, (const double *)B,
                                                   ldb, sB, beta, (double *)C, ldc, sC, batch);
}

// C = alpha A B (beta = 0) for complex A (M x K, small) times real B (K x N,
// N large), tiles ordered column band by column band so each slice of B is
// read from HBM once: the Cauchy transform of the spectral bins on the
// A route (M frequencies, N matrix entries, K bins).  Row r >= 1 is also
// written, conjugated, at row -r (C's rows are the mesh points from omega = 0
// up; the rows before C are those of -omega).  B's rows are the caller's own,
// laid out for 16-byte copies.
hipError_t launch_zdgemm_mirror(hipStream_t st, int M, int N, int K, double alpha, const zdbl *A, int64_t lda,
                                const double *B, int64_t ldb, zdbl *C, int64_t ldc) {
    if (M <= 0 || N <= 0) return hipSuccess;
    if (!rgemm_ok(N, A, lda, 0, true, B, ldb, 0)) return hipErrorInvalidValue;
    ProfScope ps(st, "cauchy_gemm", 4.0 * M * (double)N * K, 8.0 * (double)K * N + 16.0 * (double)(2 * M - 1) * N);
    const int64_t z = 0;
    hipLaunchKernelGGL((k_rgemm<true, 4, 2, 8, 2, true, true>), dim3((N + 63) / 64, (M + 127) / 128, 1), dim3(256), 0,
                       st, M, N, K, alpha, (const double *)A, lda, z, B, ldb, z, 0.0, (double *)C, ldc, z, 0,
                       (float *)nullptr, z);
    return hipGetLastError();
}

// Complex-float products of the calling thread run as split-BF16 MFMA when set
// (the long products of the BF16x factorisation and solves).
thread_local bool g_cgemm_bf16x = false;

hipError_t launch_cgemm(hipStream_t st, int M, int N, int K, float alpha, const zflt *A, int64_t lda, int64_t sA,
                        const zflt *B, int64_t ldb, int64_t sB, float beta, zflt *C, int64_t ldc, int64_t sC,
                        int batch) {
    if (g_cgemm_bf16x && K >= 32) {
        if (M <= 0 || N <= 0 || batch <= 0) return hipSuccess;
        if (OpRecorder *rec = g_rec) {
            rec->other([=](hipStream_t s2) {
                OpRecorder *saved = g_rec;
                g_rec = nullptr;
                const bool prev = g_cgemm_bf16x;
                g_cgemm_bf16x = true;
                const hipError_t e = launch_cgemm(s2, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch);
                g_cgemm_bf16x = prev;
                g_rec = saved;
                return e;
            });
            return hipSuccess;
        }
        dim3 grid((N + 63) / 64, (M + 63) / 64, batch);
        ProfScope ps(st, "cgemm_bf16x", 8.0 * M * N * (double)K * batch,
                     8.0 * ((double)M * K + (double)K * N + (beta != 0.f ? 2.0 : 1.0) * M * N) * batch);
        hipLaunchKernelGGL(k_cgemm_bf16x, grid, dim3(256), 0, st, M, N, K, alpha, (const float *)A, lda, sA,
                           (const float *)B, ldb, sB, beta, (float *)C, ldc, sC);
        return hipGetLastError();
    }
    return launch_gemm_t<float, true, true>(st, M, N, K, alpha, (const float *)A, lda, sA, (const float *)B, ldb, sB,
                                            beta, (float *)C, ldc, sC, batch);
}

hipError_t launch_formA(hipStream_t st, int n, const double *v, int64_t ldv, int v_is_diag, const zdbl *chi0,
                        int64_t s_chi,
                        zdbl *A, int64_t s_A, zflt *A32, int64_t s_A32, int batch) {
    if (v_is_diag) {
        GW_DEFER(launch_formA(st, n, v, ldv, v_is_diag, chi0, s_chi, A, s_A, A32, s_A32, batch));
        const int xb = (n + 255) / 256, zb = std::min(batch, 65535);
        dim3 grid((unsigned)xb, (unsigned)std::max(1, std::min(n, 65536 / std::max(1, xb * zb))), (unsigned)zb);
        hipLaunchKernelGGL(k_formA_diag, grid, dim3(256), 0, st, n, batch, v, chi0, s_chi, A, s_A, A32, s_A32);
        return hipGetLastError();
    }
    // A = -v * chi0 + 1 (v real, shared by the batch: batch stride 0)
    return launch_gemm_t<double, false, true>(st, n, n, n, -1.0, v, ldv, 0, (const double *)chi0, n, s_chi, 0.0,
                                              (double *)A, n, s_A, batch, 1, (float *)A32, s_A32);
}

// R = v - A W: R <- v (complex), then R -= A W.
hipError_t launch_residual(hipStream_t st, int n, const double *v, int v_is_diag, const zdbl *A, int64_t sA,
                           const zdbl *W, int64_t sW, zdbl *R, int64_t sR, int batch) {
    hipError_t e = launch_init_rhs(st, n, v, v_is_diag, R, sR, batch);
    if (e != hipSuccess) return e;
    return launch_zgemm(st, n, n, n, -1.0, A, n, sA, W, n, sW, 1.0, R, n, sR, batch);
}

// Real-times-complex and complex-times-real products exposed for the compression path.
hipError_t launch_dzgemm(hipStream_t st, int M, int N, int K, double alpha, const double *A, int64_t lda, int64_t sA,
                         const zdbl *B, int64_t ldb, int64_t sB, double beta, zdbl *C, int64_t ldc, int64_t sC,
                         int batch) {
    return launch_gemm_t<double, false, true>(st, M, N, K, alpha, A, lda, sA, (const double *)B, ldb, sB, beta,
                                              (double *)C, ldc, sC, batch);
}
hipError_t launch_zdgemm(hipStream_t st, int M, int N, int K, double alpha, const zdbl *A, int64_t lda, int64_t sA,
                         const double *B, int64_t ldb, int64_t sB, double beta, zdbl *C, int64_t ldc, int64_t sC,
                         int batch) {
    return launch_gemm_t<double, true, false>(st, M, N, K, alpha, (const double *)A, lda, sA, B, ldb, sB, beta,
                                              (double *)C, ldc, sC, batch);
}
hipError_t launch_dgemm(hipStream_t st, int M, int N, int K, double alpha, const double *A, int64_t lda, int64_t sA,
                        const double *B, int64_t ldb, int64_t sB, double beta, double *C, int64_t ldc, int64_t sC,
                        int batch) {
    return launch_gemm_t<double, false, false>(st, M, N, K, alpha, A, lda, sA, B, ldb, sB, beta, C, ldc, sC, batch);
}

thread_local OpRecorder *g_rec = nullptr;

namespace {
// (WM, WN, BK, OCC) of each work-queue key: the tiles and occupancies
// launch_gemm_t picks for the product kind and tile.
struct QShape {
    int wm, wn, bk, occ;
};
QShape qshape(int key) {
    const int kind = key / 4, tile = key % 4;
    if (kind != QK_C) {
        if (tile == 3) return {1, 1, ZBK, 8};
        if (tile == 2) return {2, 1, ZBK, 5};
        if (tile == 1) return {4, 2, ZBK, 2};
        return {2, 2, ZBK, 3};
    }
    if (tile == 3) return {4, 1, 8, 4};
    if (tile == 2) return {2, 1, 8, 4};
    if (tile == 1) return {4, 2, 8, 2};
    return {2, 2, 16, 2};
}
}  // namespace

// OP(T, WM, WN, BK, OCC, M3) for the kernel of a work-queue key.
#define GW_QKEY(OP)                                             \
    do {                                                        \
        if (kind == QK_Z3M) {                                   \
            if (tile == 3) OP(double, 1, 1, ZBK, 8, true);      \
            else if (tile == 2) OP(double, 2, 1, ZBK, 5, true); \
            else if (tile == 1) OP(double, 4, 2, ZBK, 2, true); \
            else OP(double, 2, 2, ZBK, 3, true);                \
        } else if (kind == QK_Z4M) {                            \
            if (tile == 3) OP(double, 1, 1, ZBK, 8, false);     \
            else if (tile == 2) OP(double, 2, 1, ZBK, 5, false); \
            else if (tile == 1) OP(double, 4, 2, ZBK, 2, false); \
            else OP(double, 2, 2, ZBK, 3, false);               \
        } else {                                                \
            if (tile == 3) OP(float, 4, 1, 8, 4, false);        \
            else if (tile == 2) OP(float, 2, 1, 8, 4, false);   \
            else if (tile == 1) OP(float, 4, 2, 8, 2, false);   \
            else OP(float, 2, 2, 16, 2, false);                 \
        }                                                       \
    } while (0)

int gemm_queue_occupancy(int key) {
    // workgroups of this key resident on one CU, as the runtime computes it
    // from the kernel's registers and LDS (at least the launch bound's figure)
    int occ = 0;
    hipError_t e = hipErrorInvalidValue;
    const int kind = key / 4, tile = key % 4;
    if (kind == QK_SOLVE) return block_solve_occupancy(tile);
#define GW_QOCC(T, WM, WN, BK, OCC, M3) \
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, k_gemm_queue<T, WM, WN, BK, OCC, M3>, 256, 0)
    GW_QKEY(GW_QOCC);
#undef GW_QOCC
    return e == hipSuccess && occ > 0 ? occ : qshape(key).occ;
}
void gemm_queue_tile(int key, int *bm, int *bn) {
    if (key / 4 == QK_SOLVE) {  // a strip of all the block's rows
        *bm = 256;
        *bn = block_solve_columns();
        return;
    }
    const QShape q = qshape(key);
    *bm = 32 * q.wm;
    *bn = 32 * q.wn;
}

hipError_t launch_gemm_queue(hipStream_t st, int key, const GemmItem *items, int n_items, int64_t n_tiles,
                             unsigned *queue, int grid, double flops) {
    if (n_items <= 0 || n_tiles <= 0) return hipSuccess;
    if (key < 0 || key >= 16 || (!queue && n_tiles > INT32_MAX) || (queue && grid <= 0)) return hipErrorInvalidValue;
    const int kind = key / 4, tile = key % 4;
    static const char *const names[4] = {"zgemm3m_queue", "zgemm_queue", "cgemm_queue", "block_solve_queue"};
    ProfScope ps(st, names[kind], flops, 0.0);
    if (kind == QK_SOLVE) return launch_block_solve_group(st, tile, items, n_items, n_tiles);
#define GW_QGEMM(T, WM, WN, BK, OCC, M3)                                                                       \
    do {                                                                                                       \
        if (queue)                                                                                             \
            hipLaunchKernelGGL((k_gemm_queue<T, WM, WN, BK, OCC, M3>), dim3(grid), dim3(256), 0, st, items,    \
                               n_items, n_tiles, queue);                                                       \
        else                                                                                                   \
            hipLaunchKernelGGL((k_gemm_group<T, WM, WN, BK, OCC, M3>), dim3((unsigned)n_tiles), dim3(256), 0,  \
                               st, items, n_items, n_tiles);                                                   \
    } while (0)
    GW_QKEY(GW_QGEMM);
#undef GW_QGEMM
    return hipGetLastError();
}

}  // namespace gwk

namespace gwp {
void set_thread_gemm_tile(int tile) { gwk::g_gemm_tile = tile; }
bool set_thread_cgemm_bf16x(bool on) {
    const bool prev = gwk::g_cgemm_bf16x;
    gwk::g_cgemm_bf16x = on;
    return prev;
}
}  // namespace gwp
