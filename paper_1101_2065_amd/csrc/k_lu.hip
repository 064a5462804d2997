// Blocked right-looking LU with partial pivoting, batched over frequencies,
// and the matching solve, for W(w) = (1 - v chi0(w))^{-1} v (Section 2 eq.
// Coulombscreening; the inversion is the O(N^3) step the paper's Sections 1
// and 7.B point to).
//
// Panel width 64 (inside 256-wide blocks, see getrf_impl).  Per panel: one
// workgroup per frequency factors the
// (n - kb) x 64 panel column by column (pivot = largest |re| + |im|, ties to
// the lowest row), composes the 64 row exchanges into one list of
// (destination, source) rows, and inverts the 64x64 unit-lower L11 and the
// upper U11 in LDS.  The row exchanges are then applied to the rest of the
// matrix in one pass, U12 = L11^{-1} A12 and the trailing update
// A22 -= L21 U12 run on the MFMA GEMM.  The solve uses the stored inverses the
// same way, so every O(N^3) flop of factor and solve is an MFMA product.
#include "gw_internal.h"
#include "gw_prof.h"
#include "k_mfma.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <utility>

namespace gwk {

hipError_t launch_zgemm(hipStream_t st, int M, int N, int K, double alpha, const zdbl *A, int64_t lda, int64_t sA,
                        const zdbl *B, int64_t ldb, int64_t sB, double beta, zdbl *C, int64_t ldc, int64_t sC,
                        int batch);
hipError_t launch_cgemm(hipStream_t st, int M, int N, int K, float alpha, const zflt *A, int64_t lda, int64_t sA,
                        const zflt *B, int64_t ldb, int64_t sB, float beta, zflt *C, int64_t ldc, int64_t sC,
                        int batch);

namespace {

constexpr int NB = 64;         // panel width
constexpr int SWP = 1 + 4 * NB;  // per-frequency swap list: count, dst[2NB], src[2NB]

template <typename T>
struct Cx {
    T re, im;
};
template <typename T>
__device__ inline Cx<T> cmul(Cx<T> a, Cx<T> b) {
    return Cx<T>{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
template <typename T>
__device__ inline Cx<T> crcp(Cx<T> a) {
    const T d = a.re * a.re + a.im * a.im;
    return Cx<T>{a.re / d, -a.im / d};
}
// Workgroup barrier that orders LDS accesses only: unlike __syncthreads it
// does not wait for stores to global memory to land.
__device__ __forceinline__ void lds_barrier() {
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
#endif
}

template <typename T>
__global__ __launch_bounds__(512) void k_getf2(int n, int kb, int w, Cx<T> *A, int64_t sA, int32_t *ipiv,
                                               Cx<T> *Linv, Cx<T> *Uinv, int nblk, Cx<T> *S, int32_t *swp,
                                               int32_t *info) {
    __shared__ Cx<T> Ts[NB][NB];
    __shared__ Cx<T> Xs[NB][NB];
    __shared__ Cx<T> urow[NB];
    __shared__ T red_v[8];
    __shared__ int red_i[8];
    __shared__ int lpiv[NB];
    __shared__ int piv_s;
    __shared__ int zero_s;
    __shared__ int rows[2 * NB], cont[2 * NB];
    __shared__ Cx<T> dinv[NB];

    const int b = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    A += (int64_t)b * sA;
    ipiv += (int64_t)b * n;
    S += (int64_t)b * NB * n;
    swp += (int64_t)b * SWP;
    Linv += ((int64_t)b * nblk + kb / NB) * NB * NB;
    Uinv += ((int64_t)b * nblk + kb / NB) * NB * NB;
    const int m = n - kb;

    for (int64_t idx = tid; idx < (int64_t)m * w; idx += 512) {
        const int i = (int)(idx / w), c = (int)(idx % w);
        S[(int64_t)c * m + i] = A[(int64_t)(kb + i) * n + kb + c];
    }
    __syncthreads();

    for (int j = 0; j < w; ++j) {
        const Cx<T> *col = S + (int64_t)j * m;
        T best = T(-1);
        int bi = m;
        for (int i = j + tid; i < m; i += 512) {
            const Cx<T> z = col[i];
            const T v = fabs(z.re) + fabs(z.im);
            if (v > best) {
                best = v;
                bi = i;
            }
        }
        for (int off = 32; off > 0; off >>= 1) {
            const T ov = __shfl_xor(best, off);
            const int oi = __shfl_xor(bi, off);
            if (ov > best || (ov == best && oi < bi)) {
                best = ov;
                bi = oi;
            }
        }
        if (lane == 0) {
            red_v[wave] = best;
            red_i[wave] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            T bv = red_v[0];
            int bx = red_i[0];
            for (int q = 1; q < 8; ++q)
                if (red_v[q] > bv || (red_v[q] == bv && red_i[q] < bx)) {
                    bv = red_v[q];
                    bx = red_i[q];
                }
            if (bx >= m) bx = j;
            piv_s = bx;
            lpiv[j] = bx;
            zero_s = (bv == T(0));
            if (bv == T(0) && info[b] == 0) info[b] = kb + j + 1;
        }
        __syncthreads();
        const int piv = piv_s;
        if (piv != j) {
            for (int c = tid; c < w; c += 512) {
                Cx<T> *pc = S + (int64_t)c * m;
                const Cx<T> t = pc[j];
                pc[j] = pc[piv];
                pc[piv] = t;
            }
        }
        __syncthreads();
        if (!zero_s) {
            const Cx<T> inv = crcp(S[(int64_t)j * m + j]);
            if (tid > j && tid < w) urow[tid] = S[(int64_t)tid * m + j];
            __syncthreads();
            for (int i = j + 1 + tid; i < m; i += 512) {
                Cx<T> *pj = S + (int64_t)j * m;
                const Cx<T> l = cmul(pj[i], inv);
                pj[i] = l;
                for (int c = j + 1; c < w; ++c) {
                    Cx<T> *pc = S + (int64_t)c * m;
                    const Cx<T> u = urow[c];
                    const Cx<T> x = pc[i];
                    pc[i] = Cx<T>{x.re - (l.re * u.re - l.im * u.im), x.im - (l.re * u.im + l.im * u.re)};
                }
            }
        }
        __syncthreads();
    }

    // write the factored panel back, pivots as global rows
    for (int64_t idx = tid; idx < (int64_t)m * w; idx += 512) {
        const int i = (int)(idx / w), c = (int)(idx % w);
        A[(int64_t)(kb + i) * n + kb + c] = S[(int64_t)c * m + i];
    }
    if (tid < w) ipiv[kb + tid] = kb + lpiv[tid];
    // compose the row exchanges: new row dst = old row src
    if (tid == 0) {
        int nt = 0;
        for (int j = 0; j < w; ++j) {
            const int r1 = j, r2 = lpiv[j];
            if (r1 == r2) continue;
            int i1 = -1, i2 = -1;
            for (int t = 0; t < nt; ++t) {
                if (rows[t] == r1) i1 = t;
                if (rows[t] == r2) i2 = t;
            }
            if (i1 < 0) {
                rows[nt] = r1;
                cont[nt] = r1;
                i1 = nt++;
            }
            if (i2 < 0) {
                rows[nt] = r2;
                cont[nt] = r2;
                i2 = nt++;
            }
            const int t = cont[i1];
            cont[i1] = cont[i2];
            cont[i2] = t;
        }
        swp[0] = nt;
        for (int t = 0; t < nt; ++t) {
            swp[1 + t] = kb + rows[t];
            swp[1 + 2 * NB + t] = kb + cont[t];
        }
    }
    // diagonal block into LDS (row-major), zero padded
    for (int idx = tid; idx < NB * NB; idx += 512) {
        const int i = idx / NB, c = idx % NB;
        Ts[i][c] = (i < w && c < w) ? S[(int64_t)c * m + i] : Cx<T>{T(0), T(0)};
        Xs[i][c] = Cx<T>{T(0), T(0)};
    }
    __syncthreads();
    // L11^{-1}: unit lower, column c by forward substitution
    if (tid < w) {
        const int c = tid;
        Xs[c][c] = Cx<T>{T(1), T(0)};
        for (int i = c + 1; i < w; ++i) {
            T sr = 0, si = 0;
            for (int k = c; k < i; ++k) {
                const Cx<T> l = Ts[i][k], x = Xs[k][c];
                sr += l.re * x.re - l.im * x.im;
                si += l.re * x.im + l.im * x.re;
            }
            Xs[i][c] = Cx<T>{-sr, -si};
        }
    }
    if (tid < w) dinv[tid] = crcp(Ts[tid][tid]);
    __syncthreads();
    for (int idx = tid; idx < NB * NB; idx += 512) {
        Linv[idx] = Xs[idx / NB][idx % NB];
        Xs[idx / NB][idx % NB] = Cx<T>{T(0), T(0)};
    }
    __syncthreads();
    // U11^{-1}: upper, column c by back substitution
    if (tid < w) {
        const int c = tid;
        Xs[c][c] = dinv[c];
        for (int i = c - 1; i >= 0; --i) {
            T sr = 0, si = 0;
            for (int k = i + 1; k <= c; ++k) {
                const Cx<T> u = Ts[i][k], x = Xs[k][c];
                sr += u.re * x.re - u.im * x.im;
                si += u.re * x.im + u.im * x.re;
            }
            const Cx<T> d = dinv[i];
            Xs[i][c] = Cx<T>{-(sr * d.re - si * d.im), -(sr * d.im + si * d.re)};
        }
    }
    __syncthreads();
    for (int idx = tid; idx < NB * NB; idx += 512) Uinv[idx] = Xs[idx / NB][idx % NB];
}

// Left-looking panel factorisation with the active rows in registers.
// 512 threads; thread t owns panel rows i = t + 512 r (r < R), so the panel
// height m = n - kb must be at most 512 R.  What bounds it is latency: one
// workgroup works through 64 dependent columns, so every column has a single
// barrier and memory is only touched where its latency can be covered.
//
// Rows never move while the panel is factorised: a row keeps its place in
// memory and its thread, and carries its position, which a row exchange
// relabels.  The 64 columns are processed in chunks of BW (16 for R <= 2, 8
// for R = 4, else 4: registers): (1) the chunk's columns are loaded; (2) its U rows (positions
// < j0) by forward substitution with the unit-lower corner in LDS, one or two
// columns per wave, lane = position, each x_k broadcast from its lane once final;
// (3) the other rows are updated with L[:, 0:j0] U[0:j0, chunk]; (4) the chunk
// is factorised column by column in registers: each wave's largest
// |re| + |im| (ties to the lowest position) and that row go to LDS, one
// barrier, every wave picks the largest of the eight and updates its rows with
// it; (5) written back, without waiting for the stores: a wave reads only its
// own rows back, in order.  Finally the rows that ended elsewhere than they began
// are moved, once, and listed for the other columns, and the inverses of the
// 64x64 unit-lower L11 and upper U11 are formed in registers, eight columns
// per wave, lane = row.
//
// The loads of (1) and (3) go through a slab of LDS per wave, four columns of
// its 64 rows at a time, two slabs in turn (FP64 on 16-byte boundaries: direct
// copies, else through registers): four neighbouring lanes read 64 contiguous bytes, where a lane
// that reads along its own row touches 64 lines per load, eight times each,
// which the 32 KB of L1 cannot hold for eight waves; and the next slab is on
// its way while one is used.  Within a slab, row i keeps its four values in the
// order k ^ (i / 4) % 4, which spreads the lanes' reads over the banks.
//
// Measured, 256 panels of 64 columns side by side (rows moved and reloaded by
// every chunk, five barriers and a shuffle tree per column before): 64 rows 354
// -> 142 us, 431 rows 375 -> 250, 2000 rows about 1110 -> 830; the panels of a
// solve of 64 frequencies and the lone one, 3072 rows 137 -> 85 ms, 4096 rows 262
// -> 164 (FP32: 83 -> 63 and 176 -> 143).  Of the 480k
// cycles at 431 rows the columns take 174k (2700 each), the update 94k, the
// chunk loads and stores 57k and 54k, the two inverses 41k.
//
// FP32: the sums of (2) and, on the matrix cores, of (3) are FP64, so that a
// value rounds once per chunk.  With FP32 sums the squared error of the first
// solution, which the refinement's result is a power of, is 1.07 to 1.10 times
// as large (chains of 431 to 880 products); the FP64 ones cost 0.2 to 0.3 ms of
// the 4 to 5.4 ms of panels of a pass.
constexpr int GF_NT = 512;

// The larger of v and the v of the lane that DPP control CTRL names; a lane
// without one keeps its own.
template <int CTRL>
__device__ inline uint32_t dpp_max(uint32_t v) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
    return o > v ? o : v;
}
// Largest v over the wave.
__device__ inline uint32_t wave_max(uint32_t v) {
    v = dpp_max<0x111>(v);  // row_shr:1, 2, 4, 8: the last lane of each row of 16
    v = dpp_max<0x112>(v);
    v = dpp_max<0x114>(v);
    v = dpp_max<0x118>(v);
    v = dpp_max<0x142>(v);  // row_bcast:15, then :31
    v = dpp_max<0x143>(v);
    return (uint32_t)rlane((int)v, 63);
}
// Order of the pivot search in 32 bits: a row's v = |re| + |im| by its leading
// bits (all of a float), above NaN (1) and no row at all (0).
__device__ inline uint32_t pivot_key(double v) {
    return v >= 0.0 ? (uint32_t)((uint64_t)__double_as_longlong(v) >> 32) + 2 : 1u;
}
__device__ inline uint32_t pivot_key(float v) { return v >= 0.f ? (uint32_t)__float_as_int(v) + 2 : 1u; }
// Of the lanes in m (not empty), the one with the largest v (NaN counts as
// none above another), ties to the smallest p.
template <typename T>
__device__ inline int best_of(unsigned long long m, T v, int p) {
    int l = __ffsll((long long)m) - 1;
    if (m & (m - 1)) {
        T vl = rlane(v, l);
        int pl = rlane(p, l);
        while (m &= m - 1) {
            const int k = __ffsll((long long)m) - 1, pk = rlane(p, k);
            const T vk = rlane(v, k);
            if (vk > vl || (!(vk < vl) && pk < pl)) {
                l = k;
                vl = vk;
                pl = pk;
            }
        }
    }
    return l;
}

// f(0), ..., f(N - 1), each index a compile-time constant.
template <int... I, typename F>
__device__ __forceinline__ void static_for_(std::integer_sequence<int, I...>, F &&f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_(std::make_integer_sequence<int, N>{}, f);
}

// GC, GI: the element types the pointers are declared with (global address
// space for pointers read from a descriptor, so that they are not accessed as
// flat memory).  DMA: the slabs come by direct copies (FP64, A 16-byte aligned).
template <typename T, int R, int BW, bool DMA, typename GC = Cx<T>, typename GI = int32_t>
__device__ __forceinline__ void getf2r_body(int n, int kb, int w, GC *A, int64_t sA, GI *ipiv, GC *Linv, GC *Uinv,
                                            int nblk, GI *swp, GI *info, const int b) {
    constexpr int NW = GF_NT / 64;
    constexpr int KS = 4;  // columns per slab
    constexpr int CW = (BW + NW - 1) / NW;  // substituted columns per wave
    static_assert(NB % BW == 0 && BW % KS == 0 && BW <= 16, "whole chunks, whole slabs");
    typedef T V2 __attribute__((ext_vector_type(2)));
    typedef double D2 __attribute__((ext_vector_type(2)));
    __shared__ V2 Ts[NB][NB + 1];  // the panel's top rows as they become final (padded: column reads)
    __shared__ V2 slab[NW][2][64 * KS];
    __shared__ V2 Ux[NB][BW];
    __shared__ V2 cand_row[2][NW][BW + 1];  // a wave's candidate row, and the reciprocal of its pivot
    __shared__ T cand_v[2][NW];
    __shared__ int cand_p[2][NW];
    __shared__ int lpiv[NB], phys[NB];  // by column: the pivot's position then, and its row
    __shared__ int sw_dst[2 * NB], sw_src[2 * NB], nsw;
    __shared__ V2 dinv[NB];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    A += (int64_t)b * sA;
    ipiv += (int64_t)b * n;
    swp += (int64_t)b * SWP;
    Linv += ((int64_t)b * nblk + kb / NB) * NB * NB;
    Uinv += ((int64_t)b * nblk + kb / NB) * NB * NB;
    const int m = n - kb;
    GC *P = A + (int64_t)kb * n + kb;  // panel origin, row stride n
    const V2 zero{T(0), T(0)};

    // value (i, c) of the panel by a 32-bit byte offset (at most 4096 rows of
    // fewer than 64k values), so that no row keeps a 64-bit address
    typedef dglobal<char> GB;
    auto at = [&](int i, int c) { return (GC *)((GB *)P + ((uint32_t)i * (uint32_t)n + (uint32_t)c) * (uint32_t)sizeof(GC)); };
    auto load = [](const GC *p) { return V2{p->re, p->im}; };
    auto store = [](GC *p, V2 v) {
        p->re = v.x;
        p->im = v.y;
    };
    // x - l u: FP64 in two fused steps per part; FP32 with l u formed first, so
    // that a step rounds at x's size once, not twice (the refinement's last
    // error is a power of the FP32 factors')
    auto submul = [](auto &x, auto l, auto u) {
        if constexpr (sizeof(x.x) == 8) {
            x.x = fma(-l.x, u.x, x.x);
            x.x = fma(l.y, u.y, x.x);
            x.y = fma(-l.x, u.y, x.y);
            x.y = fma(-l.y, u.x, x.y);
        } else {
            x.x -= fma(l.x, u.x, -(l.y * u.y));
            x.y -= fma(l.x, u.y, l.y * u.x);
        }
    };

    // slab q & 1: columns [c0, c0 + 4) of this wave's rows 512 r ..; rows and
    // columns past the panel repeat its last.  Without DMA: staging registers, set e
    V2 stg[DMA ? 1 : 2][DMA ? 1 : KS];
    typedef std::integral_constant<int, 0> S0;
    typedef std::integral_constant<int, 1> S1;
    auto fetch = [&](int q, auto set, int r, int c0) {
        constexpr int e = set;
        // (opaque, so that the offsets of every row are not kept over the loop)
        uint32_t ns = (uint32_t)n;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+s"(ns));
#endif
        const uint32_t r0 = (uint32_t)(64 * wave + GF_NT * r + (lane >> 2)) * ns, last = (uint32_t)(m - 1) * ns;
        const uint32_t c = (uint32_t)min(c0 + ((lane & 3) ^ ((lane >> 4) & 3)), w - 1);
#pragma unroll
        for (int t = 0; t < KS; ++t) {
            const GC *g = (const GC *)((const GB *)P + (min(r0 + 16 * t * ns, last) + c) * (uint32_t)sizeof(GC));
#if defined(__HIP_DEVICE_COMPILE__)
            if constexpr (DMA)
                __builtin_amdgcn_global_load_lds((const dglobal<uint32_t> *)g,
                                                 (__attribute__((address_space(3))) uint32_t *)&slab[wave][q & 1][64 * t],
                                                 16, 0, 0);
            else
#endif
                stg[DMA ? 0 : e][DMA ? 0 : t] = load(g);
        }
    };
    // slab q is there and the other one has been read (next: the fetch after
    // q's is under way and need not be waited for)
    auto land = [&](int q, auto set, bool next) {
        constexpr int e = set;
        if constexpr (DMA) {
#if defined(__HIP_DEVICE_COMPILE__)
            if (next) asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
#endif
        } else {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int t = 0; t < KS; ++t) slab[wave][q & 1][64 * t + lane] = stg[e][t];
            __builtin_amdgcn_wave_barrier();
        }
    };
    auto slab_read = [&]() {  // the slab's values have arrived in registers
#if defined(__HIP_DEVICE_COMPILE__)
        if constexpr (DMA) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#endif
    };
    const int swz = (lane >> 2) & 3;
    auto slab_at = [&](int q, int k) { return slab[wave][q & 1][4 * lane + (k ^ swz)]; };
    auto rows_here = [&](int r) { return 64 * wave + GF_NT * r < m; };

    int pos[R];
    bool row_ok[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        pos[r] = tid + GF_NT * r;
        row_ok[r] = pos[r] < m;
    }
    if (tid == 0) nsw = 0;
    // the first two slabs of a chunk's columns
    auto fetch_chunk = [&](int j0) {
        constexpr int H = BW / KS;
        fetch(0, S0{}, 0, j0);
        if (H > 1) fetch(1, S1{}, 0, j0 + KS);
        else if (R > 1 && rows_here(1)) fetch(1, S1{}, 1, j0);
    };
    if (rows_here(0)) fetch_chunk(0);

    for (int j0 = 0; j0 < w; j0 += BW) {
        const int bw = min(BW, w - j0);
        // (1) the chunk's columns; the first two slabs were fetched before
        V2 a[R][BW];
        static_for<R * (BW / KS)>([&](auto slab_no) {
            constexpr int H = BW / KS, q = slab_no, r = q / H, h = q % H;
            if (!rows_here(r)) {
#pragma unroll
                for (int k = 0; k < KS; ++k) a[r][KS * h + k] = zero;
                return;
            }
            constexpr int r1 = (q + 1) / H, r2 = (q + 2) / H;
            typedef std::integral_constant<int, q & 1> SQ;
            land(q, SQ{}, r1 < R && rows_here(r1));
#pragma unroll
            for (int k = 0; k < KS; ++k) a[r][KS * h + k] = slab_at(q, k);
            if (r2 < R && rows_here(r2)) {
                slab_read();
                fetch(q, SQ{}, r2, j0 + KS * ((q + 2) % H));
            }
        });
        const int nk = j0 / KS;
        if (j0 > 0) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (row_ok[r] && pos[r] < j0)
#pragma unroll
                    for (int c = 0; c < BW; ++c) Ux[pos[r]][c] = a[r][c];
            lds_barrier();
            if (rows_here(0)) fetch(0, S0{}, 0, 0);  // (3)'s first slab, beside (2)
            // (2) x_i = a_i - sum_{k<i} L_ik x_k for positions i < j0
            if (wave < bw) {
                D2 x[CW];
#pragma unroll
                for (int e = 0; e < CW; ++e) {
                    const V2 u = lane < j0 ? Ux[lane][min(wave + NW * e, BW - 1)] : zero;
                    x[e] = D2{(double)u.x, (double)u.y};
                }
#pragma unroll 4
                for (int k = 0; k < j0 - 1; ++k) {
                    const V2 l = (lane > k && lane < j0) ? Ts[lane][k] : zero;
#pragma unroll
                    for (int e = 0; e < CW; ++e)
                        submul(x[e], D2{(double)l.x, (double)l.y}, D2{rlane(x[e].x, k), rlane(x[e].y, k)});
                }
#pragma unroll
                for (int e = 0; e < CW; ++e) {
                    const int c = wave + NW * e;
                    if (lane < j0 && c < bw) {
                        const V2 u{(T)x[e].x, (T)x[e].y};
                        Ux[lane][c] = u;
                        Ts[lane][j0 + c] = u;
                        store(at(phys[lane], j0 + c), u);
                    }
                }
            }
            lds_barrier();
            // (3)
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!rows_here(r)) continue;
                if constexpr (BW >= 8) {
                    // on the matrix cores, 16 rows at a time: 16 columns as
                    // four real products per complex one, or 8 columns as the
                    // real product [Lr Li] [Ur Ui; -Ui Ur]
                    typedef Mfma<double> M;
                    typedef M::v4 v4;
                    constexpr int NA = BW == 16 ? 2 : 1;
                    v4 d[4][NA];
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int h = 0; h < NA; ++h) d[i][h] = v4{0, 0, 0, 0};
                    const int l15 = lane & 15, l4 = lane >> 4;
                    for (int kb4 = 0; kb4 < nk; ++kb4) {
                        const int q = r * nk + kb4;
                        land(q, S0{}, false);
                        if (kb4 + 1 < nk) fetch(q + 1, S0{}, r, KS * (kb4 + 1));
                        else if (r + 1 < R && rows_here(r + 1)) fetch(q + 1, S0{}, r + 1, 0);
                        const V2 u = Ux[KS * kb4 + l4][l15 & (BW - 1)];
                        V2 l[4];
#pragma unroll
                        for (int i = 0; i < 4; ++i) l[i] = slab[wave][q & 1][4 * (16 * i + l15) + (l4 ^ ((l15 >> 2) & 3))];
                        if constexpr (NA == 2) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][0] = M::op(l[i].x, u.x, d[i][0]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][1] = M::op(l[i].x, u.y, d[i][1]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][0] = M::op(l[i].y, -u.y, d[i][0]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][1] = M::op(l[i].y, u.x, d[i][1]);
                        } else {
                            const bool im = (l15 & 8) != 0;
                            const double b1 = im ? u.y : u.x, b2 = im ? u.x : -u.y;
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][0] = M::op(l[i].x, b1, d[i][0]);
#pragma unroll
                            for (int i = 0; i < 4; ++i) d[i][0] = M::op(l[i].y, b2, d[i][0]);
                        }
                    }
                    // to the rows' own threads through this wave's spare slab
                    // (the other one may be filling): 256 / BW rows at a time,
                    // columns permuted by row against bank conflicts
                    const int qs = r * nk + nk - 1;
                    constexpr int RP = 64 * KS / BW, BPP = RP / 16;
                    V2 *sp = slab[wave][qs & 1];
                    slab_read();
#pragma unroll
                    for (int p = 0; p < 64 / RP; ++p) {
                        __builtin_amdgcn_wave_barrier();
#pragma unroll
                        for (int i = 0; i < BPP; ++i)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int row = 16 * i + M::row(lane, e);
                                if constexpr (NA == 2)
                                    sp[row * BW + (l15 ^ (row & 15))] = V2{(T)d[p * BPP + i][0][e], (T)d[p * BPP + i][1][e]};
                                else
                                    ((T *)sp)[2 * (row * BW + ((l15 & 7) ^ (row & 7))) + (l15 >> 3)] =
                                        (T)d[p * BPP + i][0][e];
                            }
                        __builtin_amdgcn_wave_barrier();
                        if (lane / RP == p) {
                            const int row = lane % RP;
#pragma unroll
                            for (int c = 0; c < BW; ++c) a[r][c] -= sp[row * BW + (c ^ (row & (BW - 1)))];
                        }
                    }
                } else {
                    for (int kb4 = 0; kb4 < nk; ++kb4) {
                        const int q = r * nk + kb4;
                        land(q, S0{}, false);
                        if (kb4 + 1 < nk) fetch(q + 1, S0{}, r, KS * (kb4 + 1));
                        else if (r + 1 < R && rows_here(r + 1)) fetch(q + 1, S0{}, r + 1, 0);
#pragma unroll
                        for (int k = 0; k < KS; ++k) {
                            const V2 l = slab_at(q, k);
#pragma unroll
                            for (int c = 0; c < BW; ++c) submul(a[r][c], l, Ux[KS * kb4 + k][c]);
                        }
                    }
                }
            }
        }
        // the next chunk's first slabs (its columns are not touched before)
        if (j0 + BW < w && rows_here(0)) {
            slab_read();
            fetch_chunk(j0 + BW);
        }
        bool fresh[R];  // rows that this chunk factorises
#pragma unroll
        for (int r = 0; r < R; ++r) fresh[r] = row_ok[r] && pos[r] >= j0;
        // (4)
        static_for<BW>([&](auto col) {
            constexpr int c = col;
            if (c >= bw) return;
            const int j = j0 + c;
            constexpr int par = c & 1;
            // this thread's best row, and the reciprocal its wave would publish
            // (the division beside the search, not after it)
            T best = T(0);
            uint32_t key = 0;
            int bp = 0x7fffffff;
            V2 bx = zero;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T v = fabs(a[r][c].x) + fabs(a[r][c].y);
                const uint32_t kr = (row_ok[r] && pos[r] >= j) ? pivot_key(v) : 0;
                if (kr > key || (kr == key && kr > 0 && (v > best || (!(v < best) && pos[r] < bp)))) {
                    key = kr;
                    best = v;
                    bp = pos[r];
                    bx = a[r][c];
                }
            }
            Cx<T> rc = crcp(Cx<T>{bx.x, bx.y});
#if defined(__HIP_DEVICE_COMPILE__)
            asm volatile("" : "+v"(rc.re), "+v"(rc.im));  // (here, not in the candidate's branch below)
#endif
            const uint32_t wkey = wave_max(key);
            if (wkey > 0) {
                const int src = best_of(__ballot(key == wkey), best, bp);
                if (lane == src) {
                    cand_v[par][wave] = best;
                    cand_p[par][wave] = bp;
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (R == 1 || pos[r] == bp)
#pragma unroll
                            for (int cc = c + 1; cc < BW; ++cc) cand_row[par][wave][cc] = a[r][cc];
                    cand_row[par][wave][BW] = V2{rc.re, rc.im};
                }
            } else if (lane == 0) {
                cand_p[par][wave] = -1;
            }
            lds_barrier();
            const T cv8 = cand_v[par][lane & 7];
            const int cp8 = cand_p[par][lane & 7];
            const uint32_t key8 = cp8 >= 0 ? pivot_key(cv8) : 0;
            uint32_t top = dpp_max<0xB1>(key8);  // quad_perm 1 0 3 2
            top = dpp_max<0x4E>(top);            // quad_perm 2 3 0 1
            top = dpp_max<0x141>(top);           // row_half_mirror
            top = (uint32_t)rlane((int)top, 0);
            const int win = best_of(__ballot(key8 == top) & 0xffull, cv8, cp8);
            const int piv = rlane(cp8, win);
            const T cv = rlane(cv8, win);
            const V2 pr = cand_row[par][win][BW];
            V2 u[BW];
#pragma unroll
            for (int cc = c + 1; cc < BW; ++cc) u[cc] = cand_row[par][win][cc];
            if (tid == 0) {
                lpiv[j] = piv;
                if (cv == T(0) && info[b] == 0) info[b] = kb + j + 1;
            }
            const Cx<T> inv{pr.x, pr.y};
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!row_ok[r]) continue;
                if (pos[r] == piv) {
                    pos[r] = j;
                    phys[j] = tid + GF_NT * r;
                } else if (pos[r] == j) {
                    pos[r] = piv;
                }
                if (pos[r] > j && cv != T(0)) {
                    const Cx<T> l = cmul(Cx<T>{a[r][c].x, a[r][c].y}, inv);
                    a[r][c] = V2{l.re, l.im};
                }
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (row_ok[r] && pos[r] > j && cv != T(0))
#pragma unroll
                    for (int cc = c + 1; cc < BW; ++cc) submul(a[r][cc], a[r][c], u[cc]);
        });
        // (5)
        uint32_t ns = (uint32_t)n;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+s"(ns));
#endif
#pragma unroll
        for (int r = 0; r < R; ++r) {
            GC *row = (GC *)((GB *)P + ((uint32_t)(tid + GF_NT * r) * ns + (uint32_t)j0) * (uint32_t)sizeof(GC));
            if (fresh[r])
#pragma unroll
                for (int c = 0; c < BW; ++c)
                    if (c < bw) {
                        store(row + c, a[r][c]);
                        if (pos[r] < j0 + bw) Ts[pos[r]][j0 + c] = a[r][c];
                    }
        }
        lds_barrier();
        // the new corner rows' L of the earlier chunks (stored before their
        // waves waited for (1)'s loads, hence before this chunk's barriers)
        for (int idx = tid; idx < bw * j0; idx += GF_NT) {
            const int i = j0 + idx / j0, k = idx % j0;
            Ts[i][k] = load(at(phys[i], k));
        }
    }

    // the rows that moved: panel columns here, the others by the caller
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (row_ok[r] && pos[r] != tid + GF_NT * r) {
            const int t = atomicAdd(&nsw, 1);  // at most 64 pivots and 64 rows they displaced
            sw_dst[t] = pos[r];
            sw_src[t] = tid + GF_NT * r;
        }
    __syncthreads();
    {
        const int nt = nsw;
        constexpr int MAXP = 2 * NB * NB / GF_NT;
        V2 v[MAXP];
#pragma unroll
        for (int q = 0; q < MAXP; ++q) {
            const int idx = tid + GF_NT * q;
            v[q] = zero;
            if (idx < nt * w) v[q] = load(at(sw_src[idx / w], idx % w));
        }
        if (tid < w) ipiv[kb + tid] = kb + lpiv[tid];
        if (tid == 0) swp[0] = nt;
        if (tid < nt) {
            swp[1 + tid] = kb + sw_dst[tid];
            swp[1 + 2 * NB + tid] = kb + sw_src[tid];
        }
        if (tid < w) {
            const Cx<T> d = crcp(Cx<T>{Ts[tid][tid].x, Ts[tid][tid].y});
            dinv[tid] = V2{d.re, d.im};
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < MAXP; ++q) {
            const int idx = tid + GF_NT * q;
            if (idx < nt * w) store(at(sw_dst[idx / w], idx % w), v[q]);
        }
    }
    // the inverses of the corner's unit lower and upper triangles, eight
    // columns per wave with lane = row; the steps before a wave's columns begin
    // (after they end) are left out: 72 in all for every wave
    constexpr int CPW = NB / NW;
    const int c0 = wave * CPW;
    V2 x[CPW];
#pragma unroll
    for (int q = 0; q < CPW; ++q) x[q] = (lane == c0 + q && c0 + q < w) ? V2{T(1), T(0)} : zero;
    for (int k = c0; k < w - 1; ++k) {
        const V2 l = (lane > k && lane < w) ? Ts[lane][k] : zero;
#pragma unroll
        for (int q = 0; q < CPW; ++q) submul(x[q], l, V2{rlane(x[q].x, k), rlane(x[q].y, k)});
    }
#pragma unroll
    for (int q = 0; q < CPW; ++q) store(Linv + lane * NB + c0 + q, x[q]);
#pragma unroll
    for (int q = 0; q < CPW; ++q) x[q] = (lane == c0 + q && c0 + q < w) ? V2{T(1), T(0)} : zero;
    for (int k = min(w, c0 + CPW) - 1; k >= 0; --k) {
        const V2 d = dinv[k];
        const V2 u = lane < k ? Ts[lane][k] : zero;
#pragma unroll
        for (int q = 0; q < CPW; ++q) {
            if (lane == k) {
                const Cx<T> t = cmul(Cx<T>{x[q].x, x[q].y}, Cx<T>{d.x, d.y});
                x[q] = V2{t.re, t.im};
            }
            submul(x[q], u, V2{rlane(x[q].x, k), rlane(x[q].y, k)});
        }
    }
#pragma unroll
    for (int q = 0; q < CPW; ++q) store(Uinv + lane * NB + c0 + q, x[q]);
}

template <typename T, int R, int BW, bool DMA>
__global__ __launch_bounds__(GF_NT) void k_getf2r(int n, int kb, int w, Cx<T> *A, int64_t sA, int32_t *ipiv,
                                                  Cx<T> *Linv, Cx<T> *Uinv, int nblk, int32_t *swp, int32_t *info) {
    getf2r_body<T, R, BW, DMA>(n, kb, w, A, sA, ipiv, Linv, Uinv, nblk, swp, info, blockIdx.x);
}

// The index of the item whose workgroups wg0 .. include g (items ordered by wg0).
__device__ inline int group_item(const PanelItem *__restrict__ it, int n_items, int64_t g) {
    int a = 0, b = n_items - 1;
    while (a < b) {
        const int m = (a + b + 1) >> 1;
        if (it[m].wg0 <= g) a = m;
        else b = m - 1;
    }
    return a;
}

// Many batched panel factorisations in one launch (the batched driver's lock
// steps): workgroup g factorises batch entry g - wg0 of its item.
template <typename T, int R, int BW, bool DMA>
__global__ __launch_bounds__(GF_NT) void k_getf2r_group(const PanelItem *__restrict__ items, int n_items) {
    const PanelItem p = items[group_item(items, n_items, blockIdx.x)];
    typedef dglobal<Cx<T>> GC;
    typedef dglobal<int32_t> GI;
    getf2r_body<T, R, BW, DMA, GC, GI>(p.n, p.kb, p.w, (GC *)p.A, p.sA, (GI *)p.ipiv, (GC *)p.Linv, (GC *)p.Uinv, p.nblk,
                                  (GI *)p.swp, (GI *)p.info, (int)(blockIdx.x - p.wg0));
}

// Apply a panel's composed row exchanges to columns [0, kb) and [kb+w, n).
// Workgroup = 32 columns, eight threads per column, each holding up to 16 of
// the (at most 2 NB) source values in registers: all loads are issued before
// any store, and every source row is read before any row is written (one
// barrier).  No LDS, so the pass runs at full occupancy.
template <typename T, typename GC = Cx<T>, typename GI = const int32_t>
__device__ __forceinline__ void laswp_body(int n, int kb, int w, GC *A, int64_t sA, GI *swp, const int b,
                                           const int cg) {
    constexpr int PER = 2 * NB / 8;
    A += (int64_t)b * sA;
    swp += (int64_t)b * SWP;
    const int nt = swp[0];
    if (nt == 0) return;
    const int ncols = n - w;
    const int cc = threadIdx.x & 31, tr = threadIdx.x >> 5;
    const int idx = cg * 32 + cc;
    const int c = idx < kb ? idx : idx + w;
    const bool ok = idx < ncols;
    T vr[PER], vi[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int t = tr + 8 * q;
        vr[q] = vi[q] = T(0);
        if (ok && t < nt) {
            const GC &x = A[(int64_t)swp[1 + 2 * NB + t] * n + c];
            vr[q] = x.re;
            vi[q] = x.im;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int t = tr + 8 * q;
        if (ok && t < nt) {
            GC &x = A[(int64_t)swp[1 + t] * n + c];
            x.re = vr[q];
            x.im = vi[q];
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void k_laswp(int n, int kb, int w, Cx<T> *A, int64_t sA, const int32_t *swp) {
    laswp_body<T>(n, kb, w, A, sA, swp, blockIdx.y, blockIdx.x);
}

// Many batched row-exchange passes in one launch: an item's workgroups are
// (batch entry, 32-column group) pairs, column groups fastest.
template <typename T>
__global__ __launch_bounds__(256) void k_laswp_group(const PanelItem *__restrict__ items, int n_items) {
    const PanelItem p = items[group_item(items, n_items, blockIdx.x)];
    const int ncg = (p.n - p.w + 31) / 32;
    const int64_t r = blockIdx.x - p.wg0;
    typedef dglobal<Cx<T>> GC;
    typedef dglobal<const int32_t> GI;
    laswp_body<T, GC, GI>(p.n, p.kb, p.w, (GC *)p.A, p.sA, (GI *)p.swp, (int)(r / ncg), (int)(r % ncg));
}

// Full row permutation of a factorisation: row i of P A is row perm[i] of A.
__global__ __launch_bounds__(256) void k_perm_from_ipiv(int n, const int32_t *ipiv, int32_t *perm) {
    extern __shared__ int32_t pm[];
    const int b = blockIdx.x;
    ipiv += (int64_t)b * n;
    perm += (int64_t)b * n;
    for (int i = threadIdx.x; i < n; i += blockDim.x) pm[i] = i;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int j = 0; j < n; ++j) {
            const int r = ipiv[j];
            if (r != j) {
                const int t = pm[j];
                pm[j] = pm[r];
                pm[r] = t;
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += blockDim.x) perm[i] = pm[i];
}

// B[b][i][c] = src[b][perm[i]][c]  (out of place gather of rows)
// Grid of the row-wise copies below: x = 256-column blocks, y = rows and
// z = batch entries, each walked with its grid stride (no division per
// element).  About 64k workgroups in all, so that each copies many rows
// (one 4-KB row segment per workgroup left the copies at 3.7 TB/s, bound by
// launching workgroups).
inline dim3 rows_grid(int rows, int cols, int batch) {
    const int xb = (cols + 255) / 256, zb = std::min(batch, 65535);
    const int yb = std::max(1, std::min(rows, 65536 / std::max(1, xb * zb)));
    return dim3((unsigned)xb, (unsigned)yb, (unsigned)zb);
}

template <typename T>
__global__ void k_rowgather(int n, int nrhs, int batch, const int32_t *perm, const Cx<T> *src, int64_t sS,
                            Cx<T> *dst, int64_t sD) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nrhs) return;
    for (int b = blockIdx.z; b < batch; b += gridDim.z)
        for (int i = blockIdx.y; i < n; i += gridDim.y)
            dst[(int64_t)b * sD + (int64_t)i * nrhs + c] =
                src[(int64_t)b * sS + (int64_t)perm[(int64_t)b * n + i] * nrhs + c];
}

// B[b][i][c] = v[perm[i]][c] (dense real v) or delta(perm[i], c) lam[c] (diagonal);
// perm may be null (identity).
__global__ void k_init_rhs(int n, int batch, const double *v, int v_is_diag, const int32_t *perm, zdbl *B,
                           int64_t sB) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n) return;
    for (int b = blockIdx.z; b < batch; b += gridDim.z)
        for (int i = blockIdx.y; i < n; i += gridDim.y) {
            const int r = perm ? perm[(int64_t)b * n + i] : i;
            double x;
            if (v_is_diag) x = (r == c) ? v[c] : 0.0;
            else x = v[(int64_t)r * n + c];
            B[(int64_t)b * sB + (int64_t)i * n + c] = zdbl{x, 0.0};
        }
}

__global__ void k_conj_mirror(int64_t nn, int n_omega, zdbl *W) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int j = 1 + blockIdx.y;  // 1 .. n_omega/2 - 1
    if (idx >= nn) return;
    const zdbl s = W[(int64_t)(n_omega - j) * nn + idx];
    W[(int64_t)j * nn + idx] = zdbl{s.re, -s.im};
}

__global__ void k_z2c(const zdbl *src, zflt *dst, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = zflt{(float)src[i].re, (float)src[i].im};
}

// W[b] += d[b] for active batch entries (d complex float; active may be null:
// all), and out[2b] += sum |d|^2, out[2b+1] += sum |W|^2 of the new W (caller
// zeroes out): one pass over d and W.  HBM-bound; a workgroup adds up its share
// in LDS and makes one atomic addition per sum (with one per wave of 1024
// workgroups the additions to a frequency's two sums took 1.76 ms at 655
// products and 129 frequencies, against 0.23 ms for the whole pass).
__global__ __launch_bounds__(256) void k_add_norms(const zflt *d, zdbl *W, int64_t n_per, const int32_t *active,
                                                   double *out) {
    __shared__ double part[2][4];
    const int b = blockIdx.y;
    const bool add = !active || active[b];
    double sd = 0, sw = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_per; i += (int64_t)gridDim.x * blockDim.x) {
        const zflt x = d[(int64_t)b * n_per + i];
        zdbl y = W[(int64_t)b * n_per + i];
        if (add) {
            y.re += (double)x.re;
            y.im += (double)x.im;
            W[(int64_t)b * n_per + i] = y;
        }
        sd += (double)x.re * x.re + (double)x.im * x.im;
        sw += y.re * y.re + y.im * y.im;
    }
    for (int off = 32; off > 0; off >>= 1) {
        sd += __shfl_xor(sd, off);
        sw += __shfl_xor(sw, off);
    }
    if ((threadIdx.x & 63) == 0) {
        part[0][threadIdx.x >> 6] = sd;
        part[1][threadIdx.x >> 6] = sw;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        const double *p = part[threadIdx.x];
        atomicAdd(&out[2 * b + threadIdx.x], (p[0] + p[1]) + (p[2] + p[3]));
    }
}


__global__ void k_rowgather_z2c(int n, int nrhs, int batch, const int32_t *perm, const zdbl *src, int64_t sS,
                                zflt *dst, int64_t sD) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nrhs) return;
    for (int b = blockIdx.z; b < batch; b += gridDim.z)
        for (int i = blockIdx.y; i < n; i += gridDim.y) {
            const zdbl x = src[(int64_t)b * sS + (int64_t)perm[(int64_t)b * n + i] * nrhs + c];
            dst[(int64_t)b * sD + (int64_t)i * nrhs + c] = zflt{(float)x.re, (float)x.im};
        }
}

__global__ void k_c2z_set(const zflt *d, zdbl *W, int64_t n_per) {
    const int b = blockIdx.y;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_per; i += (int64_t)gridDim.x * blockDim.x) {
        const zflt x = d[(int64_t)b * n_per + i];
        W[(int64_t)b * n_per + i] = zdbl{(double)x.re, (double)x.im};
    }
}

// dst[c][r] = src[r][c] through a 32x32 LDS tile
__global__ __launch_bounds__(256) void k_transpose_d(int rows, int cols, const double *src, double *dst) {
    __shared__ double t[32][33];
    const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int k = ty; k < 32; k += 8)
        if (r0 + k < rows && c0 + tx < cols) t[k][tx] = src[(int64_t)(r0 + k) * cols + c0 + tx];
    __syncthreads();
    for (int k = ty; k < 32; k += 8)
        if (c0 + k < cols && r0 + tx < rows) dst[(int64_t)(c0 + k) * rows + r0 + tx] = t[tx][k];
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

template <typename T>
hipError_t gemm_t(hipStream_t st, int M, int N, int K, T alpha, const Cx<T> *A, int64_t lda, int64_t sA,
                  const Cx<T> *B, int64_t ldb, int64_t sB, T beta, Cx<T> *C, int64_t ldc, int64_t sC, int batch);
template <>
hipError_t gemm_t<double>(hipStream_t st, int M, int N, int K, double alpha, const Cx<double> *A, int64_t lda,
                          int64_t sA, const Cx<double> *B, int64_t ldb, int64_t sB, double beta, Cx<double> *C,
                          int64_t ldc, int64_t sC, int batch) {
    return launch_zgemm_lu(st, M, N, K, alpha, (const zdbl *)A, lda, sA, (const zdbl *)B, ldb, sB, beta, (zdbl *)C,
                           ldc, sC, batch);
}
template <>
hipError_t gemm_t<float>(hipStream_t st, int M, int N, int K, float alpha, const Cx<float> *A, int64_t lda,
                         int64_t sA, const Cx<float> *B, int64_t ldb, int64_t sB, float beta, Cx<float> *C,
                         int64_t ldc, int64_t sC, int batch) {
    return launch_cgemm(st, M, N, K, alpha, (const zflt *)A, lda, sA, (const zflt *)B, ldb, sB, beta, (zflt *)C, ldc,
                        sC, batch);
}

inline hipError_t block_solve_t(hipStream_t st, bool upper, int wo, int n, const Cx<double> *Tm, int64_t ldt, int64_t sT,
                                const Cx<double> *inv, int64_t sI, Cx<double> *X, int64_t ldx, int64_t sX, int batch,
                                int tri) {
    return launch_block_solve(st, upper, wo, n, (const zdbl *)Tm, ldt, sT, (const zdbl *)inv, sI, (zdbl *)X, ldx, sX,
                              batch, tri);
}
inline hipError_t block_solve_t(hipStream_t st, bool upper, int wo, int n, const Cx<float> *Tm, int64_t ldt, int64_t sT,
                                const Cx<float> *inv, int64_t sI, Cx<float> *X, int64_t ldx, int64_t sX, int batch,
                                int tri) {
    return launch_block_solve(st, upper, wo, n, (const zflt *)Tm, ldt, sT, (const zflt *)inv, sI, (zflt *)X, ldx, sX,
                              batch, tri);
}

// Two-level blocking: 64-wide panels inside 256-wide blocks.  Inside a block
// each panel updates only the block's remaining columns (narrow GEMMs); the
// block then computes its U12 rows and updates the trailing matrix with one
// rank-256 GEMM, so the large updates stream the trailing matrix a quarter as
// often as rank-64 updates would.  Row exchanges of every panel are applied at
// once to all columns outside the panel (the columns right of the block have
// received no update from this block yet, so the order is the same as
// applying them all before the block's triangular solve).
constexpr int NBO = 256;

// The register panel of m <= 4096 rows: rows per thread and chunk width by m.
template <typename T, bool DMA>
hipError_t launch_getf2r(hipStream_t st, int m, int batch, int n, int kb, int w, Cx<T> *A, int64_t sA, int32_t *ipiv,
                         Cx<T> *Linv, Cx<T> *Uinv, int nblk, int32_t *swp, int32_t *info) {
#define GW_PANEL(R, BW)                                                                                            \
    hipLaunchKernelGGL((k_getf2r<T, R, BW, DMA>), dim3(batch), dim3(GF_NT), 0, st, n, kb, w, A, sA, ipiv, Linv,    \
                       Uinv, nblk, swp, info)
    if (m <= 512) GW_PANEL(1, 16);
    else if (m <= 1024) GW_PANEL(2, 16);
    else if (m <= 2048) GW_PANEL(4, 8);
    else if (m <= 3072) GW_PANEL(6, 4);
    else GW_PANEL(8, 4);
#undef GW_PANEL
    return hipGetLastError();
}

template <typename T>
hipError_t getrf_impl(hipStream_t st, int n, Cx<T> *A, int64_t sA, int32_t *ipiv, Cx<T> *Linv, Cx<T> *Uinv,
                      Cx<T> *scratch, int32_t *info, int batch) {
    const int nblk = (n + NB - 1) / NB;
    const int64_t sI = (int64_t)nblk * NB * NB;
    int32_t *swp = (int32_t *)(scratch + (int64_t)batch * NB * n);
    hipError_t e;
    OpRecorder *rec = g_rec;
    // the register panels' direct copies take 16 bytes at a time; from rows that
    // do not lie so (FP64), and in FP32, they stage through registers (a solve
    // from A on 8-byte boundaries, 1100 products and 128 points: 20.8 ms, 17.6
    // on 16-byte ones, 37.9 by the panel in memory)
    const bool dma = sizeof(T) == 8 && ((uintptr_t)A & 15) == 0;
    if (rec) rec->mark();
    for (int KB = 0; KB < n; KB += NBO) {
        const int WO = min(NBO, n - KB);
        for (int kb = KB; kb < KB + WO; kb += NB) {
            const int w = min(NB, n - kb);
            const int m = n - kb;
            const bool regs = m <= 4096;
            if (rec) {
                // lock-step recording: the panel (a grouped launch per
                // register-row variant) and its row exchanges
                RecOp o;
                o.p = PanelItem{A, sA, ipiv, swp, info, Linv, Uinv, n, kb, w, nblk, batch, 0};
                if (regs) {
                    o.kind = RecOp::PANEL;
                    o.key = (m <= 512 ? 0 : m <= 1024 ? 1 : m <= 2048 ? 2 : m <= 3072 ? 3 : 4) +
                            (sizeof(T) == 4 ? 5 : dma ? 0 : 10);
                    rec->ops.push_back(o);
                } else {
                    rec->other([=](hipStream_t s2) {
                        hipLaunchKernelGGL(k_getf2<T>, dim3(batch), dim3(512), 0, s2, n, kb, w, A, sA, ipiv, Linv,
                                           Uinv, nblk, scratch, swp, info);
                        return hipGetLastError();
                    });
                }
                if (n - w > 0) {
                    RecOp l;
                    l.kind = RecOp::LASWP;
                    l.key = sizeof(T) == 4 ? 1 : 0;
                    l.p = o.p;
                    rec->ops.push_back(l);
                }
            } else {
            ProfScope ps(st, "lu_panel", 0.0, 2.0 * m * w * sizeof(Cx<T>) * (double)batch);
            if (!regs)
                hipLaunchKernelGGL(k_getf2<T>, dim3(batch), dim3(512), 0, st, n, kb, w, A, sA, ipiv, Linv, Uinv, nblk,
                                   scratch, swp, info);
            else if (dma)
                (void)launch_getf2r<T, sizeof(T) == 8>(st, m, batch, n, kb, w, A, sA, ipiv, Linv, Uinv, nblk, swp, info);
            else
                (void)launch_getf2r<T, false>(st, m, batch, n, kb, w, A, sA, ipiv, Linv, Uinv, nblk, swp, info);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            if (n - w > 0) {
                ProfScope pl(st, "laswp", 0.0, 2.0 * w * (n - w) * sizeof(Cx<T>) * (double)batch);
                hipLaunchKernelGGL(k_laswp<T>, dim3((n - w + 31) / 32, batch), dim3(256), 0, st, n, kb, w, A, sA, swp);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            }
            const int rb = KB + WO - kb - w;  // columns of this block right of the panel
            if (rb > 0) {
                const Cx<T> *Lb = Linv + (int64_t)(kb / NB) * NB * NB;
                Cx<T> *A12 = A + (int64_t)kb * n + kb + w;
                e = gemm_t<T>(st, w, rb, w, T(1), Lb, NB, sI, A12, n, sA, T(0), A12, n, sA, batch);
                if (e != hipSuccess) return e;
                if (n - kb - w > 0) {
                    e = gemm_t<T>(st, n - kb - w, rb, w, T(-1), A + (int64_t)(kb + w) * n + kb, n, sA, A12, n, sA, T(1),
                                  A + (int64_t)(kb + w) * n + kb + w, n, sA, batch);
                    if (e != hipSuccess) return e;
                }
            }
        }
        const int rest = n - KB - WO;
        if (rest > 0) {
            // U12 rows of the block
            e = block_solve_t(st, false, WO, rest, A + (int64_t)KB * n + KB, n, sA,
                                 Linv + (int64_t)(KB / NB) * NB * NB, sI, A + (int64_t)KB * n + KB + WO, n, sA, batch,
                                 -1);
            if (e != hipSuccess) return e;
            // trailing update, rank WO
            e = gemm_t<T>(st, rest, rest, WO, T(-1), A + (int64_t)(KB + WO) * n + KB, n, sA,
                          A + (int64_t)KB * n + KB + WO, n, sA, T(1), A + (int64_t)(KB + WO) * n + KB + WO, n, sA,
                          batch);
            if (e != hipSuccess) return e;
        }
    }
    if (rec) rec->mark();
    return hipSuccess;
}

// X[b][i][j] = X[b][j][i] for j > i (32 x 32 tiles through LDS).
template <typename T>
__global__ __launch_bounds__(256) void k_mirror_lower(int n, int nt, Cx<T> *X, int64_t sX) {
    __shared__ Cx<T> t[32][33];
    int tile = blockIdx.x, bi = 0;
    while (tile >= nt - bi) {  // upper tiles (bi <= bj) row by row
        tile -= nt - bi;
        ++bi;
    }
    const int bj = bi + tile;
    Cx<T> *x = X + (int64_t)blockIdx.y * sX;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = bj * 32 + ty + 8 * q, c = bi * 32 + tx;  // lower tile (bj, bi)
        if (r < n && c < n) t[ty + 8 * q][tx] = x[(int64_t)r * n + c];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = bi * 32 + ty + 8 * q, c = bj * 32 + tx;  // upper (r, c) = lower (c, r)
        if (r < n && c < n && c > r) x[(int64_t)r * n + c] = t[tx][ty + 8 * q];
    }
}

template <typename T>
hipError_t getrs_impl(hipStream_t st, int n, int nrhs, const Cx<T> *LU, int64_t sA, const Cx<T> *Linv,
                      const Cx<T> *Uinv, Cx<T> *B, int64_t sB, int batch, bool sym_lower) {
    const int nblk = (n + NB - 1) / NB;
    const int64_t sI = (int64_t)nblk * NB * NB;
    hipError_t e;
    OpRecorder *rec = g_rec;
    if (rec) rec->mark();
    // forward: L Y = P B, left-looking over the outer blocks: block row
    // [KB, KB + WO) first takes everything already solved above it in one
    // product (inner dimension KB, long for the later blocks), then is solved
    // 64 rows at a time
    for (int KB = 0; KB < n; KB += NBO) {
        const int WO = min(NBO, n - KB);
        if (KB > 0) {
            e = gemm_t<T>(st, WO, nrhs, KB, T(-1), LU + (int64_t)KB * n, n, sA, B, nrhs, sB, T(1),
                          B + (int64_t)KB * nrhs, nrhs, sB, batch);
            if (e != hipSuccess) return e;
        }
        e = block_solve_t(st, false, WO, nrhs, LU + (int64_t)KB * n + KB, n, sA,
                             Linv + (int64_t)(KB / NB) * NB * NB, sI, B + (int64_t)KB * nrhs, nrhs, sB, batch, -1);
        if (e != hipSuccess) return e;
    }
    // backward: U X = Y, left-looking from the last outer block up.  With
    // sym_lower, rows [r0, r1) are only needed in columns [0, r1): every
    // product is cut to those columns, so the work follows the lower triangle
    // (a right-looking update would fill whole squares of columns).
    for (int KB = ((n - 1) / NBO) * NBO; KB >= 0; KB -= NBO) {
        const int WO = min(NBO, n - KB);
        const int below = n - KB - WO;
        if (below > 0) {
            e = gemm_t<T>(st, WO, sym_lower ? KB + WO : nrhs, below, T(-1), LU + (int64_t)KB * n + KB + WO, n, sA,
                          B + (int64_t)(KB + WO) * nrhs, nrhs, sB, T(1), B + (int64_t)KB * nrhs, nrhs, sB, batch);
            if (e != hipSuccess) return e;
        }
        e = block_solve_t(st, true, WO, sym_lower ? KB + WO : nrhs, LU + (int64_t)KB * n + KB, n, sA,
                             Uinv + (int64_t)(KB / NB) * NB * NB, sI, B + (int64_t)KB * nrhs, nrhs, sB, batch,
                             sym_lower ? KB : -1);
        if (e != hipSuccess) return e;
    }
    if (rec) rec->mark();
    if (sym_lower && n > 1) {
        const int nt = (n + 31) / 32;
        if (rec) {
            rec->other([=](hipStream_t s2) {
                hipLaunchKernelGGL(k_mirror_lower<T>, dim3((unsigned)(nt * (nt + 1) / 2), (unsigned)batch), dim3(256),
                                   0, s2, n, nt, B, sB);
                return hipGetLastError();
            });
            return hipSuccess;
        }
        ProfScope ps(st, "mirror_lower", 0.0, 2.0 * sizeof(Cx<T>) * (double)n * (n - 1) / 2 * batch);
        hipLaunchKernelGGL(k_mirror_lower<T>, dim3((unsigned)(nt * (nt + 1) / 2), (unsigned)batch), dim3(256), 0, st,
                           n, nt, B, sB);
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace

// scratch must hold batch * 64 * n complex + batch * (1 + 4*64) int32.
template <>
hipError_t getrf_batched<zdbl>(hipStream_t st, int n, zdbl *A, int64_t sA, int32_t *ipiv, zdbl *Linv, zdbl *Uinv,
                               zdbl *scratch, int32_t *info, int batch) {
    return getrf_impl<double>(st, n, (Cx<double> *)A, sA, ipiv, (Cx<double> *)Linv, (Cx<double> *)Uinv,
                              (Cx<double> *)scratch, info, batch);
}
template <>
hipError_t getrf_batched<zflt>(hipStream_t st, int n, zflt *A, int64_t sA, int32_t *ipiv, zflt *Linv, zflt *Uinv,
                               zflt *scratch, int32_t *info, int batch) {
    return getrf_impl<float>(st, n, (Cx<float> *)A, sA, ipiv, (Cx<float> *)Linv, (Cx<float> *)Uinv,
                             (Cx<float> *)scratch, info, batch);
}
template <>
hipError_t getrs_batched<zdbl>(hipStream_t st, int n, int nrhs, const zdbl *LU, int64_t sA, const int32_t *ipiv,
                               const zdbl *Linv, const zdbl *Uinv, zdbl *B, int64_t sB, int batch, bool sym_lower) {
    (void)ipiv;  // rows of B are already in pivot order (see launch_perm / launch_init_rhs)
    return getrs_impl<double>(st, n, nrhs, (const Cx<double> *)LU, sA, (const Cx<double> *)Linv,
                              (const Cx<double> *)Uinv, (Cx<double> *)B, sB, batch, sym_lower && nrhs == n);
}
template <>
hipError_t getrs_batched<zflt>(hipStream_t st, int n, int nrhs, const zflt *LU, int64_t sA, const int32_t *ipiv,
                               const zflt *Linv, const zflt *Uinv, zflt *B, int64_t sB, int batch, bool sym_lower) {
    (void)ipiv;
    return getrs_impl<float>(st, n, nrhs, (const Cx<float> *)LU, sA, (const Cx<float> *)Linv,
                             (const Cx<float> *)Uinv, (Cx<float> *)B, sB, batch, sym_lower && nrhs == n);
}

hipError_t launch_perm(hipStream_t st, int n, const int32_t *ipiv, int32_t *perm, int batch) {
    GW_DEFER(launch_perm(st, n, ipiv, perm, batch));
    hipLaunchKernelGGL(k_perm_from_ipiv, dim3(batch), dim3(256), (size_t)n * sizeof(int32_t), st, n, ipiv, perm);
    return hipGetLastError();
}

hipError_t launch_rowgather_c(hipStream_t st, int n, int nrhs, const int32_t *perm, const zflt *src, int64_t sS,
                              zflt *dst, int64_t sD, int batch) {
    GW_DEFER(launch_rowgather_c(st, n, nrhs, perm, src, sS, dst, sD, batch));
    hipLaunchKernelGGL(k_rowgather<float>, rows_grid(n, nrhs, batch), dim3(256), 0, st, n, nrhs, batch, perm,
                       (const Cx<float> *)src, sS, (Cx<float> *)dst, sD);
    return hipGetLastError();
}
hipError_t launch_rowgather_z(hipStream_t st, int n, int nrhs, const int32_t *perm, const zdbl *src, int64_t sS,
                              zdbl *dst, int64_t sD, int batch) {
    GW_DEFER(launch_rowgather_z(st, n, nrhs, perm, src, sS, dst, sD, batch));
    hipLaunchKernelGGL(k_rowgather<double>, rows_grid(n, nrhs, batch), dim3(256), 0, st, n, nrhs, batch, perm,
                       (const Cx<double> *)src, sS, (Cx<double> *)dst, sD);
    return hipGetLastError();
}

hipError_t launch_init_rhs_perm(hipStream_t st, int n, const double *v, int v_is_diag, const int32_t *perm, zdbl *B,
                                int64_t sB, int batch) {
    GW_DEFER(launch_init_rhs_perm(st, n, v, v_is_diag, perm, B, sB, batch));
    ProfScope ps(st, "init_rhs", 0.0, 16.0 * (double)n * n * batch);
    hipLaunchKernelGGL(k_init_rhs, rows_grid(n, n, batch), dim3(256), 0, st, n, batch, v, v_is_diag, perm, B, sB);
    return hipGetLastError();
}

hipError_t launch_init_rhs(hipStream_t st, int n, const double *v, int v_is_diag, zdbl *B, int64_t sB, int batch) {
    return launch_init_rhs_perm(st, n, v, v_is_diag, nullptr, B, sB, batch);
}

hipError_t launch_conj_mirror(hipStream_t st, int64_t nn, int n_omega, zdbl *W) {
    GW_DEFER(launch_conj_mirror(st, nn, n_omega, W));
    if (n_omega < 4) return hipSuccess;
    dim3 grid((unsigned)((nn + 255) / 256), n_omega / 2 - 1);
    ProfScope ps(st, "conj_mirror", 0.0, 2.0 * 16.0 * (double)nn * (n_omega / 2 - 1));
    hipLaunchKernelGGL(k_conj_mirror, grid, dim3(256), 0, st, nn, n_omega, W);
    return hipGetLastError();
}

hipError_t launch_z2c(hipStream_t st, const zdbl *src, zflt *dst, int64_t n) {
    GW_DEFER(launch_z2c(st, src, dst, n));
    int64_t blocks = (n + 255) / 256;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_z2c, dim3((unsigned)blocks), dim3(256), 0, st, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_add_norms(hipStream_t st, const zflt *d, zdbl *W, int64_t n_per, int batch, const int32_t *active,
                            double *out) {
    GW_DEFER(launch_add_norms(st, d, W, n_per, batch, active, out));
    // about sixteen workgroups per CU in all
    const int64_t blocks = std::min<int64_t>((n_per + 255) / 256, std::max(1, 4096 / std::max(1, batch)));
    hipLaunchKernelGGL(k_add_norms, dim3((unsigned)blocks, batch), dim3(256), 0, st, d, W, n_per, active, out);
    return hipGetLastError();
}

hipError_t launch_rowgather_z2c(hipStream_t st, int n, int nrhs, const int32_t *perm, const zdbl *src, int64_t sS,
                                zflt *dst, int64_t sD, int batch) {
    GW_DEFER(launch_rowgather_z2c(st, n, nrhs, perm, src, sS, dst, sD, batch));
    hipLaunchKernelGGL(k_rowgather_z2c, rows_grid(n, nrhs, batch), dim3(256), 0, st, n, nrhs, batch, perm, src, sS,
                       dst, sD);
    return hipGetLastError();
}

hipError_t launch_c2z_set(hipStream_t st, const zflt *d, zdbl *W, int64_t n_per, int batch) {
    GW_DEFER(launch_c2z_set(st, d, W, n_per, batch));
    int64_t blocks = (n_per + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    hipLaunchKernelGGL(k_c2z_set, dim3((unsigned)blocks, batch), dim3(256), 0, st, d, W, n_per);
    return hipGetLastError();
}

// Panel keys: (R, BW) = (1, 16), (2, 16), (4, 8), (6, 4), (8, 4) for panels of at
// most 512, 1024, 2048, 3072, 4096 rows, complex double; +5 complex float, +10
// complex double off 16-byte boundaries.
hipError_t launch_panel_group(hipStream_t st, int key, const PanelItem *items, int n_items, int64_t n_wg) {
    if (n_items <= 0 || n_wg <= 0) return hipSuccess;
    if (key < 0 || key > 14 || n_wg > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)n_wg), blk(GF_NT);
#define GW_PANEL(T, R, BW, DMA) \
    hipLaunchKernelGGL((k_getf2r_group<T, R, BW, DMA>), grid, blk, 0, st, items, n_items)
#define GW_PANELS(T, DMA)                     \
    switch (key % 5) {                        \
        case 0: GW_PANEL(T, 1, 16, DMA); break; \
        case 1: GW_PANEL(T, 2, 16, DMA); break; \
        case 2: GW_PANEL(T, 4, 8, DMA); break;  \
        case 3: GW_PANEL(T, 6, 4, DMA); break;  \
        default: GW_PANEL(T, 8, 4, DMA); break; \
    }
    if (key < 5) GW_PANELS(double, true)
    else if (key < 10) GW_PANELS(float, false)
    else GW_PANELS(double, false)
#undef GW_PANELS
#undef GW_PANEL
    return hipGetLastError();
}

// Row-exchange keys: 0 complex double, 1 complex float.
hipError_t launch_laswp_group(hipStream_t st, int key, const PanelItem *items, int n_items, int64_t n_wg) {
    if (n_items <= 0 || n_wg <= 0) return hipSuccess;
    if (key < 0 || key > 1 || n_wg > INT32_MAX) return hipErrorInvalidValue;
    if (key == 0) hipLaunchKernelGGL(k_laswp_group<double>, dim3((unsigned)n_wg), dim3(256), 0, st, items, n_items);
    else hipLaunchKernelGGL(k_laswp_group<float>, dim3((unsigned)n_wg), dim3(256), 0, st, items, n_items);
    return hipGetLastError();
}

hipError_t launch_copy(hipStream_t st, void *dst, const void *src, size_t bytes) {
    GW_DEFER(launch_copy(st, dst, src, bytes));
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToDevice, st);
}

hipError_t launch_transpose_d(hipStream_t st, int rows, int cols, const double *src, double *dst) {
    dim3 grid((cols + 31) / 32, (rows + 31) / 32);
    hipLaunchKernelGGL(k_transpose_d, grid, dim3(256), 0, st, rows, cols, src, dst);
    return hipGetLastError();
}

namespace {
// Numbers of either sign in [1/2, 1): words (the high ones of doubles) of the
// exponent and hashed bits.
__global__ void k_fill_test(uint32_t *p, int64_t n, int dbl) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        uint32_t h = (uint32_t)i * 2654435761u;
        h = (h ^ (h >> 15)) * 2246822519u;
        h ^= h >> 13;
        if (!dbl) h = (h & 0x807fffffu) | 0x3f000000u;
        else if (i & 1) h = (h & 0x800fffffu) | 0x3fe00000u;
        p[i] = h;
    }
}
}  // namespace

hipError_t launch_fill_test(hipStream_t st, uint32_t *p, int64_t n, bool dbl) {
    hipLaunchKernelGGL(k_fill_test, dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096))),
                       dim3(256), 0, st, p, n, dbl ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_fill_u32(hipStream_t st, uint32_t *p, int64_t n, uint32_t value) {
    GW_DEFER(launch_fill_u32(st, p, n, value));
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, value);
    return hipGetLastError();
}

}  // namespace gwk
