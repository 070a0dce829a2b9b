// HIP kernels for gfx950 (CDNA4, wave64).
//
// The contraction of one term network is a fixed sequence of pairwise
// contractions; each step here is a bit permutation of the operand legs
// (TTGT transpose) followed by a complex GEMM batched over the term
// instances that step serves.  Complex values are interleaved (re, im).

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <type_traits>
#include <cstdint>

#include "kernels.h"

namespace tn {

// Events of the next grouped launch on this thread (set by the executor when
// it times launches): they are recorded by the dispatch itself at the
// kernel's start and end, so the interval is the kernel's execution only.
static thread_local hipEvent_t g_ev_start = nullptr, g_ev_stop = nullptr;

void set_launch_events(hipEvent_t start, hipEvent_t stop) {
    g_ev_start = start;
    g_ev_stop = stop;
}

template <typename... Args, typename F>
static void launch_k(F kernel, dim3 grid, dim3 block, hipStream_t s, Args... args) {
    if (g_ev_start || g_ev_stop) {
        hipEvent_t a = g_ev_start, b = g_ev_stop;
        g_ev_start = g_ev_stop = nullptr;
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, a, b, 0, args...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
    }
}


typedef float v16f __attribute__((ext_vector_type(16)));
typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int64_t pick(int mode, const int32_t* map, int64_t i) {
    return mode == 0 ? i : (mode == 1 ? 0 : (int64_t)map[i]);
}

// ---------------------------------------------------------------------------
// K1: FP32 complex GEMM on MFMA.
//
// The complex product C = A B (m x k times k x n) is the real product
// C_r = A_r B_e of the interleaved real view A_r (m x 2k) with the embedding
// B_e (2k x 2n), B_e[2p+s][2j+t] = [[Re, Im], [-Im, Re]][s][t] of B[p][j]; the
// output comes out interleaved.  Each v_mfma_f32_32x32x2f32 covers one complex
// k index, 32 rows and 16 complex columns: 8 m n k real flops per complex MAC,
// as in the four-real-product form.  Block tile BM x BNC complex, k staged
// through LDS in chunks of 8 (planar re/im for A so that a half-wave reads
// consecutive words).
// ---------------------------------------------------------------------------
template <int BM, int BNC>
__global__ __launch_bounds__(64 * (BM >= 64 ? BM / 64 : 1) * (BNC >= 32 ? BNC / 32 : 1))
void k_gemm_mfma(GemmArgs g) {
    constexpr int WM = BM >= 64 ? BM / 64 : 1;
    constexpr int WN = BNC >= 32 ? BNC / 32 : 1;
    constexpr int NT = 64 * WM * WN;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BNC / WN / 16;
    constexpr int BKC = 8;
    constexpr int AE = (BM * BKC + NT - 1) / NT;     // A elements per thread per chunk
    constexpr int BE = (BKC * BNC + NT - 1) / NT;    // B elements per thread per chunk
    // double-buffered LDS: A planar (re, im) [k][row], B interleaved [k][col];
    // rows padded by one element so that threads staging consecutive k of the
    // same row (or column) land in different banks
    __shared__ float As_re[2][BKC][BM + 1];
    __shared__ float As_im[2][BKC][BM + 1];
    __shared__ float2 Bs[2][BKC][BNC + 1];

    const int m_log = g.m_log, n_log = g.n_log, k_log = g.k_log;
    const int64_t m = int64_t(1) << m_log, n = int64_t(1) << n_log, k = int64_t(1) << k_log;
    // n < BNC happens only for the 16-column tiles: the tile is padded with
    // zero columns that are never stored
    const int tn_log = n_log >= __builtin_ctz(BNC) ? n_log - __builtin_ctz(BNC) : 0;
    const int64_t tiles = (m / BM) << tn_log;
    const int64_t blk = blockIdx.x;
    const int64_t inst = blk / tiles;
    const int64_t tile = blk - inst * tiles;
    const int64_t tm0 = (tile >> tn_log) * BM;
    const int64_t tn0 = (tile & ((int64_t(1) << tn_log) - 1)) * BNC;
    const float2* __restrict__ A = (const float2*)g.A + pick(g.ia_mode, g.ia, inst) * g.strideA;
    const float2* __restrict__ B = (const float2*)g.B + pick(g.ib_mode, g.ib, inst) * g.strideB;
    float* __restrict__ C = (float*)g.C + inst * (2 * m * n);

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM;
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

    const int kc = k < BKC ? (int)k : BKC;
    const int kc_log = k_log < 3 ? k_log : 3;
    const int half = lane >> 5;             // 0: real slice, 1: imaginary slice
    const int sub = lane & 31;
    float2 ra[AE], rb[BE];
    // global -> registers for the chunk starting at k0
    auto load = [&](int64_t k0) {
#pragma unroll
        for (int q = 0; q < AE; ++q) {
            const int e = threadIdx.x + q * NT;
            float2 v = make_float2(0.0f, 0.0f);
            if (e < BM * kc) {
                if (!g.transA) {
                    const int r = e >> kc_log, p = e & (kc - 1);
                    v = A[(tm0 + r) * k + k0 + p];
                } else {
                    const int p = e / BM, r = e % BM;
                    v = A[(k0 + p) * m + tm0 + r];
                }
            }
            ra[q] = v;
        }
#pragma unroll
        for (int q = 0; q < BE; ++q) {
            const int e = threadIdx.x + q * NT;
            float2 v = make_float2(0.0f, 0.0f);
            if (e < kc * BNC) {
                int p, c;
                if (!g.transB) {
                    p = e / BNC;
                    c = e % BNC;
                } else {
                    c = e >> kc_log;
                    p = e & (kc - 1);
                }
                if (tn0 + c < n) v = g.transB ? B[(tn0 + c) * k + k0 + p] : B[(k0 + p) * n + tn0 + c];
            }
            rb[q] = v;
        }
    };
    // registers -> LDS buffer `buf`
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AE; ++q) {
            const int e = threadIdx.x + q * NT;
            if (e < BM * kc) {
                int r, p;
                if (!g.transA) {
                    r = e >> kc_log;
                    p = e & (kc - 1);
                } else {
                    p = e / BM;
                    r = e % BM;
                }
                As_re[buf][p][r] = ra[q].x;
                As_im[buf][p][r] = ra[q].y;
            }
        }
#pragma unroll
        for (int q = 0; q < BE; ++q) {
            const int e = threadIdx.x + q * NT;
            if (e < kc * BNC) {
                int p, c;
                if (!g.transB) {
                    p = e / BNC;
                    c = e % BNC;
                } else {
                    c = e >> kc_log;
                    p = e & (kc - 1);
                }
                Bs[buf][p][c] = rb[q];
            }
        }
    };
    const int64_t nchunks = k / kc;
    load(0);
    stash(0);
    __syncthreads();
    for (int64_t ch = 0; ch < nchunks; ++ch) {
        const int buf = (int)(ch & 1);
        if (ch + 1 < nchunks) load((ch + 1) * kc);     // in flight during the MFMAs below
        for (int p = 0; p < kc; ++p) {
            float a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * (TM * 32) + i * 32 + sub;
                a[i] = half ? As_im[buf][p][row] : As_re[buf][p][row];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = wn * (TN * 16) + j * 16 + (sub >> 1);
                const float2 bv = Bs[buf][p][col];
                const int t = sub & 1;
                b[j] = half == 0 ? (t == 0 ? bv.x : bv.y) : (t == 0 ? -bv.y : bv.x);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (ch + 1 < nchunks) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t colf = 2 * (tn0 + wn * (TN * 16) + j * 16) + sub;
            if (colf >= 2 * n) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = tm0 + wm * (TM * 32) + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                C[row * (2 * n) + colf] = acc[i][j][r];
            }
        }
}

// ---------------------------------------------------------------------------
// K1 with gathered operands: the same MFMA tiling, but A and B are read in
// their stored leg order (no transpose pass).  Offsets of the low row /
// column / inner bits come from small LDS tables; the high parts are added
// once per tile and per k chunk.
// ---------------------------------------------------------------------------
// Device-memory (global address space) views of pointers read from job
// descriptors: generic pointers would compile to flat loads, which count on
// the LDS wait counter as well, so every LDS wait would also wait for the
// global prefetch in flight.
#define TN_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const TN_GLOBAL T* gload(const void* p) {
    return (const TN_GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ TN_GLOBAL T* gstore(void* p) {
    return (TN_GLOBAL T*)p;
}
#define TN_CONST __attribute__((address_space(4)))
// read-only view of memory that no block of the launch writes: uniform
// addresses become scalar loads
template <typename T>
__device__ __forceinline__ const TN_CONST T* cload(const void* p) {
    return (const TN_CONST T*)p;
}

// element loads from global views (HIP's vector types do not copy across
// address spaces): one 8-byte load for complex64, two for complex128
__device__ __forceinline__ float2 gld(const TN_GLOBAL float2* p) {
    const uint64_t u = *(const TN_GLOBAL uint64_t*)p;
    float2 r;
    __builtin_memcpy(&r, &u, 8);
    return r;
}
__device__ __forceinline__ double2 gld(const TN_GLOBAL double2* p) {
    const TN_GLOBAL double* q = (const TN_GLOBAL double*)p;
    return make_double2(q[0], q[1]);
}
__device__ __forceinline__ void gst(TN_GLOBAL float2* p, float2 v) {
    uint64_t u;
    __builtin_memcpy(&u, &v, 8);
    *(TN_GLOBAL uint64_t*)p = u;
}
__device__ __forceinline__ void gst(TN_GLOBAL double2* p, double2 v) {
    TN_GLOBAL double* q = (TN_GLOBAL double*)p;
    q[0] = v.x;
    q[1] = v.y;
}

__device__ __forceinline__ int64_t deposit(int64_t x, const int8_t* pos, int lo, int hi) {
    // the positions are the same for every lane (a job record's legs): read
    // as eight words into scalar registers, then applied without per-lane
    // branches in a loop that stops at hi
    const uint32_t* pw = reinterpret_cast<const uint32_t*>(pos);
    uint32_t w[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) w[q] = __builtin_amdgcn_readfirstlane(pw[q]);
    int64_t o = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        if (j >= hi) break;
        if (j >= lo) o |= (int64_t)((x >> j) & 1) << (int)((w[j >> 2] >> (8 * (j & 3))) & 63u);
    }
    return o;
}

// the same from a record in constant memory
__device__ __forceinline__ int64_t deposit(int64_t x, const TN_CONST int8_t* pos, int lo, int hi) {
    const TN_CONST uint32_t* pw = (const TN_CONST uint32_t*)pos;
    int64_t o = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        if (j >= hi) break;
        if (j >= lo) o |= (int64_t)((x >> j) & 1) << (int)((pw[j >> 2] >> (8 * (j & 3))) & 63u);
    }
    return o;
}

// Offset steps of a chunk counter: with chunk index h (inner index h << lo),
// deposit(h + 1) = deposit(h) + step[ctz(~h)], where step[t] is the offset of
// inner bit lo + t minus the offsets of the bits below it, lo <= bit < lo + t.
// The sums run in scalar registers; thread t writes entry t (t < 32; entries past
// the last bit are 0: the step after the last chunk).  (Placing
// the whole counter anew for each chunk instead cost long tiles 7 %.)
__device__ __forceinline__ void chunk_steps(const TN_CONST int8_t* pos, int lo, int hi, int64_t* step) {
    const TN_CONST uint32_t* pw = (const TN_CONST uint32_t*)pos;
    int64_t below = 0, mine = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
        if (j >= hi) break;
        if (j < lo) continue;
        const int64_t at = int64_t(1) << ((pw[j >> 2] >> (8 * (j & 3))) & 63u);
        if ((int)threadIdx.x == j - lo) mine = at - below;
        below += at;
    }
    if (threadIdx.x < 32) step[threadIdx.x] = mine;
}

// Output offset (element index into C) of row i / column j of a grouped tile,
// -1 for padding: merge 2 stacks `cnt` slices along the rows, merge 1 along
// the columns, merge 0 holds one slice at origin (tm0, tn0).  Shared by the
// tile kernels and the split-sum reduction, so both address the same outputs.
template <typename Job>
__device__ __forceinline__ int64_t tile_out_row(const Job& J, const MfmaTile& T, int i) {
    const int m_log = J.m_log;
    const int64_t m = int64_t(1) << m_log, n = int64_t(1) << J.n_log;
    if (J.merge == 2) {
        const int seg = i >> m_log;
        return seg < T.cnt ? gload<int64_t>(J.oc)[T.s0 + seg] + (i & (m - 1)) * n : -1;
    }
    const int64_t r = T.tm0 + i;
    return r < m ? (J.merge == 1 ? 0 : gload<int64_t>(J.oc)[T.s0]) + r * n : -1;
}
template <typename Job>
__device__ __forceinline__ int64_t tile_out_col(const Job& J, const MfmaTile& T, int j) {
    const int n_log = J.n_log;
    const int64_t n = int64_t(1) << n_log;
    if (J.merge == 1) {
        const int seg = j >> n_log;
        return seg < T.cnt ? gload<int64_t>(J.oc)[T.s0 + seg] + (j & (n - 1)) : -1;
    }
    const int64_t c = T.tn0 + j;
    return c < n ? c : -1;
}

// Offset tables of a grouped tile: A / B element offsets of its rows and columns
// and of the inner indices of a chunk, C offsets of its rows and columns (-1 =
// padding).  One entry per thread where the block has that many; the job record
// is read with scalar loads.  (With the record copied to LDS by one thread and
// the step tables summed entry by entry, a FP64 level of 131072 tiles of k = 16
// took 741 us, now 597; 65536 of k = 32 617 -> 518; the 12 packed circuits 2196
// -> 2092 us.)
template <int BM, int BN, int BK, int NT>
__device__ __forceinline__ void tile_tables(const TN_CONST MfmaJob& J, const MfmaTile& T, int kc_log, int64_t* row_a,
                                            int64_t* row_c, int64_t* col_b, int64_t* col_c, int64_t* ak_lo,
                                            int64_t* bk_lo) {
    const int m_log = J.m_log, n_log = J.n_log;
    const int64_t m = int64_t(1) << m_log, n = int64_t(1) << n_log;
    const int merge = J.merge, kc = 1 << kc_log;
    for (int e = threadIdx.x; e < BM + BN + BK; e += NT) {
        if (e < BM) {
            const int seg = merge == 2 ? e >> m_log : 0;
            const int64_t r = merge == 2 ? e & (m - 1) : T.tm0 + e;
            const bool ok = merge == 2 ? seg < T.cnt : r < m;
            row_a[e] = ok ? gload<int64_t>(J.oa)[T.s0 + seg] + deposit(r, J.a_row, 0, m_log) : -1;
            row_c[e] = tile_out_row(J, T, e);
        } else if (e < BM + BN) {
            const int j = e - BM;
            const int seg = merge == 1 ? j >> n_log : 0;
            const int64_t c = merge == 1 ? j & (n - 1) : T.tn0 + j;
            const bool ok = merge == 1 ? seg < T.cnt : c < n;
            col_b[j] = ok ? gload<int64_t>(J.ob)[T.s0 + seg] + deposit(c, J.b_col, 0, n_log) : -1;
            col_c[j] = tile_out_col(J, T, j);
        } else {
            const int i = e - BM - BN;
            ak_lo[i] = i < kc ? deposit(i, J.a_k, 0, kc_log) : 0;
            bk_lo[i] = i < kc ? deposit(i, J.b_k, 0, kc_log) : 0;
        }
    }
}

template <int BM, int BNC>
__global__ __launch_bounds__(64 * (BM >= 64 ? BM / 64 : 1) * (BNC >= 32 ? BNC / 32 : 1))
void k_gemm_mfma_g(GemmArgs g) {
    constexpr int WM = BM >= 64 ? BM / 64 : 1;
    constexpr int WN = BNC >= 32 ? BNC / 32 : 1;
    constexpr int NT = 64 * WM * WN;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BNC / WN / 16;
    constexpr int BKC = 8;
    constexpr int BM_LOG = __builtin_ctz(BM), BN_LOG = __builtin_ctz(BNC);
    constexpr int AE = (BM * BKC + NT - 1) / NT;
    constexpr int BE = (BKC * BNC + NT - 1) / NT;
    __shared__ float As_re[2][BKC][BM + 1];
    __shared__ float As_im[2][BKC][BM + 1];
    __shared__ float2 Bs[2][BKC][BNC + 1];
    __shared__ int64_t row_lo[BM], col_lo[BNC], ak_lo[BKC], bk_lo[BKC];

    const int m_log = g.m_log, n_log = g.n_log, k_log = g.k_log;
    const int64_t m = int64_t(1) << m_log, n = int64_t(1) << n_log, k = int64_t(1) << k_log;
    const int tn_log = n_log >= BN_LOG ? n_log - BN_LOG : 0;
    const int64_t tiles = (m / BM) << tn_log;
    const int64_t inst = (int64_t)blockIdx.x / tiles;
    const int64_t tile = (int64_t)blockIdx.x - inst * tiles;
    const int64_t tm0 = (tile >> tn_log) * BM;
    const int64_t tn0 = (tile & ((int64_t(1) << tn_log) - 1)) * BNC;
    const int kc = k < BKC ? (int)k : BKC;
    const int kc_log = k_log < 3 ? k_log : 3;
    const int nb_bits = n_log < BN_LOG ? n_log : BN_LOG;
    for (int i = threadIdx.x; i < BM; i += NT) row_lo[i] = deposit(i, g.a_row, 0, BM_LOG);
    for (int i = threadIdx.x; i < BNC; i += NT) col_lo[i] = deposit(i, g.b_col, 0, nb_bits);
    for (int i = threadIdx.x; i < BKC; i += NT) {
        ak_lo[i] = deposit(i, g.a_k, 0, kc_log);
        bk_lo[i] = deposit(i, g.b_k, 0, kc_log);
    }
    const float2* __restrict__ A = (const float2*)g.A + g.oa[inst] + deposit(tm0, g.a_row, BM_LOG, m_log);
    const float2* __restrict__ B = (const float2*)g.B + g.ob[inst] + deposit(tn0, g.b_col, nb_bits, n_log);
    float* __restrict__ C = (float*)g.C + inst * (2 * m * n);
    __syncthreads();

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM;
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int half = lane >> 5;
    const int sub = lane & 31;
    float2 ra[AE], rb[BE];
    auto load = [&](int64_t k0) {
        const int64_t akh = deposit(k0, g.a_k, kc_log, k_log);
        const int64_t bkh = deposit(k0, g.b_k, kc_log, k_log);
#pragma unroll
        for (int q = 0; q < AE; ++q) {
            const int e = threadIdx.x + q * NT;
            float2 v = make_float2(0.0f, 0.0f);
            if (e < BM * kc) {
                int r, p;
                if (g.a_rowfast) {
                    r = e & (BM - 1);
                    p = e >> BM_LOG;
                } else {
                    p = e & (kc - 1);
                    r = e >> kc_log;
                }
                v = A[row_lo[r] + ak_lo[p] + akh];
            }
            ra[q] = v;
        }
#pragma unroll
        for (int q = 0; q < BE; ++q) {
            const int e = threadIdx.x + q * NT;
            float2 v = make_float2(0.0f, 0.0f);
            if (e < kc * BNC) {
                int p, c;
                if (g.b_colfast) {
                    c = e & (BNC - 1);
                    p = e >> BN_LOG;
                } else {
                    p = e & (kc - 1);
                    c = e >> kc_log;
                }
                if (tn0 + c < n) v = B[col_lo[c] + bk_lo[p] + bkh];
            }
            rb[q] = v;
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < AE; ++q) {
            const int e = threadIdx.x + q * NT;
            if (e < BM * kc) {
                int r, p;
                if (g.a_rowfast) {
                    r = e & (BM - 1);
                    p = e >> BM_LOG;
                } else {
                    p = e & (kc - 1);
                    r = e >> kc_log;
                }
                As_re[buf][p][r] = ra[q].x;
                As_im[buf][p][r] = ra[q].y;
            }
        }
#pragma unroll
        for (int q = 0; q < BE; ++q) {
            const int e = threadIdx.x + q * NT;
            if (e < kc * BNC) {
                int p, c;
                if (g.b_colfast) {
                    c = e & (BNC - 1);
                    p = e >> BN_LOG;
                } else {
                    p = e & (kc - 1);
                    c = e >> kc_log;
                }
                Bs[buf][p][c] = rb[q];
            }
        }
    };
    const int64_t nchunks = k / kc;
    load(0);
    stash(0);
    __syncthreads();
    for (int64_t ch = 0; ch < nchunks; ++ch) {
        const int buf = (int)(ch & 1);
        if (ch + 1 < nchunks) load((ch + 1) * kc);
        for (int p = 0; p < kc; ++p) {
            float a[TM], b[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * (TM * 32) + i * 32 + sub;
                a[i] = half ? As_im[buf][p][row] : As_re[buf][p][row];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int col = wn * (TN * 16) + j * 16 + (sub >> 1);
                const float2 bv = Bs[buf][p][col];
                const int t = sub & 1;
                b[j] = half == 0 ? (t == 0 ? bv.x : bv.y) : (t == 0 ? -bv.y : bv.x);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
        if (ch + 1 < nchunks) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int64_t colf = 2 * (tn0 + wn * (TN * 16) + j * 16) + sub;
            if (colf >= 2 * n) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int64_t row = tm0 + wm * (TM * 32) + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
                C[row * (2 * n) + colf] = acc[i][j][r];
            }
        }
}

// ---------------------------------------------------------------------------
// Wave layout of the grouped matrix-core kernel: WM x WN waves, each holding
// TM x TN 32 x 32 real MFMA blocks (32 rows x 16 complex columns each).  Tiles of
// 64 and 128 rows run 32-row waves (half the accumulators of a 64-row wave) in a
// register budget of four waves per SIMD: 848 tiles of 128 x 32, k = 256, took
// 100 us against 113 us with 64-row waves at two.  (A loop of independent
// 32 x 32 x 2 MFMAs reaches 136, 144 and 154 TFLOP/s with one, two and four waves
// per SIMD.)  The 128 x 64 tile keeps 64-row waves: its 32-row form, eight waves
// per block that each read B again, measured slower.
template <int BM, int BNC>
struct MfmaGroupShape {
    static constexpr bool WIDE = BM == 128 && BNC == 64;
    static constexpr bool ROWS32 = BM >= 64 && !WIDE;
    static constexpr int WM = ROWS32 ? BM / 32 : (BM >= 64 ? BM / 64 : 1);
    static constexpr int WN = BNC >= 32 ? BNC / 32 : 1;
    static constexpr int NT = 64 * WM * WN;
    static constexpr int WAVES = ROWS32 || WIDE ? 4 : 2;      // register budget, waves per SIMD
};
// Grouped matrix-core contractions (FP32 complex on mfma_f32_32x32x2f32, the
// real embedding of K1).  One block per tile descriptor; the tile's row and
// column offsets (A / B element offsets, C row / column offsets, -1 = padding)
// are built in LDS from the job's slice tables, so slices that share an
// operand can fill one tile (merge modes) and any stored layout is read
// without a transpose pass.
//
// Bound by the matrix cores where a level fills the chip (1.1e11 FLOP of k = 1024
// at 117 of 154 TFLOP/s), by waves in flight where it has fewer tiles than two per
// compute unit.  The inner loop is a software pipeline over chunks of 8 (chunks of
// 16 were much slower: LDS per block) that has no branches, so global loads, LDS
// writes, LDS reads and MFMAs of different chunks overlap inside one wave; with
// the reads of a chunk ahead of its own MFMAs and branches on padding it took
// 2107 us for 12 packed circuits (now 2041), 538 us for a 36-qubit QAOA estimate
// (519) and 1128 us for a 25-qubit grid estimate (1113).
// ---------------------------------------------------------------------------
template <int BM, int BNC>
__global__ __launch_bounds__((MfmaGroupShape<BM, BNC>::NT), (MfmaGroupShape<BM, BNC>::WAVES))
void k_mfma_group(const MfmaJob* __restrict__ jobs, const MfmaTile* __restrict__ tiles) {
    constexpr int WM = MfmaGroupShape<BM, BNC>::WM;
    constexpr int WN = MfmaGroupShape<BM, BNC>::WN;
    constexpr int NT = MfmaGroupShape<BM, BNC>::NT;
    constexpr int TM = BM / WM / 32;
    constexpr int TN = BNC / WN / 16;
    constexpr int BKC = 8, BKC_LOG = 3;
    constexpr int BM_LOG = __builtin_ctz(BM), BN_LOG = __builtin_ctz(BNC);
    constexpr int AE = BM * BKC / NT;
    constexpr int BE = (BKC * BNC + NT - 1) / NT;
    // LDS staging, flat: A as [half][p][row] (half 0 real, 1 imaginary parts),
    // B once as [p][2 col + t] (re, im).  The real embedding's second B row
    // (-im, re) is read by the upper half-wave as the swapped pair with the
    // real-part slot negated, so every lane reads its MFMA operand with one
    // 4-byte load and B is staged once.  Row pitch +8 words keeps k-fast
    // staging writes (8 rows x 8 inner indices per 64 lanes) in distinct banks;
    // the +32-word gap between A's halves keeps the two half-waves' reads apart.
    constexpr int AP = BM + 8, AH = BKC * AP + 32, ABUF = 2 * AH;
    constexpr int BP = 2 * BNC + 8, BBUF = BKC * BP;
    __shared__ __align__(16) float As[2 * ABUF];
    __shared__ __align__(16) float Bs[2 * (BBUF + 2)];
    __shared__ int64_t row_a[BM], row_c[BM], col_b[BNC], col_c[BNC], ak_lo[BKC], bk_lo[BKC];
    __shared__ int64_t a_step[32], b_step[32];
    const MfmaTile T = tiles[blockIdx.x];
    const TN_CONST MfmaJob& J = cload<MfmaJob>(jobs)[T.job];
    const int k_log = J.k_log;
    const int64_t k = int64_t(1) << k_log;
    const int kc = k < BKC ? (int)k : BKC;
    const int kc_log = k_log < BKC_LOG ? k_log : BKC_LOG;
    chunk_steps(J.a_k, kc_log, k_log, a_step);
    chunk_steps(J.b_k, kc_log, k_log, b_step);
    tile_tables<BM, BNC, BKC, NT>(J, T, kc_log, row_a, row_c, col_b, col_c, ak_lo, bk_lo);
    __syncthreads();
    const TN_GLOBAL float2* __restrict__ A = gload<float2>(J.A);
    const TN_GLOBAL float2* __restrict__ B = gload<float2>(J.B);
    TN_GLOBAL float* __restrict__ C = gstore<float>(J.C);
    const bool a_rowfast = J.a_rowfast, b_colfast = J.b_colfast;

    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int wm = wave % WM, wn = wave / WM;
    v16f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;
    const int half = lane >> 5;
    const int sub = lane & 31;
    // staging order: element e of a chunk is (row r, inner p) with r fast when
    // the operand's lowest stored bit is a row bit, else p fast; inner indices
    // p >= kc (k < 8) are zero
    auto a_rp = [&](int e, int& r, int& p) {
        if (a_rowfast) {
            r = e & (BM - 1);
            p = e >> BM_LOG;
        } else {
            p = e & (BKC - 1);
            r = e >> BKC_LOG;
        }
    };
    auto b_pc = [&](int e, int& p, int& c) {
        if (b_colfast) {
            c = e & (BNC - 1);
            p = e >> BN_LOG;
        } else {
            p = e & (BKC - 1);
            c = e >> BKC_LOG;
        }
    };
    // chunks of this block: all, or part kpart of ksplit equal parts (split
    // inner sum; the host keeps ksplit a power of two dividing the chunk count)
    const int64_t nch_all = k >= BKC ? k / BKC : 1;
    const int64_t c_begin = nch_all / J.ksplit * T.kpart;
    const int64_t c_end = c_begin + nch_all / J.ksplit;
    // offsets of the high inner bits of the chunk being loaded (chunks are
    // loaded in order: advanced by the step table after each load)
    int64_t kchunk = c_begin;
    int64_t akh = deposit(c_begin << kc_log, J.a_k, kc_log, k_log);
    int64_t bkh = deposit(c_begin << kc_log, J.b_k, kc_log, k_log);
    // this thread's staged elements in the first chunk (a chunk adds akh / bkh).
    // Padding reads an element that the tile reads anyway (its first row or column,
    // inner index 0 of a chunk) and is zeroed when staged (mask bits: q of A, 16 + q of B)
    const TN_GLOBAL float2* pa[AE];
    const TN_GLOBAL float2* pb[BE];
    uint32_t live = 0;
#pragma unroll
    for (int q = 0; q < AE; ++q) {
        int r, p;
        a_rp(threadIdx.x + q * NT, r, p);
        const int64_t base = row_a[r];
        pa[q] = A + ((base >= 0 ? base : row_a[0]) + ak_lo[p]);
        live |= base >= 0 && p < kc ? 1u << q : 0u;
    }
#pragma unroll
    for (int q = 0; q < BE; ++q) {
        const int e = threadIdx.x + q * NT;
        int p = 0, c = 0;
        if (e < BKC * BNC) b_pc(e, p, c);
        const int64_t base = col_b[c];
        pb[q] = B + ((base >= 0 ? base : col_b[0]) + bk_lo[p]);
        live |= e < BKC * BNC && base >= 0 && p < kc ? 1u << (16 + q) : 0u;
    }
    auto load = [&](float2* ra, float2* rb) {
#pragma unroll
        for (int q = 0; q < AE; ++q) ra[q] = gld(pa[q] + akh);
#pragma unroll
        for (int q = 0; q < BE; ++q) rb[q] = gld(pb[q] + bkh);
        const int t = __builtin_ctzll(~(uint64_t)kchunk);      // (past the last chunk: an entry of 0)
        akh += a_step[t];
        bkh += b_step[t];
        ++kchunk;
        // (the scheduler would sink the loads to their first use)
        __builtin_amdgcn_sched_barrier(0);
    };
    // LDS slots of the staged elements: element q is q steps past the first.
    // Threads past the chunk's B elements write to a slot that nobody reads, so
    // staging has no branches and its writes spread over the MFMAs.
    int sa, sb;
    {
        int r, p;
        a_rp(threadIdx.x, r, p);
        sa = p * AP + r;
        b_pc(threadIdx.x, p, r);
        sb = BKC * BNC >= NT || (int)threadIdx.x < BKC * BNC ? p * BP + 2 * r : BBUF;
    }
    const int sa_step = a_rowfast ? NT / BM * AP : NT / BKC;
    const int sb_step = BE == 1 ? 0 : b_colfast ? NT / BNC * BP : 2 * (NT / BKC);
    static_assert(AE == 1 || (NT % BM == 0 && NT % BKC == 0), "staged elements are a fixed step apart");
    static_assert(BE == 1 || (NT % BNC == 0 && NT % BKC == 0), "staged elements are a fixed step apart");
    auto stash = [&](int buf, const float2* ra, const float2* rb) {
        float* as = As + buf * ABUF + sa;
        float* bs = Bs + buf * (BBUF + 2) + sb;
#pragma unroll
        for (int q = 0; q < AE; ++q) {
            const bool ok = live >> q & 1u;
            as[q * sa_step] = ok ? ra[q].x : 0.0f;
            as[AH + q * sa_step] = ok ? ra[q].y : 0.0f;
        }
#pragma unroll
        for (int q = 0; q < BE; ++q)
            *(float2*)&bs[q * sb_step] = live >> (16 + q) & 1u ? rb[q] : make_float2(0.0f, 0.0f);
    };
    // per-lane LDS offsets of the MFMA operands
    int a_off[TM], b_off[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a_off[i] = half * AH + wm * (TM * 32) + i * 32 + sub;
#pragma unroll
    for (int j = 0; j < TN; ++j) b_off[j] = 2 * (wn * (TN * 16) + j * 16) + (half ? (sub ^ 1) : sub);
    const uint32_t b_sign = (half && !(sub & 1)) ? 0x80000000u : 0u;
    // Operands are read from LDS in groups of two inner indices, each group while
    // the MFMAs of the group before run (groups of four: up to 1.5 % slower).
    constexpr int RA = 2, G = BKC / RA;
    static_assert(G % 2 == 0, "the two operand sets alternate");
    // column blocks of 16 that a wave runs: those holding outputs in the block's first
    // wave column (padding is a suffix of the tile's columns: slices past cnt, columns
    // past n), all TN or the first only.  The second wave column of a 64-wide tile runs
    // as many, on padding where the tile has at most 32 columns (a 32-wide tile's case).
    // Every thread reads the same entries, so the choice is the same for the whole block.
    // It is kept in a vector register: a scalar branch makes the accumulators 16 registers
    // larger (108 against 92 on 128 x 32) and the 128 x 64 tile spills.
    int tn_act = 1;
#pragma unroll
    for (int j = 1; j < TN; ++j)
        if (col_c[j * 16] >= 0) tn_act = j + 1;
    if (TN > 1) asm("" : "+v"(tn_act));
    const int64_t nchunks = c_end - c_begin;
    constexpr int WPP = (2 * AE + BE + RA - 1) / RA;      // LDS writes per inner index of a group
    // The inner sum over TNA column blocks.  The block takes one of two forms as a whole:
    // each has the barriers of its chunks, so the choice may not differ between waves.
    auto sum = [&](auto tna) {
        constexpr int TNA = decltype(tna)::value;
        float a[2][RA][TM], b[2][RA][TNA];
        // operands of group g of the chunk in LDS buffer buf
        auto read = [&](int buf, int g, float (&x)[RA][TM], float (&y)[RA][TNA]) {
            const float* as = As + buf * ABUF + g * RA * AP;
            const float* bs = Bs + buf * (BBUF + 2) + g * RA * BP;
#pragma unroll
            for (int p = 0; p < RA; ++p) {
#pragma unroll
                for (int i = 0; i < TM; ++i) x[p][i] = as[p * AP + a_off[i]];
#pragma unroll
                for (int j = 0; j < TNA; ++j) y[p][j] = bs[p * BP + b_off[j]];
            }
            __builtin_amdgcn_sched_barrier(0);             // ahead of the MFMAs that follow
        };
        auto multiply = [&](const float (&x)[RA][TM], const float (&y)[RA][TNA], bool staged) {
#pragma unroll
            for (int p = 0; p < RA; ++p) {
                float z[TNA];
#pragma unroll
                for (int j = 0; j < TNA; ++j) z[j] = __uint_as_float(__float_as_uint(y[p][j]) ^ b_sign);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TNA; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[p][i], z[j], acc[i][j], 0, 0, 0);
            }
            if (staged) {
                // the LDS writes and their VALU work between the MFMAs
#pragma unroll
                for (int p = 0; p < RA; ++p) {
                    __builtin_amdgcn_sched_group_barrier(0x008, TM * TNA, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 3 * WPP, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, WPP, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        float2 ra[AE], rb[BE];
        load(ra, rb);
        stash(0, ra, rb);
        if (nchunks > 1) load(ra, rb);
        __syncthreads();
        read(0, 0, a[0], b[0]);
        // chunk c sits in LDS buffer c & 1, its first group in operand set 0, and
        // chunk c + 1 in the registers (or on its way there).  During the first
        // group's MFMAs chunk c + 1 goes to LDS and the loads of chunk c + 2 are
        // issued after it (a whole chunk of MFMAs before they are needed); the
        // barrier comes before the last group's MFMAs, which cover the reads of
        // the next chunk's first group.
        auto chunk = [&](int buf, auto next, auto after) {
            constexpr bool NEXT = decltype(next)::value, AFTER = decltype(after)::value;
#pragma unroll
            for (int g = 0; g + 1 < G; ++g) {
                read(buf, g + 1, a[(g + 1) & 1], b[(g + 1) & 1]);
                if (NEXT && g == 0) stash(buf ^ 1, ra, rb);
                multiply(a[g & 1], b[g & 1], NEXT && g == 0);
                if (AFTER && g == 0) load(ra, rb);
            }
            if constexpr (NEXT) {
                __syncthreads();
                read(buf ^ 1, 0, a[0], b[0]);
            }
            multiply(a[1], b[1], false);
        };
        constexpr std::integral_constant<bool, true> yes{};
        constexpr std::integral_constant<bool, false> no{};
        int buf = 0;
        for (int64_t ch = 0; ch + 2 < nchunks; ++ch, buf ^= 1) chunk(buf, yes, yes);
        if (nchunks > 1) {
            chunk(buf, yes, no);
            buf ^= 1;
        }
        chunk(buf, no, no);
    };
    if (TN == 1 || tn_act == TN) sum(std::integral_constant<int, TN>{});
    else sum(std::integral_constant<int, 1>{});

    // split inner sum: this block's part goes to its row-major [BM][BNC] partial
    // tile (padding skipped), added to the others' by k_split_reduce
    const bool to_partial = J.ksplit > 1;
    TN_GLOBAL float* __restrict__ O =
        to_partial ? gstore<float>(J.partial) + ((int64_t)T.pair * J.ksplit + T.kpart) * (2 * BM * BNC) : C;
    // output offsets of this lane's 16 rows and TN columns read ahead of the
    // stores (one LDS wait per row block instead of one per store)
    const int part = sub & 1;
    int64_t ccs[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int col = wn * (TN * 16) + j * 16 + (sub >> 1);
        ccs[j] = to_partial ? (col_c[col] < 0 ? -1 : col) : col_c[col];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        int64_t rcs[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int row = wm * (TM * 32) + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3);
            const int64_t rc = row_c[row];
            rcs[r] = to_partial ? (rc < 0 ? -1 : (int64_t)row * BNC) : rc;
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (ccs[j] < 0) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (rcs[r] >= 0) O[2 * (rcs[r] + ccs[j]) + part] = acc[i][j][r];
        }
    }
}

// ---------------------------------------------------------------------------
// Grouped gathered contractions: every small step of one tree level (all
// clusters, all plans) in one launch.  A block finds its job with one load
// (block table).  Operands are read in their stored order (no transpose pass):
// a row's or column's offset is its index cut into the runs of stored bits it
// covers, an inner index's offset comes from the job's table (the first eight
// entries inline in the record).  Records, tables and all that is the same for
// a block are scalar loads, so a step without long sums has no barrier and no
// LDS: its time is the chain block table -> record -> slice offsets -> operands.
//   split == 0: a thread computes 2^rl rows x 2^cl adjacent columns, inner loop
//               in registers, products added in inner-index order;
//   split == 1: a block computes 2^rl x 2^cl outputs (long inner sums), each
//               operand element read once for all of them, partial sums reduced
//               in FP64 in a fixed order;
//   split == 2: a block computes 64 outputs, each of its four waves a quarter of
//               every chunk of the inner sum; the four partial sums are added in
//               FP64 in order (few outputs, sums long enough that one thread's
//               chain of loads is what the launch takes).
// Bound: memory (L2 and HBM) for large steps, the chain of loads for small ones.
// Against one output per thread and block with the record in LDS: 32 slices of
// 2 x 2^19 over 4 terms 251 -> 116 us (302 MB), 1446 slices of 4 x 2 over 8192
// terms 207 -> 82 us, 352 of 4 x 4 over 16384 102 -> 54 us, a level of 8 x 8
// sums of 1024 terms 12.4 -> 6.0 us.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t run_offset(const TN_CONST uint32_t* runs, int n, uint32_t x) {
    int64_t o = 0;
    for (int i = 0; i < n; ++i) {
        const uint32_t q = runs[i];
        o |= (int64_t)((x >> (q & 31u)) & ((2u << ((q >> 8) & 31u)) - 1u)) << ((q >> 16) & 63u);
    }
    return o;
}

// V adjacent complex numbers (FP32: two per 16-byte load)
typedef float f4 __attribute__((ext_vector_type(4)));
template <typename R, typename C2, int V>
__device__ __forceinline__ void vload(const TN_GLOBAL C2* p, R (&re)[V], R (&im)[V]) {
    if constexpr (V == 1) {
        const C2 v = gld(p);
        re[0] = v.x;
        im[0] = v.y;
    } else {
        static_assert(sizeof(R) == 4, "FP64 elements are 16 bytes each");
#pragma unroll
        for (int q = 0; q < V; q += 2) {
            const f4 v = *(const TN_GLOBAL f4*)(p + q);
            re[q] = v[0];
            im[q] = v[1];
            re[q + 1] = v[2];
            im[q + 1] = v[3];
        }
    }
}
template <typename R, typename C2, int V>
__device__ __forceinline__ void vstore(TN_GLOBAL C2* p, const R (&re)[V], const R (&im)[V]) {
    if constexpr (V == 1) {
        C2 v;
        v.x = re[0];
        v.y = im[0];
        gst(p, v);
    } else {
#pragma unroll
        for (int q = 0; q < V; q += 2) *(TN_GLOBAL f4*)(p + q) = f4{re[q], im[q], re[q + 1], im[q + 1]};
    }
}

// One thread of a small step.  UNI: the block's outputs lie in one row group
// of one slice, whose elements are then the same for every thread: scalar loads.
// QUARTER: this thread's wave sums a quarter of the inner indices of its output
// and leaves the partial sum in red.
template <typename R, typename C2, int RL, int CL, bool UNI, bool QUARTER = false>
__device__ __forceinline__ void gett_rows(const TN_CONST GettJob* J, int64_t local, int tid, double2* red = nullptr) {
    constexpr int RPT = 1 << RL, V = 1 << CL;
    constexpr int W = RPT * V * (sizeof(R) / 4);               // accumulated words / 2
    // inner indices whose loads are in flight together
    constexpr int P = UNI ? (RPT * (int)sizeof(R) <= 8 ? 4 : 2)
                          : W == 1 ? 8 : W <= 4 ? 4 : (W == 8 ? 4 : 2) / (sizeof(R) / 4);
    const int m_log = J->m_log, n_log = J->n_log, k_log = J->k_log;
    const int mn_log = m_log + n_log;
    const int cw = n_log - CL;                                 // log2 column groups of a row group
    const int64_t o = QUARTER ? local * 64 + (tid & 63) : local * 256 + tid;
    if (!UNI && o >= (J->n_inst << (mn_log - RL - CL))) return;
    const int64_t c = (o & ((int64_t(1) << cw) - 1)) << CL;
    const int64_t rest = (UNI ? local * 256 : o) >> cw;
    const int64_t r0 = (rest & ((int64_t(1) << (m_log - RL)) - 1)) << RL;
    const int64_t inst = rest >> (m_log - RL);
    int64_t ao, bo;
    if constexpr (UNI) {
        ao = cload<int64_t>(J->oa)[inst];
        bo = cload<int64_t>(J->ob)[inst];
    } else {
        ao = gload<int64_t>(J->oa)[inst];
        bo = gload<int64_t>(J->ob)[inst];
    }
    const C2* Ag = (const C2*)J->A + (ao + run_offset(J->row_runs, J->n_row_runs, (uint32_t)r0));
    const TN_GLOBAL C2* Bp = gload<C2>(J->B) + (bo + run_offset(J->col_runs, J->n_col_runs, (uint32_t)c));
    int64_t rlo[RPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i) rlo[i] = J->rlo[i];
    R sr[RPT][V], si[RPT][V];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int v = 0; v < V; ++v) sr[i][v] = si[i][v] = 0;
    auto lda = [&](int64_t off) {
        if constexpr (UNI) {
            const TN_CONST R* q = cload<R>(Ag + off);
            C2 v;
            v.x = q[0];
            v.y = q[1];
            return v;
        } else {
            return gld(gload<C2>(Ag) + off);
        }
    };
    const int kc_log = J->kc_log;
    const int kc = QUARTER ? 1 << (kc_log - 2) : 1 << kc_log;
    const TN_CONST GettOff* kt = kc_log <= 3 ? J->k8 : cload<GettOff>(J->koff);
    if (QUARTER) kt += __builtin_amdgcn_readfirstlane(tid >> 6) << (kc_log - 2);
    const TN_CONST GettStep* steps = cload<GettStep>(J->steps);
    const int64_t nh = int64_t(1) << (k_log - kc_log);
    int64_t ahh = 0, bhh = 0;
    // P inner indices: their loads, then their products (in order)
    auto batch = [&](const GettOff (&kk)[P], auto all, int n, auto&& between) {
        constexpr bool ALL = decltype(all)::value;
        R br[P][V], bi[P][V];
        C2 a[P][RPT];
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (ALL || u < n) {
                vload<R, C2, V>(Bp + (bhh + kk[u].b), br[u], bi[u]);
                const int64_t ap = ahh + kk[u].a;
#pragma unroll
                for (int i = 0; i < RPT; ++i) a[u][i] = lda(rlo[i] + ap);
            }
        between();
#pragma unroll
        for (int u = 0; u < P; ++u)
            if (ALL || u < n) {
#pragma unroll
                for (int i = 0; i < RPT; ++i)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        sr[i][v] += a[u][i].x * br[u][v] - a[u][i].y * bi[u][v];
                        si[i][v] += a[u][i].x * bi[u][v] + a[u][i].y * br[u][v];
                    }
            }
    };
    GettOff kk[P];
#pragma unroll
    for (int u = 0; u < P; ++u)
        if (u < kc) kk[u] = GettOff{kt[u].a, kt[u].b};
    for (int64_t h = 0;;) {
        if (kc < P) {                                          // a chunk is one short batch
            batch(kk, std::integral_constant<bool, false>{}, kc, [] {});
        } else {
            for (int p = 0; p < kc; p += P) {
                // the next batch's offsets arrive during this one's loads
                GettOff nx[P];
                const int q0 = (p + P) & (kc - 1);
                batch(kk, std::integral_constant<bool, true>{}, P, [&] {
#pragma unroll
                    for (int u = 0; u < P; ++u) nx[u] = GettOff{kt[q0 + u].a, kt[q0 + u].b};
                });
#pragma unroll
                for (int u = 0; u < P; ++u) kk[u] = nx[u];
            }
        }
        if (++h >= nh) break;
        const int t = __builtin_ctzll((uint64_t)h);            // chunk h - 1 -> h
        ahh += steps[t].a;
        bhh += steps[t].b;
    }
    if constexpr (QUARTER) {
        red[tid] = make_double2((double)sr[0][0], (double)si[0][0]);
        return;
    }
    TN_GLOBAL C2* Cp = gstore<C2>(J->C) + ((inst << mn_log) + (r0 << n_log) + c);
#pragma unroll
    for (int i = 0; i < RPT; ++i) vstore<R, C2, V>(Cp + ((int64_t)i << n_log), sr[i], si[i]);
}

// A block's partial sums of 2^RL x 2^CL outputs: thread t takes inner indices
// t + 256 h.  The wave's sums go to red[64 wave + output] (FP64, a fixed-order
// butterfly that halves the outputs a lane holds at each exchange).
template <typename R, typename C2, int RL, int CL>
__device__ __forceinline__ void gett_dot(const TN_CONST GettJob* J, int64_t local, int tid, double2* red) {
    constexpr int NR = 1 << RL, NC = 1 << CL, N = NR * NC;
    // U inner indices' loads are in flight together (NR + NC elements each)
    constexpr int U = (sizeof(R) == 4 ? 16 : 8) / (N == 1 ? 1 : N == 2 ? 2 : N == 4 ? (sizeof(R) == 4 ? 2 : 4)
                                                                                     : N == 8 ? 4 : 8);
    const int tm = J->m_log - RL, tc = J->n_log - CL;
    const int64_t inst = local >> (tm + tc);
    const uint32_t r0 = (uint32_t)((local >> tc) & ((int64_t(1) << tm) - 1)) << RL;
    const uint32_t c0 = (uint32_t)(local & ((int64_t(1) << tc) - 1)) << CL;
    const TN_GLOBAL C2* Ap = gload<C2>(J->A) + (cload<int64_t>(J->oa)[inst] + run_offset(J->row_runs, J->n_row_runs, r0));
    const TN_GLOBAL C2* Bp = gload<C2>(J->B) + (cload<int64_t>(J->ob)[inst] + run_offset(J->col_runs, J->n_col_runs, c0));
    const TN_GLOBAL uint32_t* kt = gload<uint32_t>(J->koff);
    const TN_CONST GettStep* steps = cload<GettStep>(J->steps);
    int64_t ah = kt[2 * tid], bh = kt[2 * tid + 1];
    int64_t rlo[NR], clo[NC];
#pragma unroll
    for (int i = 0; i < NR; ++i) rlo[i] = J->rlo[i];
#pragma unroll
    for (int j = 0; j < NC; ++j) clo[j] = J->clo[j];
    R sr[N], si[N];
#pragma unroll
    for (int q = 0; q < N; ++q) sr[q] = si[q] = 0;
    const int64_t nh = int64_t(1) << (J->k_log - 8);
    const int64_t step = nh >= U ? U : nh;
    for (int64_t h0 = 0; h0 < nh; h0 += step) {
        C2 a[U][NR], b[U][NC];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < step) {
#pragma unroll
                for (int i = 0; i < NR; ++i) a[u][i] = gld(Ap + (ah + rlo[i]));
#pragma unroll
                for (int j = 0; j < NC; ++j) b[u][j] = gld(Bp + (bh + clo[j]));
                if (h0 + u + 1 < nh) {
                    const int t = __builtin_ctzll((uint64_t)(h0 + u + 1));
                    ah += steps[t].a;
                    bh += steps[t].b;
                }
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (u < step) {
#pragma unroll
                for (int i = 0; i < NR; ++i)
#pragma unroll
                    for (int j = 0; j < NC; ++j) {
                        sr[i * NC + j] += a[u][i].x * b[u][j].x - a[u][i].y * b[u][j].y;
                        si[i * NC + j] += a[u][i].x * b[u][j].y + a[u][i].y * b[u][j].x;
                    }
            }
    }
    double vr[N], vi[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        vr[q] = (double)sr[q];
        vi[q] = (double)si[q];
    }
    const int lane = tid & 63;
    constexpr int NLOG = RL + CL;
#pragma unroll
    for (int s = 0; s < NLOG; ++s) {
        const int half = N >> (s + 1), off = 32 >> s;
        const bool up = lane & off;             // keeps the upper half of the outputs
#pragma unroll
        for (int q = 0; q < N / 2; ++q) {
            if (q >= half) break;
            const double kr = up ? vr[q + half] : vr[q], ki = up ? vi[q + half] : vi[q];
            const double gr = up ? vr[q] : vr[q + half], gi = up ? vi[q] : vi[q + half];
            vr[q] = kr + __shfl_xor(gr, off);
            vi[q] = ki + __shfl_xor(gi, off);
        }
    }
#pragma unroll
    for (int s = NLOG; s < 6; ++s) {
        vr[0] += __shfl_xor(vr[0], 32 >> s);
        vi[0] += __shfl_xor(vi[0], 32 >> s);
    }
    if ((lane & ((64 >> NLOG) - 1)) == 0) red[(tid >> 6) * 64 + (lane >> (6 - NLOG))] = make_double2(vr[0], vi[0]);
}

// after a barrier: the four waves' sums in order, one thread per output
template <typename R, typename C2>
__device__ __forceinline__ void gett_finish(const TN_CONST GettJob* J, int64_t local, int tid, const double2* red) {
    const int rl = J->rl, cl = J->cl, n_log = J->n_log;
    int64_t at;
    if (J->split == 2) {
        at = local * 64 + tid;
        if (tid >= 64 || at >= (J->n_inst << (J->m_log + n_log))) return;
    } else {
        if (tid >= 1 << (rl + cl)) return;
        const int tm = J->m_log - rl, tc = n_log - cl;
        const int64_t inst = local >> (tm + tc);
        const int64_t r = (((local >> tc) & ((int64_t(1) << tm) - 1)) << rl) + (tid >> cl);
        const int64_t c = ((local & ((int64_t(1) << tc) - 1)) << cl) + (tid & ((1 << cl) - 1));
        at = (((inst << J->m_log) + r) << n_log) + c;
    }
    C2 out;
    out.x = (R)(((red[tid].x + red[64 + tid].x) + red[128 + tid].x) + red[192 + tid].x);
    out.y = (R)(((red[tid].y + red[64 + tid].y) + red[128 + tid].y) + red[192 + tid].y);
    gst(gstore<C2>(J->C) + at, out);
}

// One 256-thread block of a job with one output per thread (per wave, per block),
// up to the split sums' barrier; no scalar loads of operands.
template <typename R, typename C2>
__device__ __forceinline__ void gett_block_one(const TN_CONST GettJob* J, int64_t local, int tid, double2* red) {
    if (J->split == 2) gett_rows<R, C2, 0, 0, false, true>(J, local, tid, red);
    else if (J->split) gett_dot<R, C2, 0, 0>(J, local, tid, red);
    else gett_rows<R, C2, 0, 0, false>(J, local, tid);
}

// The same for every job.  Rows that are the same for a whole block are read
// with scalar loads (nothing in the launch writes them).
template <typename R, typename C2>
__device__ __forceinline__ void gett_block(const TN_CONST GettJob* J, int64_t local, int tid, double2* red) {
    constexpr bool F32 = sizeof(R) == 4;
    const int shape = J->rl * 4 + J->cl;
    if (shape == 0 || J->split == 2) {
        gett_block_one<R, C2>(J, local, tid, red);
        return;
    }
    if (J->split) {
        switch (shape) {
        case 1: gett_dot<R, C2, 0, 1>(J, local, tid, red); break;
        case 4: gett_dot<R, C2, 1, 0>(J, local, tid, red); break;
        case 5: gett_dot<R, C2, 1, 1>(J, local, tid, red); break;
        }
        if constexpr (F32) switch (shape) {
        case 6: gett_dot<R, C2, 1, 2>(J, local, tid, red); break;
        case 9: gett_dot<R, C2, 2, 1>(J, local, tid, red); break;
        case 10: gett_dot<R, C2, 2, 2>(J, local, tid, red); break;
        }
        return;
    }
    if (J->n_log - J->cl >= 8) {
        if constexpr (F32) switch (shape) {
        case 1: gett_rows<R, C2, 0, 1, true>(J, local, tid); return;
        case 5: gett_rows<R, C2, 1, 1, true>(J, local, tid); return;
        case 9: gett_rows<R, C2, 2, 1, true>(J, local, tid); return;
        case 2: gett_rows<R, C2, 0, 2, true>(J, local, tid); return;
        case 6: gett_rows<R, C2, 1, 2, true>(J, local, tid); return;
        case 10: gett_rows<R, C2, 2, 2, true>(J, local, tid); return;
        } else switch (shape) {
        case 4: gett_rows<R, C2, 1, 0, true>(J, local, tid); return;
        case 8: gett_rows<R, C2, 2, 0, true>(J, local, tid); return;
        case 12: gett_rows<R, C2, 3, 0, true>(J, local, tid); return;
        }
    }
    switch (shape) {
    case 4: gett_rows<R, C2, 1, 0, false>(J, local, tid); break;
    case 8: gett_rows<R, C2, 2, 0, false>(J, local, tid); break;
    case 12: gett_rows<R, C2, 3, 0, false>(J, local, tid); break;
    }
    if constexpr (F32) switch (shape) {
    case 1: gett_rows<R, C2, 0, 1, false>(J, local, tid); break;
    case 5: gett_rows<R, C2, 1, 1, false>(J, local, tid); break;
    case 9: gett_rows<R, C2, 2, 1, false>(J, local, tid); break;
    }
}

// One launch for the small steps of one tree level: block b runs job
// block_job[b] & 0x7fffffff, in FP64 when bit 31 is set (the dominant-term
// pass's jobs of the same level), else in FP32.  The table is built on the
// host, so a block finds its job with one load.
__global__ __launch_bounds__(256, 4) void k_gett_group(const GettJob* __restrict__ jobs,
                                                       const int32_t* __restrict__ block_job) {
    __shared__ double2 red[256];
    const uint32_t e = (uint32_t)cload<int32_t>(block_job)[blockIdx.x];
    const TN_CONST GettJob* J = cload<GettJob>(jobs) + (e & 0x7fffffffu);
    const int64_t local = (int64_t)blockIdx.x - J->block0;
    const int tid = (int)threadIdx.x;
    if (e >> 31) gett_block<double, double2>(J, local, tid, red);
    else gett_block<float, float2>(J, local, tid, red);
    if (!J->split) return;
    __syncthreads();
    if (e >> 31) gett_finish<double, double2>(J, local, tid, red);
    else gett_finish<float, float2>(J, local, tid, red);
}

// Consecutive small levels in one launch.  The launch's blocks are the
// independent parts of those levels (no part touches memory that another one
// writes): a block of four 256-thread groups walks its part's levels, four
// 256-thread blocks of a level at a time, with a barrier after each level, so no
// block waits for another.  The values of a level are read back by the same
// block through the L1 that it wrote them through; only records and tables
// (written by no block) use scalar loads.
//   Bound: the chain of loads of each level, about 1.2 us with its records in
//   the caches (8-qubit chain: its three levels 5.3 us; as launches 3.4 + 3.2 +
//   3.5 us and the gaps between them), 3 to 4 us in the first pass over a schedule.
__global__ __launch_bounds__(1024) void k_gett_chain(const GettChainPart* __restrict__ parts,
                                                     const GettChainBlock* __restrict__ blocks) {
    __shared__ double2 red[2][1024];
    const TN_CONST GettChainPart* P = cload<GettChainPart>(parts) + blockIdx.x;
    const TN_CONST GettChainBlock* list = cload<GettChainBlock>(blocks);
    const int grp = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8), tid = (int)threadIdx.x & 255;
    const int nl = P->n_levels, last = P->start[nl] - 1;
    const uint32_t split_levels = P->split_levels;
    // the record of this group's next block is read during the current one
    const TN_CONST GettChainBlock* B = list + (P->start[0] + grp < last ? P->start[0] + grp : last);
    const TN_CONST GettJob* J = cload<GettJob>(B->job);
    int64_t local = B->local;
    int wide = B->fp64, par = 0;
    for (int l = 0; l < nl; ++l) {
        const int at = P->start[l], n = P->start[l + 1] - at;
        const bool split = split_levels >> l & 1;
        if (l) __syncthreads();                // the level before is written
        for (int v = 0; v < n; v += 4, par ^= 1) {
            const bool mine = v + grp < n;
            const int next = (v + 4 < n ? at + v + 4 : at + n) + grp;
            const TN_CONST GettChainBlock* Bn = list + (next < last ? next : last);
            const TN_CONST GettJob* Jn = cload<GettJob>(Bn->job);
            const int64_t local_n = Bn->local;
            const int wide_n = Bn->fp64;
            double2* r = red[par] + 256 * grp;
            if (mine) {
                if (wide) gett_block_one<double, double2>(J, local, tid, r);
                else gett_block_one<float, float2>(J, local, tid, r);
            }
            if (split) {
                __syncthreads();               // (the other buffer's sums were finished before it)
                if (mine && J->split) {
                    if (wide) gett_finish<double, double2>(J, local, tid, r);
                    else gett_finish<float, float2>(J, local, tid, r);
                }
            }
            J = Jn;
            local = local_n;
            wide = wide_n;
        }
    }
}

// ---------------------------------------------------------------------------
// Small shapes: one thread per output element, k loop in registers.
// ---------------------------------------------------------------------------
template <typename R, typename C2>
__global__ __launch_bounds__(256) void k_gemm_small(GemmArgs g) {
    const int64_t total = g.n_inst << (g.m_log + g.n_log);
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int64_t n = int64_t(1) << g.n_log, m = int64_t(1) << g.m_log, k = int64_t(1) << g.k_log;
    const int64_t inst = idx >> (g.m_log + g.n_log);
    const int64_t rc = idx & ((int64_t(1) << (g.m_log + g.n_log)) - 1);
    const int64_t r = rc >> g.n_log, c = rc & (n - 1);
    const C2* A = (const C2*)g.A + pick(g.ia_mode, g.ia, inst) * g.strideA;
    const C2* B = (const C2*)g.B + pick(g.ib_mode, g.ib, inst) * g.strideB;
    R sr = 0, si = 0;
    for (int64_t p = 0; p < k; ++p) {
        const C2 a = g.transA ? A[p * m + r] : A[r * k + p];
        const C2 b = g.transB ? B[c * k + p] : B[p * n + c];
        sr += a.x * b.x - a.y * b.y;
        si += a.x * b.y + a.y * b.x;
    }
    C2 o;
    o.x = sr;
    o.y = si;
    ((C2*)g.C)[idx] = o;
}

// ---------------------------------------------------------------------------
// Tiny outputs with long k (inner products): one block per output element,
// strided partial sums, FP64 tree reduction in LDS.
// ---------------------------------------------------------------------------
template <typename R, typename C2>
__global__ __launch_bounds__(256) void k_gemm_splitk(GemmArgs g) {
    __shared__ double red_r[256];
    __shared__ double red_i[256];
    const int64_t n = int64_t(1) << g.n_log, m = int64_t(1) << g.m_log, k = int64_t(1) << g.k_log;
    const int64_t out = blockIdx.x;
    const int64_t inst = out >> (g.m_log + g.n_log);
    const int64_t rc = out & ((int64_t(1) << (g.m_log + g.n_log)) - 1);
    const int64_t r = rc >> g.n_log, c = rc & (n - 1);
    const C2* A = (const C2*)g.A + pick(g.ia_mode, g.ia, inst) * g.strideA;
    const C2* B = (const C2*)g.B + pick(g.ib_mode, g.ib, inst) * g.strideB;
    R sr = 0, si = 0;
    for (int64_t p = threadIdx.x; p < k; p += blockDim.x) {
        const C2 a = g.transA ? A[p * m + r] : A[r * k + p];
        const C2 b = g.transB ? B[c * k + p] : B[p * n + c];
        sr += a.x * b.x - a.y * b.y;
        si += a.x * b.y + a.y * b.x;
    }
    red_r[threadIdx.x] = (double)sr;
    red_i[threadIdx.x] = (double)si;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            red_r[threadIdx.x] += red_r[threadIdx.x + s];
            red_i[threadIdx.x] += red_i[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        C2 o;
        o.x = (R)red_r[0];
        o.y = (R)red_i[0];
        ((C2*)g.C)[out] = o;
    }
}

// ---------------------------------------------------------------------------
// FP64 tiled GEMM (complex128) for the dominant-term pass: 64x64 output tile,
// 256 threads each holding a 4x4 block, k staged through LDS in chunks of 8.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_gemm_tiled_c128(GemmArgs g) {
    constexpr int BM = 64, BN = 64, BK = 8;
    __shared__ double2 As[BK][BM];
    __shared__ double2 Bs[BK][BN];
    const int64_t m = int64_t(1) << g.m_log, n = int64_t(1) << g.n_log, k = int64_t(1) << g.k_log;
    const int tn_log = g.n_log - 6;
    const int64_t tiles = (m / BM) << tn_log;
    const int64_t inst = blockIdx.x / tiles;
    const int64_t tile = blockIdx.x - inst * tiles;
    const int64_t tm0 = (tile >> tn_log) * BM, tn0 = (tile & ((int64_t(1) << tn_log) - 1)) * BN;
    const double2* A = (const double2*)g.A + pick(g.ia_mode, g.ia, inst) * g.strideA;
    const double2* B = (const double2*)g.B + pick(g.ib_mode, g.ib, inst) * g.strideB;
    double2* C = (double2*)g.C + inst * m * n;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    double accr[4][4], acci[4][4];
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) accr[i][j] = acci[i][j] = 0.0;
    const int kc = k < BK ? (int)k : BK;
    for (int64_t k0 = 0; k0 < k; k0 += kc) {
        for (int e = threadIdx.x; e < BM * kc; e += 256) {
            int r, p;
            if (!g.transA) { r = e / kc; p = e % kc; As[p][r] = A[(tm0 + r) * k + k0 + p]; }
            else { p = e / BM; r = e % BM; As[p][r] = A[(k0 + p) * m + tm0 + r]; }
        }
        for (int e = threadIdx.x; e < kc * BN; e += 256) {
            int p, c;
            if (!g.transB) { p = e / BN; c = e % BN; Bs[p][c] = B[(k0 + p) * n + tn0 + c]; }
            else { c = e / kc; p = e % kc; Bs[p][c] = B[(tn0 + c) * k + k0 + p]; }
        }
        __syncthreads();
        for (int p = 0; p < kc; ++p) {
            double2 a[4], b[4];
            for (int i = 0; i < 4; ++i) a[i] = As[p][ty + 16 * i];
            for (int j = 0; j < 4; ++j) b[j] = Bs[p][tx + 16 * j];
            for (int i = 0; i < 4; ++i)
                for (int j = 0; j < 4; ++j) {
                    accr[i][j] += a[i].x * b[j].x - a[i].y * b[j].y;
                    acci[i][j] += a[i].x * b[j].y + a[i].y * b[j].x;
                }
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) {
            double2 o;
            o.x = accr[i][j];
            o.y = acci[i][j];
            C[(tm0 + ty + 16 * i) * n + tn0 + tx + 16 * j] = o;
        }
}

// ---------------------------------------------------------------------------
// Grouped FP64 tiles (complex128 FMA): the descriptors of the grouped
// matrix-core launch (merge modes, slice tables, per-bit positions) on
// 16TT x 16TT output tiles (TT = 4: 64 x 64; TT = 2: 32 x 32, four times the tiles
// for jobs that would leave CUs idle); 256 threads, TT x TT outputs each, inner
// chunks of 8 staged in LDS through the tile's row / column offset tables.
// ---------------------------------------------------------------------------
#ifndef TILE64_MFMA
#define TILE64_MFMA 1
#endif
// MF = 1: the products run on the FP64 matrix cores (v_mfma_f64_16x16x4f64 on the
// real embedding, as the FP32 kernel: one instruction is 16 rows x 8 complex
// columns x 2 complex inner indices); the four waves take the tile's quadrants.
// Operands come from the same LDS rows; each lane reads one double per operand
// per instruction instead of a thread reading TT complex values of A and of B
// per inner index (the FMA form reads 1 byte of LDS per flop).
template <int TT, bool MF>
__global__ __launch_bounds__(256) void k_tile64_group(const MfmaJob* __restrict__ jobs,
                                                      const MfmaTile* __restrict__ tiles) {
    constexpr int BM = 16 * TT, BN = 16 * TT, BK = 8, BK_LOG = 3;
    constexpr int BM_LOG = __builtin_ctz(BM), BN_LOG = __builtin_ctz(BN);
    constexpr int SE = (BM * BK + 255) / 256;   // staged elements per thread and operand
    // +2 elements per row: k-fast staging writes of 16 lanes fall in distinct banks;
    // two buffers: chunk ch + 1 is stashed while chunk ch is multiplied
    __shared__ double2 As2[2][BK][BM + 2];
    __shared__ double2 Bs2[2][BK][BN + 2];
    __shared__ int64_t row_a[BM], row_c[BM], col_b[BN], col_c[BN], ak_lo[BK], bk_lo[BK];
    __shared__ int64_t a_step[32], b_step[32];
    const MfmaTile T = tiles[blockIdx.x];
    const TN_CONST MfmaJob& J = cload<MfmaJob>(jobs)[T.job];
    const int k_log = J.k_log;
    const int64_t k = int64_t(1) << k_log;
    const int kc = k < BK ? (int)k : BK;
    const int kc_log = k_log < BK_LOG ? k_log : BK_LOG;
    chunk_steps(J.a_k, kc_log, k_log, a_step);
    chunk_steps(J.b_k, kc_log, k_log, b_step);
    tile_tables<BM, BN, BK, 256>(J, T, kc_log, row_a, row_c, col_b, col_c, ak_lo, bk_lo);
    __syncthreads();
    const TN_GLOBAL double2* __restrict__ A = gload<double2>(J.A);
    const TN_GLOBAL double2* __restrict__ B = gload<double2>(J.B);
    TN_GLOBAL double2* __restrict__ C = gstore<double2>(J.C);
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    double accr[MF ? 1 : TT][MF ? 1 : TT], acci[MF ? 1 : TT][MF ? 1 : TT];
    // matrix-core form: wave quadrant (rows wr0.., complex columns wc0..), WR x WC
    // instructions of 16 rows x 8 complex columns each
    constexpr int WR = MF ? BM / 32 : 1, WC = MF ? BN / 16 : 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr0 = (wave & 1) * (BM / 2), wc0 = (wave >> 1) * (BN / 2);
    const int kpart = (lane >> 4) & 1;           // real-embedding row: 0 = Re, 1 = Im of A's element
    const int tcol = lane & 1;                   // output component of this lane's column
    v4d acc[WR][WC];
    if constexpr (MF) {
#pragma unroll
        for (int i = 0; i < WR; ++i)
#pragma unroll
            for (int j = 0; j < WC; ++j) acc[i][j] = v4d{0.0, 0.0, 0.0, 0.0};
    } else {
#pragma unroll
        for (int i = 0; i < TT; ++i)
#pragma unroll
            for (int j = 0; j < TT; ++j) accr[i][j] = acci[i][j] = 0.0;
    }
    const int64_t nch_all = k >= BK ? k / BK : 1;
    const int64_t c_begin = nch_all / J.ksplit * T.kpart;
    const int64_t c_end = c_begin + nch_all / J.ksplit;
    int64_t akh = deposit(c_begin << kc_log, J.a_k, kc_log, k_log);
    int64_t bkh = deposit(c_begin << kc_log, J.b_k, kc_log, k_log);
    // this thread's staged elements: LDS slots and offsets inside a chunk
    // (fixed over the chunks; -1 = padding, staged as zero)
    int sa_r[SE], sa_p[SE], sb_c[SE], sb_p[SE];
    int64_t aoff[SE], boff[SE];
#pragma unroll
    for (int q = 0; q < SE; ++q) {
        const int e = threadIdx.x + q * 256;
        int r = 0, p = 0, pb = 0, c = 0;
        if (J.a_rowfast) {
            r = e & (BM - 1);
            p = e >> BM_LOG;
        } else {
            p = e & (BK - 1);
            r = e >> BK_LOG;
        }
        if (J.b_colfast) {
            c = e & (BN - 1);
            pb = e >> BN_LOG;
        } else {
            pb = e & (BK - 1);
            c = e >> BK_LOG;
        }
        const bool in = e < BM * BK;
        sa_r[q] = r;
        sa_p[q] = p;
        sb_c[q] = c;
        sb_p[q] = pb;
        aoff[q] = (in && row_a[r] >= 0 && p < kc) ? row_a[r] + ak_lo[p] : -1;
        boff[q] = (in && col_b[c] >= 0 && pb < kc) ? col_b[c] + bk_lo[pb] : -1;
    }
    // chunk ch + 1 is loaded into registers while chunk ch is multiplied
    double2 ra[SE], rb[SE];
    auto load = [&]() {
#pragma unroll
        for (int q = 0; q < SE; ++q) {
            ra[q] = aoff[q] >= 0 ? gld(A + (aoff[q] + akh)) : make_double2(0.0, 0.0);
            rb[q] = boff[q] >= 0 ? gld(B + (boff[q] + bkh)) : make_double2(0.0, 0.0);
        }
    };
    auto advance = [&](int64_t ch) {
        const int t = __builtin_ctzll(~(uint64_t)ch);
        if (t < k_log - kc_log) {
            akh += a_step[t];
            bkh += b_step[t];
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int q = 0; q < SE; ++q) {
            if (threadIdx.x + q * 256 >= BM * BK) break;
            As2[buf][sa_p[q]][sa_r[q]] = ra[q];
            Bs2[buf][sb_p[q]][sb_c[q]] = rb[q];
        }
    };
    if (c_begin < c_end) {
        load();
        advance(c_begin);
        stash(0);
        __syncthreads();
    }
    for (int64_t ch = c_begin; ch < c_end; ++ch) {
        const int buf = (int)((ch - c_begin) & 1);
        const double2(*As)[BM + 2] = As2[buf];
        const double2(*Bs)[BN + 2] = Bs2[buf];
        if (ch + 1 < c_end) {
            load();
            advance(ch + 1);
        }
        if constexpr (MF) {
            // lane: A row (lane & 15), B real column (lane & 15) of its block,
            // real inner index lane >> 4 = 2 (complex inner) + kpart
#pragma unroll
            for (int ks = 0; ks < BK / 2; ++ks) {
                const int p = 2 * ks + (lane >> 5);
                double a[WR], b[WC];
#pragma unroll
                for (int i = 0; i < WR; ++i)
                    a[i] = reinterpret_cast<const double*>(&As[p][wr0 + 16 * i + (lane & 15)])[kpart];
#pragma unroll
                for (int j = 0; j < WC; ++j) {
                    const double v =
                        reinterpret_cast<const double*>(&Bs[p][wc0 + 8 * j + ((lane & 15) >> 1)])[tcol ^ kpart];
                    b[j] = (kpart && !tcol) ? -v : v;
                }
#pragma unroll
                for (int i = 0; i < WR; ++i)
#pragma unroll
                    for (int j = 0; j < WC; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[j], acc[i][j], 0, 0, 0);
            }
        } else {
#pragma unroll
            for (int p = 0; p < BK; ++p) {
                double2 a[TT], b[TT];
#pragma unroll
                for (int i = 0; i < TT; ++i) a[i] = As[p][ty + 16 * i];
#pragma unroll
                for (int j = 0; j < TT; ++j) b[j] = Bs[p][tx + 16 * j];
#pragma unroll
                for (int i = 0; i < TT; ++i)
#pragma unroll
                    for (int j = 0; j < TT; ++j) {
                        accr[i][j] += a[i].x * b[j].x - a[i].y * b[j].y;
                        acci[i][j] += a[i].x * b[j].y + a[i].y * b[j].x;
                    }
            }
        }
        // the other buffer was last read before the previous barrier
        if (ch + 1 < c_end) stash(buf ^ 1);
        __syncthreads();
    }
    // split inner sum: this block's part goes to its row-major [BM][BN] partial
    // tile (padding skipped), added to the others' by k_split_reduce
    const bool to_partial = J.ksplit > 1;
    TN_GLOBAL double2* __restrict__ O =
        to_partial ? gstore<double2>(J.partial) + ((int64_t)T.pair * J.ksplit + T.kpart) * (BM * BN) : C;
    if constexpr (MF) {
        // element e of a lane's result is row (lane >> 4) + 4 e of its
        // instruction's block (the FP64 instruction interleaves its rows, unlike
        // the FP32 one), real column lane & 15: complex column (lane & 15) / 2,
        // component tcol
        TN_GLOBAL double* __restrict__ Od = reinterpret_cast<TN_GLOBAL double*>(O);
#pragma unroll
        for (int j = 0; j < WC; ++j) {
            const int col = wc0 + 8 * j + ((lane & 15) >> 1);
            const int64_t cc = col_c[col];
            if (cc < 0) continue;
#pragma unroll
            for (int i = 0; i < WR; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = wr0 + 16 * i + (lane >> 4) + 4 * e;
                    const int64_t rc = row_c[row];
                    if (rc >= 0)
                        Od[2 * (to_partial ? (int64_t)row * BN + col : rc + cc) + tcol] = acc[i][j][e];
                }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TT; ++i) {
        const int row = ty + 16 * i;
        const int64_t rc = row_c[row];
        if (rc < 0) continue;
#pragma unroll
        for (int j = 0; j < TT; ++j) {
            const int col = tx + 16 * j;
            const int64_t cc = col_c[col];
            if (cc >= 0) gst(O + (to_partial ? (int64_t)row * BN + col : rc + cc), make_double2(accr[i][j], acci[i][j]));
        }
    }
}

void launch_tile64_group(int tile, const MfmaJob* d_jobs, const MfmaTile* d_tiles, int64_t n_tiles,
                         hipStream_t s) {
    if (n_tiles == 0) return;
    if (tile == 4)
        launch_k(k_tile64_group<2, TILE64_MFMA>, dim3((unsigned)n_tiles), dim3(256), s, d_jobs, d_tiles);
    else
        launch_k(k_tile64_group<4, TILE64_MFMA>, dim3((unsigned)n_tiles), dim3(256), s, d_jobs, d_tiles);
}

// ---------------------------------------------------------------------------
// Split inner sums: the S blocks of a tile group each wrote one partial tile;
// this launch (same job and tile lists, after the tile launch on the same
// stream, so the partials are complete and visible) adds them in part order
// 0, 1, ..., S-1 and writes C.  Block b takes rows [kpart BM / S, (kpart + 1)
// BM / S) of its group's tile; tiles of unsplit jobs return at once.
// ---------------------------------------------------------------------------
template <typename C2>
__global__ __launch_bounds__(256) void k_split_reduce(const MfmaJob* __restrict__ jobs,
                                                      const MfmaTile* __restrict__ tiles, int bm_log,
                                                      int bn_log) {
    __shared__ int64_t rc_s[128], cc_s[64];
    __shared__ double red_r[256], red_i[256];
    const MfmaTile T = tiles[blockIdx.x];
    const MfmaJob& J = jobs[T.job];
    const int S = J.ksplit;
    if (S <= 1) return;
    const int BM = 1 << bm_log, BN = 1 << bn_log;
    if (S > BM) {
        // more parts than tile rows (very long inner sums): block kpart takes
        // elements [kpart E, (kpart + 1) E) of the row-major tile, E = BM BN / S,
        // its threads add strided subsets of the S partials in FP64 and a fixed
        // tree combines them (deterministic)
        const int64_t E = ((int64_t)BM * BN) / S;
        const int64_t PT = (int64_t)BM * BN;
        const TN_GLOBAL C2* __restrict__ P = gload<C2>(J.partial) + (int64_t)T.pair * S * PT;
        TN_GLOBAL C2* __restrict__ C = gstore<C2>(J.C);
        for (int64_t e = 0; e < E; ++e) {
            const int64_t o = (int64_t)T.kpart * E + e;
            const int i = (int)(o >> bn_log), j = (int)(o & (BN - 1));
            double sr = 0.0, si = 0.0;
            for (int q = threadIdx.x; q < S; q += 256) {
                const C2 v = gld(P + ((int64_t)q * PT + o));
                sr += (double)v.x;
                si += (double)v.y;
            }
            red_r[threadIdx.x] = sr;
            red_i[threadIdx.x] = si;
            __syncthreads();
            for (int w = 128; w > 0; w >>= 1) {
                if ((int)threadIdx.x < w) {
                    red_r[threadIdx.x] += red_r[threadIdx.x + w];
                    red_i[threadIdx.x] += red_i[threadIdx.x + w];
                }
                __syncthreads();
            }
            if (threadIdx.x == 0) {
                const int64_t rc = tile_out_row(J, T, i), cc = tile_out_col(J, T, j);
                if (rc >= 0 && cc >= 0) {
                    C2 t;
                    t.x = red_r[0];
                    t.y = red_i[0];
                    gst(C + (rc + cc), t);
                }
            }
            __syncthreads();
        }
        return;
    }
    const int rows = BM / S, r0 = T.kpart * rows;
    for (int i = threadIdx.x; i < rows; i += 256) rc_s[i] = tile_out_row(J, T, r0 + i);
    for (int j = threadIdx.x; j < BN; j += 256) cc_s[j] = tile_out_col(J, T, j);
    __syncthreads();
    const TN_GLOBAL C2* __restrict__ P = gload<C2>(J.partial) + (int64_t)T.pair * S * (BM * BN);
    TN_GLOBAL C2* __restrict__ C = gstore<C2>(J.C);
    const int64_t PT = (int64_t)BM * BN;
    for (int e = threadIdx.x; e < rows * BN; e += 256) {
        const int i = e >> bn_log, j = e & (BN - 1);
        const int64_t rc = rc_s[i], cc = cc_s[j];
        if (rc < 0 || cc < 0) continue;
        const int64_t o = (int64_t)(r0 + i) * BN + j;
        C2 t = gld(P + o);
        for (int q = 1; q < S; ++q) {
            const C2 v = gld(P + (q * PT + o));
            t.x += v.x;
            t.y += v.y;
        }
        gst(C + (rc + cc), t);
    }
}

void launch_split_reduce(int fp64, int tile, const MfmaJob* d_jobs, const MfmaTile* d_tiles, int64_t n_tiles,
                         hipStream_t s) {
    if (n_tiles == 0) return;
    const int bm_log = __builtin_ctz(mfma_tile_bm(tile)), bn_log = __builtin_ctz(mfma_tile_bn(tile));
    if (fp64)
        launch_k(k_split_reduce<double2>, dim3((unsigned)n_tiles), dim3(256), s, d_jobs, d_tiles, bm_log, bn_log);
    else
        launch_k(k_split_reduce<float2>, dim3((unsigned)n_tiles), dim3(256), s, d_jobs, d_tiles, bm_log, bn_log);
}

// ---------------------------------------------------------------------------
// K2: batched bit permutation, staged through LDS.  A tile covers the lowest
// bits of both the input and the output index (up to 10 bits), so loads run
// along the input's fastest legs and stores along the output's.  The offsets
// inside a tile come from a precomputed table (staged in LDS once per block);
// the remaining (high) bits select the tile, whose base is computed once.
// A block moves kPermElems elements (several tiles when tiles are small).
// Consecutive load slots are consecutive input addresses and consecutive
// store slots consecutive output addresses, so when the tile has at least two
// low bits each thread moves element pairs (16 B for complex64).
// ---------------------------------------------------------------------------
// elements per block: 16 KB of tile data (2048 complex64; the best of a sweep
// over 2^9..2^12 on 2^22-element tensors); at most 256 tiles per block, so the
// whole LDS use (tiles, 12 KB table, bases) stays under 32 KB
template <typename T>
__host__ __device__ constexpr int perm_elems() { return 16384 / (int)sizeof(T); }
__host__ __device__ inline int perm_tiles_per_block(int tsize, int elems) {
    const int u = tsize >= elems ? 1 : elems / tsize;
    return u > 256 ? 256 : u;
}

template <typename T>
__host__ __device__ inline int perm_block_elems(const PermArgs& p) {
    return p.elems_log > 0 ? (1 << p.elems_log) : perm_elems<T>();
}

template <typename T>
__global__ __launch_bounds__(256) void k_permute(PermArgs p) {
    extern __shared__ unsigned char smem_raw[];
    const int tsize = 1 << p.tb;
    const int upb = perm_tiles_per_block(tsize, perm_block_elems<T>(p));  // tiles per block
    // tile elements, one padding element after every 32 (transposes write the
    // tile with a stride of 32 elements)
    T* tile = (T*)smem_raw;                                          // upb * tsize * 33 / 32 elements
    int32_t* tab = (int32_t*)(tile + (int64_t)upb * tsize + ((int64_t)upb * tsize >> 5));  // 3 * tsize
    int64_t* in_base = (int64_t*)(tab + ((3 * tsize + 1) & ~1));     // upb (8-byte aligned)
    int64_t* out_base = in_base + upb;                               // upb
    const int64_t highs = int64_t(1) << p.n_high;
    const int64_t units = p.n_inst * highs;
    const int64_t unit0 = (int64_t)blockIdx.x * upb;
    const int64_t size = int64_t(1) << p.r;
    for (int i = threadIdx.x; i < 3 * tsize; i += blockDim.x) tab[i] = p.table[i];
    for (int u = threadIdx.x; u < upb; u += blockDim.x) {
        const int64_t unit = unit0 + u;
        int64_t ib = 0, ob = 0;
        if (unit < units) {
            const int64_t inst = unit >> p.n_high;
            const int64_t h = unit & (highs - 1);
            for (int i = 0; i < p.n_high; ++i)
                if ((h >> i) & 1) {
                    ib |= int64_t(1) << p.high_in[i];
                    ob |= int64_t(1) << p.high_out[i];
                }
            ib += inst * size;
            ob += inst * size;
        }
        in_base[u] = unit < units ? ib : -1;
        out_base[u] = ob;
    }
    __syncthreads();
    const int32_t* ld_in = tab;
    const int32_t* ld_pos = tab + tsize;
    const int32_t* st_out = tab + 2 * tsize;
    const int total = upb * tsize;
    const T* __restrict__ src = (const T*)p.src;
    T* __restrict__ dst = (T*)p.dst;
    if (p.pair) {
        for (int e2 = threadIdx.x; e2 < total / 2; e2 += blockDim.x) {
            const int e = 2 * e2;
            const int u = e >> p.tb, l = e & (tsize - 1);
            if (in_base[u] < 0) continue;
            const T* s2 = src + in_base[u] + ld_in[l];
            const T a = s2[0], b = s2[1];
            const int t0 = u * tsize + ld_pos[l], t1 = u * tsize + ld_pos[l + 1];
            tile[t0 + (t0 >> 5)] = a;
            tile[t1 + (t1 >> 5)] = b;
        }
    } else {
        for (int e = threadIdx.x; e < total; e += blockDim.x) {
            const int u = e >> p.tb, l = e & (tsize - 1);
            if (in_base[u] < 0) continue;
            const int t0 = u * tsize + ld_pos[l];
            tile[t0 + (t0 >> 5)] = src[in_base[u] + ld_in[l]];
        }
    }
    __syncthreads();
    if (p.pair) {
        for (int e2 = threadIdx.x; e2 < total / 2; e2 += blockDim.x) {
            const int e = 2 * e2;
            const int u = e >> p.tb, l = e & (tsize - 1);
            if (in_base[u] < 0) continue;
            T* d2 = dst + out_base[u] + st_out[l];
            const int t0 = u * tsize + l;
            d2[0] = tile[t0 + (t0 >> 5)];
            d2[1] = tile[t0 + 1 + ((t0 + 1) >> 5)];
        }
    } else {
        for (int e = threadIdx.x; e < total; e += blockDim.x) {
            const int u = e >> p.tb, l = e & (tsize - 1);
            if (in_base[u] < 0) continue;
            const int t0 = u * tsize + l;
            dst[out_base[u] + st_out[l]] = tile[t0 + (t0 >> 5)];
        }
    }
}

// ---------------------------------------------------------------------------
// K3: per-term finalize (FP64): amplitude = scalar * prod of cluster values,
// X = w |amplitude|^2 (a doubled network's value is the amplitude itself:
// X = w Re(amplitude)).
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// K4: Neumaier-compensated level sums in a fixed order (deterministic): each
// thread sums a fixed strided subset, then pairs (sum, comp) are combined in a
// fixed tree.  One block per level.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void neumaier_add(double& s, double& c, double x) {
    const double t = s + x;
    if (fabs(s) >= fabs(x)) c += (s - t) + x;
    else c += (x - t) + s;
    s = t;
}

// (sum, comp) pairs of a block's threads combined in a fixed tree (NT threads,
// NT a power of two); thread 0 gets the block's pair.
template <int NT>
__device__ __forceinline__ void neumaier_block(double& s, double& c, double* ss, double* cc) {
    ss[threadIdx.x] = s;
    cc[threadIdx.x] = c;
    __syncthreads();
    for (int w = NT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            double s1 = ss[threadIdx.x], c1 = cc[threadIdx.x] + cc[threadIdx.x + w];
            neumaier_add(s1, c1, ss[threadIdx.x + w]);
            ss[threadIdx.x] = s1;
            cc[threadIdx.x] = c1;
        }
        __syncthreads();
    }
    s = ss[0];
    c = cc[0];
    __syncthreads();
}

// The same with wave shuffles (a fixed butterfly within each wave of 64 lanes),
// then the waves' pairs added by thread 0 in wave order: one barrier.  Only
// thread 0's pair is the block's.
template <int NT>
__device__ __forceinline__ void neumaier_block_shfl(double& s, double& c, double* ss, double* cc) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double s2 = __shfl_xor(s, off), c2 = __shfl_xor(c, off);
        c += c2;
        neumaier_add(s, c, s2);
    }
    const int w = (int)threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        ss[w] = s;
        cc[w] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double S = ss[0], C = cc[0];
        for (int q = 1; q < NT / 64; ++q) {
            C += cc[q];
            neumaier_add(S, C, ss[q]);
        }
        s = S;
        c = C;
    }
    __syncthreads();
}

// Thread t adds elements b + t, b + t + 256, ... of [b, e) in that order; the
// loads of 8 elements are issued before their adds (the adds form a chain).
__device__ __forceinline__ void level_sum_block(const double* x, const int64_t* starts, double* out, int u) {
    __shared__ double ss[256];
    __shared__ double cc[256];
    const int64_t b = starts[u], e = starts[u + 1];
    double s = 0.0, c = 0.0;
    constexpr int U = 8;
    for (int64_t i0 = b + threadIdx.x; i0 < e; i0 += 256 * U) {
        double v[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int64_t i = i0 + (int64_t)q * 256;
            v[q] = i < e ? x[i] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < U; ++q)
            if (i0 + (int64_t)q * 256 < e) neumaier_add(s, c, v[q]);
    }
    neumaier_block<256>(s, c, ss, cc);
    if (threadIdx.x == 0) {
        out[2 * u] = s + c;
        out[2 * u + 1] = c;
    }
}

__global__ __launch_bounds__(256) void k_level_sum(const double* x, const int64_t* starts, double* out) {
    level_sum_block(x, starts, out, blockIdx.x);
}

// The tail of all packed circuits: 256 terms at a time are finalized
// (X_t = w |a_t|^2 and a_t written to the per-term outputs) and, for every level
// u, the Neumaier pair of their terms of level u is formed by a fixed tree over
// the lanes; a circuit's pairs of level u are then added in block order (again a
// fixed tree): deterministic.  Circuits of up to 8 blocks run in one launch, one
// block per circuit (k_tail_small: 1771 terms in two rounds of four blocks);
// larger ones as k_tail_terms, which leaves the pairs in part[block][u], and
// k_tail_sums.  Both orders are the same, so the sums do not depend on the form.
constexpr int kTailSmallBlocks = 8;

__device__ __forceinline__ int tail_job_of(const TN_CONST TailJob* jobs, int n_jobs, int64_t b) {
    int lo = 0, hi = n_jobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].block0 <= b) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Finalize of one term (FP64): amplitude = scalar * prod of the term's cluster
// values in cluster order, X = w |amplitude|^2 (a doubled network's value is the
// amplitude itself: X = w Re(amplitude)).  The term `zero_term` takes its
// cluster values from the FP64 roots, and its product over the FP32 roots goes
// to the results as a diagnostic.  Each thread loads kFinBatch cluster indices,
// then their values, before multiplying, so a term costs two dependent loads
// per batch; the root addresses are scalar loads.  Returns X (0: not live).
constexpr int kFinBatch = 8;

__device__ __forceinline__ double tail_term(const TN_CONST FinalizeArgs* f, int64_t t, int64_t res_shift) {
    if (t >= f->n_terms) return 0.0;
    const int32_t li = gload<int32_t>(f->live_index)[t];
    if (li < 0) {
        gstore<double>(f->x_out)[t] = 0.0;
        gst(gstore<float2>(f->amp_out) + t, make_float2(0.0f, 0.0f));
        return 0.0;
    }
    const double wt = gload<double>(f->w)[t];
    const bool hi = t == f->zero_term;
    const int ncl = f->n_clusters;
    const TN_GLOBAL int32_t* ri = gload<int32_t>(f->root_idx) + (int64_t)li * ncl;
    const TN_CONST int64_t* rp32 = cload<int64_t>(f->root_ptrs);
    const TN_CONST int64_t* rp64 = cload<int64_t>(f->root64_ptrs);
    double ar = f->scalar_re, ai = f->scalar_im;      // over the FP32 roots
    double hr = ar, hm = ai;                          // over the FP64 roots (zero_term)
    for (int c0 = 0; c0 < ncl; c0 += kFinBatch) {
        int32_t j[kFinBatch];
        float2 v[kFinBatch];
        // loads past the last cluster repeat it (in bounds, not used):
        // unconditional loads are all issued before the first wait
#pragma unroll
        for (int q = 0; q < kFinBatch; ++q) j[q] = ri[c0 + q < ncl ? c0 + q : ncl - 1];
#pragma unroll
        for (int q = 0; q < kFinBatch; ++q)
            v[q] = gld(gload<float2>((const void*)rp32[c0 + q < ncl ? c0 + q : ncl - 1]) + j[q]);
#pragma unroll
        for (int q = 0; q < kFinBatch; ++q)
            if (c0 + q < ncl) {
                const double vr = (double)v[q].x, vi = (double)v[q].y;
                const double nr = ar * vr - ai * vi;
                const double ni = ar * vi + ai * vr;
                ar = nr;
                ai = ni;
            }
        if (hi) {
            double2 w[kFinBatch];
#pragma unroll
            for (int q = 0; q < kFinBatch; ++q)
                w[q] = gld(gload<double2>((const void*)rp64[c0 + q < ncl ? c0 + q : ncl - 1]) + j[q]);
#pragma unroll
            for (int q = 0; q < kFinBatch; ++q)
                if (c0 + q < ncl) {
                    const double nr = hr * w[q].x - hm * w[q].y;
                    const double ni = hr * w[q].y + hm * w[q].x;
                    hr = nr;
                    hm = ni;
                }
        }
    }
    const double pr = hi ? hr : ar, pi = hi ? hm : ai;
    const double x = wt * (f->re_value ? pr : pr * pr + pi * pi);
    gstore<double>(f->x_out)[t] = x;
    gst(gstore<float2>(f->amp_out) + t, make_float2((float)pr, (float)pi));
    if (hi && f->x0_fp32_out) *(double*)((char*)f->x0_fp32_out + res_shift) = wt * (f->re_value ? ar : ar * ar + ai * ai);
    return x;
}

// Neumaier pairs of a wave's terms t (value x), per level, to pairs[u][wave].
struct TailPairs {
    double s[TN_MAX_LEVEL + 1][4], c[TN_MAX_LEVEL + 1][4];
};
__device__ __forceinline__ void tail_wave_pairs(const TN_CONST TailJob* J, int64_t t, double x, int wave,
                                                TailPairs& out) {
    const TN_CONST int64_t* starts = cload<int64_t>(J->starts);
    const int64_t t0 = t & ~int64_t(63);                   // the wave's first term
    for (int u = 0; u < J->n_levels; ++u) {
        const int64_t lb = starts[u], le = starts[u + 1];
        double s = 0.0, c = 0.0;
        if (le > t0 && lb < t0 + 64) {
            s = t >= lb && t < le ? x : 0.0;
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
                const double s2 = __shfl_xor(s, off), c2 = __shfl_xor(c, off);
                c += c2;
                neumaier_add(s, c, s2);
            }
        }
        if ((threadIdx.x & 63) == 0) {
            out.s[u][wave] = s;
            out.c[u][wave] = c;
        }
    }
}
// the four waves' pairs of level u in order
__device__ __forceinline__ void tail_block_pair(const TailPairs& p, int u, double& s, double& c) {
    s = p.s[u][0];
    c = p.c[u][0];
#pragma unroll
    for (int q = 1; q < 4; ++q) {
        c += p.c[u][q];
        neumaier_add(s, c, p.s[u][q]);
    }
}

__global__ __launch_bounds__(256) void k_tail_terms(const TailJob* __restrict__ jobs, int n_jobs,
                                                    double* __restrict__ part, int64_t res_shift) {
    __shared__ TailPairs pairs;
    const int64_t b = blockIdx.x;
    const TN_CONST TailJob* J = cload<TailJob>(jobs) + tail_job_of(cload<TailJob>(jobs), n_jobs, b);
    const int64_t t = (b - J->block0) * 256 + threadIdx.x;
    const double x = tail_term(&J->f, t, res_shift);
    tail_wave_pairs(J, t, x, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), pairs);
    __syncthreads();
    if ((int)threadIdx.x < J->n_levels) {
        double s, c;
        tail_block_pair(pairs, (int)threadIdx.x, s, c);
        double* out = part + b * (2 * (TN_MAX_LEVEL + 1)) + 2 * threadIdx.x;
        out[0] = s;
        out[1] = c;
    }
}

__global__ __launch_bounds__(256) void k_tail_sums(const TailJob* __restrict__ jobs, const double* __restrict__ part,
                                                   int64_t res_shift) {
    __shared__ double ss[256];
    __shared__ double cc[256];
    const TN_CONST TailJob* J = cload<TailJob>(jobs) + blockIdx.x;
    const int u = blockIdx.y;
    if (u >= J->n_levels) return;
    const int64_t nb = (J->f.n_terms + 255) / 256;
    double s = 0.0, c = 0.0;
    for (int64_t q = threadIdx.x; q < nb; q += 256) {
        const double* pr = part + (J->block0 + q) * (2 * (TN_MAX_LEVEL + 1)) + 2 * u;
        neumaier_add(s, c, pr[0]);
        c += pr[1];
    }
    neumaier_block_shfl<256>(s, c, ss, cc);
    if (threadIdx.x == 0) {
        double* sums = (double*)((char*)J->sums + res_shift);
        sums[2 * u] = s + c;
        sums[2 * u + 1] = c;
    }
}

// One block per circuit of at most kTailSmallBlocks blocks of terms: four
// 256-thread groups take a block each, then wave u adds the blocks' pairs of
// level u in the order of k_tail_sums.
__global__ __launch_bounds__(1024) void k_tail_small(const TailJob* __restrict__ jobs, int64_t res_shift) {
    __shared__ TailPairs pairs[kTailSmallBlocks];
    const TN_CONST TailJob* J = cload<TailJob>(jobs) + blockIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nb = (int)((J->f.n_terms + 255) / 256);
    for (int b = wave >> 2; b < nb; b += 4) {
        const int64_t t = (int64_t)b * 256 + (threadIdx.x & 255);
        const double x = tail_term(&J->f, t, res_shift);
        tail_wave_pairs(J, t, x, wave & 3, pairs[b]);
    }
    __syncthreads();
    if (wave >= J->n_levels) return;
    const int lane = (int)threadIdx.x & 63;
    double s = 0.0, c = 0.0;
    if (lane < nb) tail_block_pair(pairs[lane], wave, s, c);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double s2 = __shfl_xor(s, off), c2 = __shfl_xor(c, off);
        c += c2;
        neumaier_add(s, c, s2);
    }
    if (lane == 0) {
        double* sums = (double*)((char*)J->sums + res_shift);
        sums[2 * wave] = s + c;
        sums[2 * wave + 1] = c;
    }
}

__global__ void k_slot_fill(SlotFillArgs a) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n * 8) return;
    const int leaf = i >> 3, w = i & 7;
    const int s = a.noise[leaf];
    const int choice = a.pattern[a.term * a.n_noise + s];
    ((float*)a.dst[leaf])[w] = a.bank[(s * 4 + choice) * 8 + w];
}

__global__ void k_copy_c64(const float2* src, float2* dst, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
static inline unsigned grid1(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

struct TileCfg {
    int bm, bnc;
};
static const TileCfg kTiles[K_MFMA_TILES] = {{128, 64}, {64, 64}, {128, 32}, {64, 32},
                                               {32, 32}, {128, 16}, {64, 16}, {32, 16}};

bool mfma_tile_fits(int tile, const GemmArgs& g) {
    if (tile < 0 || tile >= K_MFMA_TILES) return false;
    if (g.m_log < 5 || (int64_t(1) << g.m_log) < kTiles[tile].bm) return false;
    // 16-column tiles also take n < 16 (zero-padded columns) when the GEMM is
    // long enough in m and k to be worth the matrix cores
    if (kTiles[tile].bnc == 16 && g.n_log < 4) return g.n_log >= 1 && g.m_log >= 7 && g.k_log >= 3;
    return (int64_t(1) << g.n_log) >= kTiles[tile].bnc;
}

int select_gemm(const GemmArgs& g, int fp64, int tile_hint) {
    const int mn_log = g.m_log + g.n_log;
    if (mn_log <= 4 && g.k_log >= 8) return fp64 ? K_SPLITK64 : K_SPLITK32;
    if (fp64) return (g.m_log >= 6 && g.n_log >= 6) ? K_TILED64 : K_SMALL64;
    if (mfma_tile_fits(tile_hint, g)) return tile_hint;
    for (int i = 0; i < K_MFMA_TILES; ++i)
        if (mfma_tile_fits(i, g)) return i;
    return K_SMALL32;
}

const char* kernel_name(int id) {
    static const char* mg[K_MFMA_TILES] = {"k_gemm_mfma_g<128,64>", "k_gemm_mfma_g<64,64>", "k_gemm_mfma_g<128,32>",
                                           "k_gemm_mfma_g<64,32>",  "k_gemm_mfma_g<32,32>", "k_gemm_mfma_g<128,16>",
                                           "k_gemm_mfma_g<64,16>",  "k_gemm_mfma_g<32,16>"};
    if (id >= K_GATHER_BASE && id < K_GATHER_BASE + K_MFMA_TILES) return mg[id - K_GATHER_BASE];
    static const char* mq[K_MFMA_TILES] = {"k_mfma_group<128,64>", "k_mfma_group<64,64>", "k_mfma_group<128,32>",
                                           "k_mfma_group<64,32>",  "k_mfma_group<32,32>", "k_mfma_group<128,16>",
                                           "k_mfma_group<64,16>",  "k_mfma_group<32,16>"};
    if (id >= K_MFMA_GROUP_BASE && id < K_MFMA_GROUP_BASE + K_MFMA_TILES) return mq[id - K_MFMA_GROUP_BASE];
    static const char* mf[K_MFMA_TILES] = {"k_gemm_mfma<128,64>", "k_gemm_mfma<64,64>", "k_gemm_mfma<128,32>",
                                           "k_gemm_mfma<64,32>",  "k_gemm_mfma<32,32>", "k_gemm_mfma<128,16>",
                                           "k_gemm_mfma<64,16>",  "k_gemm_mfma<32,16>"};
    if (id >= 0 && id < K_MFMA_TILES) return mf[id];
    switch (id) {
    case K_SMALL32: return "k_gemm_small<float>";
    case K_SPLITK32: return "k_gemm_splitk<float>";
    case K_SMALL64: return "k_gemm_small<double>";
    case K_SPLITK64: return "k_gemm_splitk<double>";
    case K_TILED64: return "k_gemm_tiled_c128";
    case K_PERM32: return "k_permute<float2>";
    case K_PERM64: return "k_permute<double2>";
    // k_gett_group by the precision of a launch's jobs (one kernel serves all)
    case K_GROUP32: return "k_gett_group<float>";
    case K_GROUP64: return "k_gett_group<double>";
    case K_GROUPMIX: return "k_gett_group<mixed>";
    case K_TILE64_GROUP: return "k_tile64_group";
    case K_SPLIT_REDUCE32: return "k_split_reduce<float>";
    case K_SPLIT_REDUCE64: return "k_split_reduce<double>";
    }
    return "unknown";
}

int kernel_class(int id) {
    if (id >= 0 && id < K_MFMA_TILES) return KC_MFMA;
    if (id >= K_GATHER_BASE && id < K_GATHER_BASE + K_MFMA_TILES) return KC_MFMA;
    if (id == K_SMALL32 || id == K_SMALL64) return KC_SMALL;
    if (id == K_SPLITK32 || id == K_SPLITK64) return KC_SPLITK;
    if (id == K_GROUP32 || id == K_GROUP64 || id == K_GROUPMIX || id == K_TILE64_GROUP ||
        id == K_SPLIT_REDUCE32 || id == K_SPLIT_REDUCE64)
        return KC_GROUP;
    if (id >= K_MFMA_GROUP_BASE && id < K_MFMA_GROUP_BASE + K_MFMA_TILES) return KC_GROUP;
    return KC_TILED;
}

int mfma_tile_bm(int tile) { return kTiles[tile].bm; }
int mfma_tile_bn(int tile) { return kTiles[tile].bnc; }

void launch_mfma_group(int tile, const MfmaJob* d_jobs, const MfmaTile* d_tiles, int64_t n_tiles,
                       hipStream_t s) {
    if (n_tiles == 0) return;
    const TileCfg& t = kTiles[tile];
#define TN_GLAUNCH(BM_, BN_)                                                                  \
    if (t.bm == BM_ && t.bnc == BN_) {                                                         \
        constexpr int nt = MfmaGroupShape<BM_, BN_>::NT;                                      \
        launch_k(k_mfma_group<BM_, BN_>, dim3((unsigned)n_tiles), dim3(nt), s, d_jobs, d_tiles);  \
        return;                                                                                \
    }
    TN_GLAUNCH(128, 64)
    TN_GLAUNCH(64, 64)
    TN_GLAUNCH(128, 32)
    TN_GLAUNCH(64, 32)
    TN_GLAUNCH(32, 32)
    TN_GLAUNCH(128, 16)
    TN_GLAUNCH(64, 16)
    TN_GLAUNCH(32, 16)
#undef TN_GLAUNCH
}

void launch_gett_group(const GettJob* d_jobs, const int32_t* d_block_job, int64_t blocks, hipStream_t s) {
    if (blocks == 0) return;
    launch_k(k_gett_group, dim3((unsigned)blocks), dim3(256), s, d_jobs, d_block_job);
}

void launch_gett_chain(const GettChainPart* d_parts, int n_parts, const GettChainBlock* d_blocks, hipStream_t s) {
    launch_k(k_gett_chain, dim3((unsigned)n_parts), dim3(1024), s, d_parts, d_blocks);
}

static void launch_mfma_tile(const TileCfg& t, const GemmArgs& g, hipStream_t s, bool gather) {
    const int64_t ntiles = std::max<int64_t>(1, (int64_t(1) << g.n_log) / t.bnc);
    const int64_t tiles = ((int64_t(1) << g.m_log) / t.bm) * ntiles;
    const unsigned blocks = (unsigned)(tiles * g.n_inst);
#define TN_LAUNCH(BM_, BN_)                                                                   \
    if (t.bm == BM_ && t.bnc == BN_) {                                                         \
        constexpr int nt = 64 * (BM_ >= 64 ? BM_ / 64 : 1) * (BN_ >= 32 ? BN_ / 32 : 1);       \
        if (gather)                                                                            \
            hipLaunchKernelGGL((k_gemm_mfma_g<BM_, BN_>), dim3(blocks), dim3(nt), 0, s, g);    \
        else                                                                                   \
            hipLaunchKernelGGL((k_gemm_mfma<BM_, BN_>), dim3(blocks), dim3(nt), 0, s, g);      \
        return;                                                                                \
    }
    TN_LAUNCH(128, 64)
    TN_LAUNCH(64, 64)
    TN_LAUNCH(128, 32)
    TN_LAUNCH(64, 32)
    TN_LAUNCH(32, 32)
    TN_LAUNCH(128, 16)
    TN_LAUNCH(64, 16)
    TN_LAUNCH(32, 16)
#undef TN_LAUNCH
}

void launch_gemm_id(int id, const GemmArgs& g, hipStream_t s) {
    const int mn_log = g.m_log + g.n_log;
    const int64_t total = g.n_inst << mn_log;
    if (id >= 0 && id < K_MFMA_TILES) {
        launch_mfma_tile(kTiles[id], g, s, false);
        return;
    }
    if (id >= K_GATHER_BASE && id < K_GATHER_BASE + K_MFMA_TILES) {
        launch_mfma_tile(kTiles[id - K_GATHER_BASE], g, s, true);
        return;
    }
    switch (id) {
    case K_SMALL32:
        hipLaunchKernelGGL((k_gemm_small<float, float2>), dim3(grid1(total, 256)), dim3(256), 0, s, g);
        return;
    case K_SPLITK32:
        hipLaunchKernelGGL((k_gemm_splitk<float, float2>), dim3((unsigned)total), dim3(256), 0, s, g);
        return;
    case K_SMALL64:
        hipLaunchKernelGGL((k_gemm_small<double, double2>), dim3(grid1(total, 256)), dim3(256), 0, s, g);
        return;
    case K_SPLITK64:
        hipLaunchKernelGGL((k_gemm_splitk<double, double2>), dim3((unsigned)total), dim3(256), 0, s, g);
        return;
    case K_TILED64: {
        const int64_t tiles = (int64_t(1) << (g.m_log - 6)) << (g.n_log - 6);
        hipLaunchKernelGGL(k_gemm_tiled_c128, dim3((unsigned)(tiles * g.n_inst)), dim3(256), 0, s, g);
        return;
    }
    }
}

int launch_gemm_c64(const GemmArgs& g, hipStream_t s, int tile_hint) {
    const int id = select_gemm(g, 0, tile_hint);
    launch_gemm_id(id, g, s);
    return id;
}

int launch_gemm_c128(const GemmArgs& g, hipStream_t s) {
    const int id = select_gemm(g, 1, -1);
    launch_gemm_id(id, g, s);
    return id;
}

template <typename T>
static void launch_perm(const PermArgs& p, hipStream_t s) {
    const int tsize = 1 << p.tb;
    const int upb = perm_tiles_per_block(tsize, perm_block_elems<T>(p));
    const int64_t units = p.n_inst << p.n_high;
    const unsigned blocks = (unsigned)((units + upb - 1) / upb);
    const size_t elems = (size_t)upb * tsize;
    const size_t lds = (elems + (elems >> 5)) * sizeof(T) + ((3 * tsize + 1) & ~1) * sizeof(int32_t) +
                       2 * upb * sizeof(int64_t);
    hipLaunchKernelGGL((k_permute<T>), dim3(blocks), dim3(256), lds, s, p);
}

void launch_permute_c64(const PermArgs& p, hipStream_t s) { launch_perm<float2>(p, s); }
void launch_permute_c128(const PermArgs& p, hipStream_t s) { launch_perm<double2>(p, s); }

void launch_level_sum(const double* x, const int64_t* starts, int n_levels, double* out,
                      hipStream_t s) {
    hipLaunchKernelGGL(k_level_sum, dim3(n_levels), dim3(256), 0, s, x, starts, out);
}

int tail_launches(int64_t most_blocks) { return most_blocks <= kTailSmallBlocks ? 1 : 2; }

void launch_tail(const TailJob* d_jobs, int n_jobs, int64_t blocks, int64_t most_blocks, int max_levels,
                 double* d_part, int64_t res_shift, hipStream_t s) {
    if (n_jobs == 0) return;
    if (tail_launches(most_blocks) == 1) {
        hipLaunchKernelGGL(k_tail_small, dim3((unsigned)n_jobs), dim3(1024), 0, s, d_jobs, res_shift);
        return;
    }
    hipLaunchKernelGGL(k_tail_terms, dim3((unsigned)blocks), dim3(256), 0, s, d_jobs, n_jobs, d_part, res_shift);
    hipLaunchKernelGGL(k_tail_sums, dim3((unsigned)n_jobs, (unsigned)max_levels), dim3(256), 0, s, d_jobs,
                       (const double*)d_part, res_shift);
}

void launch_slot_fill(const SlotFillArgs& a, hipStream_t s) {
    if (a.n == 0) return;
    hipLaunchKernelGGL(k_slot_fill, dim3(grid1(a.n * 8, 256)), dim3(256), 0, s, a);
}

void launch_copy_c64(const void* src, void* dst, int64_t n, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_copy_c64, dim3(grid1(n, 256)), dim3(256), 0, s, (const float2*)src,
                       (float2*)dst, n);
}

}  // namespace tn
