// Expert computation: moe_grouped_ffn_fwd and moe_grouped_ffn_bwd.
//
// Every expert is a SwiGLU MLP (paper section 3.1) applied to the rows the gate
// sent to it; the rows of one expert are contiguous after moe_permute and their
// number is whatever the (skewed) routing produced.  All six products are
// "grouped GEMMs": one GEMM per expert whose ragged dimension is the expert's
// row count, either as M (forward, dgrad) or as the contraction length K
// (wgrad).  One kernel template covers them:
//
//   C[m,n] = sum_k A(m,k) * B(k,n)          per expert, fp32 accumulate
//
//   forward 1   [A|B] = Xp_e * [W1_e|W3_e]         -> H = silu(A) (.) B
//   forward 2   Yp_e  = H_e * W2_e
//   dgrad 1     dH    = dYp_e * W2_e^T              -> dA, dB (and H again)
//   dgrad 2     dXp_e = dA_e * W1_e^T + dB_e * W3_e^T      (two K segments)
//   wgrad       dW2_e = H_e^T * dYp_e,  [dW1_e|dW3_e] = Xp_e^T * [dA_e|dB_e]
//
// bf16 path: persistent 256x256x64 kernels, 8 wavefronts, fp32 accumulators, operands brought into LDS by DMA in
// memory order, transposing LDS reads where the contraction index is not the contiguous one: gg_quad_kernel
// (grouped_gemm_quad.h), and gg256_kernel (grouped_gemm_bf16.h) for the gradients of few rows.  A K that is no
// multiple of 64 ends in a stage padded with zeros.  The plain 128x128x64 kernel below is left for leading
// dimensions beyond the 32-bit offsets of these, and for operands of 2^32 elements and more.
// fp32 path: 64x64 tiles on the fp32 matrix instructions (grouped_gemm_f32.h), 128x128 ones for products with many of them
// (grouped_gemm_f32_large.h), 32x32 ones with the contraction split over the wavefronts for products with few
// (grouped_gemm_f32_split.h), same tile walk and epilogues.
#include "moe_internal.h"

namespace moe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

enum { EPI_STORE = 0, EPI_STORE2 = 1, EPI_SWIGLU = 2, EPI_DH = 3, EPI_STORE_F32 = 4, EPI_ADD = 5, EPI_DHP = 6 };

struct Seg {
    const void* A;
    const void* B;
    const void* B2;
};

struct GArgs {
    const int32_t* offsets;  // [E+1] rows of each expert
    int E;
    int M, N, K;           // fixed extents (M unused when M is ragged, K unused when K is ragged)
    int nseg;              // K segments accumulated into one tile
    Seg seg[2];
    int64_t lda, ldb;      // leading dimensions in elements
    int64_t strideB;       // per-expert stride of B (ragged M);
    int64_t strideC;       // per-expert stride of C (ragged K)
    void* C0;
    void* C1;
    void* C2;
    const void* S0;        // saved A (EPI_DH: read; EPI_SWIGLU: written if non-null)
    const void* S1;        // saved B
    int products;          // the saved pair is P = B*silu'(A), Q = silu(A) instead of A, B (EPI_SWIGLU writes it, EPI_DHP reads it)
    int64_t ldc;
    const int32_t* order;  // ragged K: experts by row count, heaviest first (may be null)
    const void* zero_row;  // ragged K: 512 bytes of zeros in device memory
    const int32_t* expert_of_group;  // ragged M: weights of group e are those of expert expert_of_group[e] (null: e itself)
    int n_weights;                   // experts in the weight arrays (the table's entries are clamped to it)
    uint32_t* sched;                 // tile queues of the persistent kernel (kSchedWords words, zero at launch); null: static tile order
};

// index of the weight matrices of group e
__device__ __forceinline__ int weight_index(const GArgs& g, int e) {
    if (!g.expert_of_group) return e;
    const int w = g.expert_of_group[e];
    return w < 0 ? 0 : (w >= g.n_weights ? g.n_weights - 1 : w);
}

template <class T, int EPI>
__device__ __forceinline__ void epilogue_elem(const GArgs& g, int64_t idx, float a, float b) {
    if constexpr (EPI == EPI_STORE_F32) {
        static_cast<float*>(g.C0)[idx] = a;
    } else if constexpr (EPI == EPI_STORE) {
        Elem<T>::store(static_cast<T*>(g.C0) + idx, a);
    } else if constexpr (EPI == EPI_STORE2) {
        Elem<T>::store(static_cast<T*>(g.C0) + idx, a);
        Elem<T>::store(static_cast<T*>(g.C1) + idx, b);
    } else if constexpr (EPI == EPI_SWIGLU) {
        Elem<T>::store(static_cast<T*>(g.C0) + idx, silu_f(a) * b);
        if (g.S0) {
            Elem<T>::store(const_cast<T*>(static_cast<const T*>(g.S0)) + idx, g.products ? b * silu_grad_f(a) : a);
            Elem<T>::store(const_cast<T*>(static_cast<const T*>(g.S1)) + idx, g.products ? silu_f(a) : b);
        }
    } else if constexpr (EPI == EPI_DHP) {  // a = dH; saved P, Q
        const float P = Elem<T>::load(static_cast<const T*>(g.S0) + idx);
        const float Q = Elem<T>::load(static_cast<const T*>(g.S1) + idx);
        Elem<T>::store(static_cast<T*>(g.C1) + idx, a * P);
        Elem<T>::store(static_cast<T*>(g.C2) + idx, a * Q);
    } else {  // EPI_DH: a = dH
        const float A = Elem<T>::load(static_cast<const T*>(g.S0) + idx);
        const float B = Elem<T>::load(static_cast<const T*>(g.S1) + idx);
        const float sA = silu_f(A);
        Elem<T>::store(static_cast<T*>(g.C0) + idx, sA * B);
        Elem<T>::store(static_cast<T*>(g.C1) + idx, a * B * silu_grad_f(A));
        Elem<T>::store(static_cast<T*>(g.C2) + idx, a * sA);
    }
}

// Which expert and which row block does m-tile `mt` (counted over all experts) belong to?
// Returns false if mt is past the last tile.  Uniform across the workgroup.
template <int BM>
__device__ __forceinline__ bool find_m_tile(const int32_t* __restrict__ offsets, int E, int mt, int& e_out,
                                            int& row0, int& row_end) {
    int acc = 0;
    for (int e = 0; e < E; ++e) {
        const int b = offsets[e], en = offsets[e + 1];
        const int nt = (en - b + BM - 1) / BM;
        if (mt < acc + nt) {
            e_out = e;
            row0 = b + (mt - acc) * BM;
            row_end = en;
            return true;
        }
        acc += nt;
    }
    return false;
}

// =============================== bf16 MFMA path ===============================
constexpr int BM = 128, BN = 128, BK = 64, BKP = BK + 8;

// contraction-contiguous source: tile rows [row0, row0+128) x k [k0, k0+64)
__device__ __forceinline__ void ld_kcontig(u32x4 (&r)[4], const bf16_t* __restrict__ base, int64_t ld, int row0,
                                           int row_lim, int k0, int k_lim) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = threadIdx.x + i * 256;
        const int row = row0 + (v >> 3), kk = k0 + (v & 7) * 8;
        if (row < row_lim && kk < k_lim)
            r[i] = *reinterpret_cast<const u32x4*>(base + (int64_t)row * ld + kk);
        else
            r[i] = (u32x4){0, 0, 0, 0};
    }
}
__device__ __forceinline__ void st_kcontig(bf16_t (*dst)[BKP], const u32x4 (&r)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = threadIdx.x + i * 256;
        *reinterpret_cast<u32x4*>(&dst[v >> 3][(v & 7) * 8]) = r[i];
    }
}
// other-index-contiguous source: k rows [k0, k0+64) x cols [col0, col0+128)
__device__ __forceinline__ void ld_strided(u32x4 (&r)[4], const bf16_t* __restrict__ base, int64_t ld, int k0,
                                           int k_lim, int col0, int col_lim) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = threadIdx.x + i * 256;
        const int kk = k0 + (v >> 4), col = col0 + (v & 15) * 8;
        if (kk < k_lim && col < col_lim)
            r[i] = *reinterpret_cast<const u32x4*>(base + (int64_t)kk * ld + col);
        else
            r[i] = (u32x4){0, 0, 0, 0};
    }
}
__device__ __forceinline__ void st_strided(bf16_t (*dst)[BKP], const u32x4 (&r)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int v = threadIdx.x + i * 256;
        const int kk = v >> 4, c = (v & 15) * 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t w = r[i][j];
            dst[c + 2 * j][kk] = (bf16_t)(w & 0xFFFFu);
            dst[c + 2 * j + 1][kk] = (bf16_t)(w >> 16);
        }
    }
}

// AT: 0 = A stored [M][K] (K contiguous), 1 = A stored [K][M]
// BT: 0 = B stored [K][N] (N contiguous), 1 = B stored [N][K]
template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
__global__ __launch_bounds__(256) void gg_bf16_kernel(const GArgs g) {
    __shared__ __attribute__((aligned(16))) bf16_t As[BM][BKP];
    __shared__ __attribute__((aligned(16))) bf16_t Bs[BN][BKP];
    __shared__ __attribute__((aligned(16))) bf16_t Bs2[DUAL ? BN : 1][BKP];

    int e, m0, m_lim, kbeg, kend;
    const int n0 = blockIdx.x * BN;
    if constexpr (RAGK) {
        e = blockIdx.z;
        m0 = blockIdx.y * BM;
        m_lim = g.M;
        kbeg = g.offsets[e];
        kend = g.offsets[e + 1];
    } else {
        if (!find_m_tile<BM>(g.offsets, g.E, blockIdx.y, e, m0, m_lim)) return;
        kbeg = 0;
        kend = g.K;
    }

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

    f32x16 acc[2][2], acc2[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                acc[i][j][r] = 0.f;
                acc2[i][j][r] = 0.f;
            }

    const int nk = (kend - kbeg + BK - 1) / BK;
    const int total = nk * g.nseg;
    u32x4 ra[4], rb[4], rb2[4];

    auto gload = [&](int it) {
        const int sg = it / nk, k0 = kbeg + (it - sg * nk) * BK;
        const bf16_t* A = static_cast<const bf16_t*>(g.seg[sg].A);
        const bf16_t* B = static_cast<const bf16_t*>(g.seg[sg].B) + (RAGK ? 0 : (int64_t)weight_index(g, e) * g.strideB);
        if constexpr (AT == 0) ld_kcontig(ra, A, g.lda, m0, m_lim, k0, kend);
        else ld_strided(ra, A, g.lda, k0, kend, m0, m_lim);
        if constexpr (BT == 1) ld_kcontig(rb, B, g.ldb, n0, g.N, k0, kend);
        else ld_strided(rb, B, g.ldb, k0, kend, n0, g.N);
        if constexpr (DUAL) {
            const bf16_t* B2 = static_cast<const bf16_t*>(g.seg[sg].B2) + (RAGK ? 0 : (int64_t)weight_index(g, e) * g.strideB);
            if constexpr (BT == 1) ld_kcontig(rb2, B2, g.ldb, n0, g.N, k0, kend);
            else ld_strided(rb2, B2, g.ldb, k0, kend, n0, g.N);
        }
    };

    if (total > 0) gload(0);
    for (int it = 0; it < total; ++it) {
        __syncthreads();  // previous tile fully consumed
        if constexpr (AT == 0) st_kcontig(As, ra); else st_strided(As, ra);
        if constexpr (BT == 1) st_kcontig(Bs, rb); else st_strided(Bs, rb);
        if constexpr (DUAL) { if constexpr (BT == 1) st_kcontig(Bs2, rb2); else st_strided(Bs2, rb2); }
        __syncthreads();
        if (it + 1 < total) gload(it + 1);  // next tile's HBM reads overlap the MFMAs below
#pragma unroll
        for (int kk = 0; kk < BK; kk += 16) {
            bf16x8 a[2], b[2], b2[2];
            const int ko = kk + (lane >> 5) * 8;
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8*>(&As[wm + i * 32 + (lane & 31)][ko]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                b[j] = *reinterpret_cast<const bf16x8*>(&Bs[wn + j * 32 + (lane & 31)][ko]);
                if constexpr (DUAL) b2[j] = *reinterpret_cast<const bf16x8*>(&Bs2[wn + j * 32 + (lane & 31)][ko]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
                    if constexpr (DUAL)
                        acc2[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b2[j], acc2[i][j], 0, 0, 0);
                }
        }
    }

    // epilogue: 32x32 accumulator layout: col = lane%32, row = 8*(r/4) + 4*(lane/32) + r%4
    const int64_t cbase = RAGK ? (int64_t)e * g.strideC : 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn + j * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = m0 + wm + i * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                if (row < m_lim && col < g.N)
                    epilogue_elem<bf16_t, EPI>(g, cbase + (int64_t)row * g.ldc + col, acc[i][j][r],
                                               DUAL ? acc2[i][j][r] : 0.f);
            }
        }
}

}  // namespace moe
#include "grouped_gemm_bf16.h"
#include "grouped_gemm_quad.h"
namespace moe {

// Ragged M: the expert e whose tiles hold tile L of the launch, its rows [row0, row_end) and the tile's index among
// the expert's.  False past the last tile.  Every wavefront looks it up by itself: lane l counts the tiles of
// experts 4l .. 4l+3, then a scan over the lanes.
template <int BM>
__device__ __forceinline__ bool find_tile(const GArgs& g, int L, int n_tiles, int& e, int& row0, int& row_end, int& local) {
    const int lane = threadIdx.x & 63;
    int cnt[4], beg[4], end[4], sum = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int x = lane * 4 + u;
        beg[u] = x < g.E ? g.offsets[x] : 0;
        end[u] = x < g.E ? g.offsets[x + 1] : 0;
        cnt[u] = (end[u] - beg[u] + BM - 1) / BM * n_tiles;
        sum += cnt[u];
    }
    int incl = sum;
#pragma unroll
    for (int dlt = 1; dlt < 64; dlt <<= 1) {
        const int o = __shfl_up(incl, dlt, 64);
        if (lane >= dlt) incl += o;
    }
    int run = incl - sum, fe = 0, fl = 0, fb = 0, fn = 0;
    bool mine = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (L >= run && L < run + cnt[u]) {
            mine = true;
            fe = lane * 4 + u;
            fl = L - run;
            fb = beg[u];
            fn = end[u];
        }
        run += cnt[u];
    }
    const uint64_t who = __ballot(mine);
    if (!who) return false;  // (the same in every wavefront)
    const int src = __builtin_ctzll(who);
    e = __builtin_amdgcn_readlane(fe, src);
    local = __builtin_amdgcn_readlane(fl, src);
    row0 = __builtin_amdgcn_readlane(fb, src);
    row_end = __builtin_amdgcn_readlane(fn, src);
    return true;
}

// four consecutive columns of one output row
__device__ __forceinline__ void put4(float* p, const f32x4v v) { *reinterpret_cast<f32x4v*>(p) = v; }
__device__ __forceinline__ void put4(bf16_t* p, const f32x4v v) {
    *reinterpret_cast<u32x2*>(p) = (u32x2){pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
}
__device__ __forceinline__ f32x4v get4(const float* p) { return *reinterpret_cast<const f32x4v*>(p); }
__device__ __forceinline__ f32x4v get4(const bf16_t* p) {
    const u32x2 u = *reinterpret_cast<const u32x2*>(p);
    return (f32x4v){__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xFFFF0000u), __uint_as_float(u[1] << 16),
                    __uint_as_float(u[1] & 0xFFFF0000u)};
}
template <class T, int EPI>
__device__ __forceinline__ void epilogue_x4(const GArgs& g, int64_t idx, const f32x4v a, const f32x4v b) {
    auto to = [&](const void* p) { return static_cast<T*>(const_cast<void*>(p)) + idx; };
    if constexpr (EPI == EPI_STORE) {
        put4(to(g.C0), a);
    } else if constexpr (EPI == EPI_STORE2) {
        put4(to(g.C0), a);
        put4(to(g.C1), b);
    } else if constexpr (EPI == EPI_SWIGLU) {
        f32x4v h, p, q;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const float sA = silu_f(a[z]);
            h[z] = sA * b[z];
            p[z] = g.products ? b[z] * silu_grad_f(a[z]) : a[z];
            q[z] = g.products ? sA : b[z];
        }
        put4(to(g.C0), h);
        if (g.S0) {
            put4(to(g.S0), p);
            put4(to(g.S1), q);
        }
    } else if constexpr (EPI == EPI_DHP) {  // a = dH; saved P, Q
        const f32x4v P = get4(to(g.S0)), Q = get4(to(g.S1));
        f32x4v da, db;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            da[z] = a[z] * P[z];
            db[z] = a[z] * Q[z];
        }
        put4(to(g.C1), da);
        put4(to(g.C2), db);
    } else {
        static_assert(EPI == EPI_DH, "one of the epilogues above");  // a = dH
        const f32x4v A = get4(to(g.S0)), B = get4(to(g.S1));
        f32x4v h, da, db;
#pragma unroll
        for (int z = 0; z < 4; ++z) {
            const float sA = silu_f(A[z]);
            h[z] = sA * B[z];
            da[z] = a[z] * B[z] * silu_grad_f(A[z]);
            db[z] = a[z] * sA;
        }
        put4(to(g.C0), h);
        put4(to(g.C1), da);
        put4(to(g.C2), db);
    }
}

}  // namespace moe
#include "grouped_gemm_few_rows.h"
namespace moe {

}  // namespace moe
#include "grouped_gemm_f32.h"
#include "grouped_gemm_f32_large.h"
#include "grouped_gemm_f32_split.h"
namespace moe {

// =============================== host dispatch ================================
// Few rows per expert: the kernel of grouped_gemm_few_rows.h where it is the faster one.  The rows of each expert are
// known on the device only, so the rule goes by their mean, and by whether gg_quad_kernel's tiles would leave a part (two matrices)
// or half of the chip idle.  Where the lines lie, as whole calls (us, this kernel -> gg_quad_kernel in the products that
// change at the line; even to Zipf-skewed rows):
//   two matrices, 64 experts of 2048 x 1408, forward: mean 16 207 -> 214 (with the second product), 24 222 -> 217, 32 225 -> 219,
//     48 247 -> 228, 64 249 -> 234; training: 48 780 -> 757; 128 of 2048 x 768, forward: 20 260 -> 254, 64 333 -> 284
//   a part of the chip idle (32 of 512 x 768), training: 64 164 -> 167
//   half of it idle in the products that end in d columns (8 of 4096 x 14336), forward: 32 508 -> 583, 48 565 -> 590
//   dgrad, 64 of 2048 x 1408, training: mean 24 731 -> 727, 32 734 -> 735
template <int BT, bool DUAL, int EPI>
static bool launch_few_rows(const GArgs& g, int64_t R, hipStream_t st) {
    auto go = [&](auto kern, int bm, int n_out, int lds) {
        const int64_t tiles = (g.N + n_out - 1) / n_out * (R / bm + (R < g.E ? R : g.E));  // (upper bound)
        ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
        kern<<<(unsigned)((tiles + 63) / 64 * 64), kFewThreads, lds, st>>>(g);
        return true;
    };
    const int64_t n256 = (g.N + (DUAL ? 127 : 255)) / (DUAL ? 128 : 256);
    const bool half_idle = 2 * n256 * g.E <= 256;
    if (R > 64 * (int64_t)g.E) return false;
    const bool to32 = R <= 32 * (int64_t)g.E;
    if constexpr (DUAL) {
        const bool part_idle = n256 * g.E < 256;
        if (R <= 16 * (int64_t)g.E || (part_idle && to32))
            return go(gg_few_rows_kernel<BT, DUAL, EPI, 64, 2, 3>, 64, 64, few_rows_lds<64, 2, 3>());
        if (part_idle) return go(gg_few_rows_kernel<BT, DUAL, EPI, 128, 2, 2>, 128, 64, few_rows_lds<128, 2, 2>());
    } else if constexpr (BT == 0) {
        if (R <= 16 * (int64_t)g.E || (half_idle && to32))
            return go(gg_few_rows_kernel<BT, DUAL, EPI, 64, 2, 3>, 64, 128, few_rows_lds<64, 2, 3>());
        if (half_idle) return go(gg_few_rows_kernel<BT, DUAL, EPI, 128, 2, 3>, 128, 128, few_rows_lds<128, 2, 3>());
    } else {
        if (to32) return go(gg_few_rows_kernel<BT, DUAL, EPI, 64, 1, 3>, 64, 64, few_rows_lds<64, 1, 3>());
        if (half_idle) return go(gg_few_rows_kernel<BT, DUAL, EPI, 128, 1, 3>, 128, 64, few_rows_lds<128, 1, 3>());
    }
    return false;
}

// Whether the weight gradients are stored non-temporally.  Plain stores leave the memory-side cache full of their dirty
// lines, which the kernels after them pay for, and where the products are bound by their output (few rows per
// group) they pay for it themselves.  us, plain and non-temporal, both gradients alone, with the exchange that reads them
// next (reshard of one device's experts), and with the next forward products:
//   64 groups of 2048 x 1408, mean 128 rows: 732, 679; 1106, 1056; 990, 938     mean 512: 1338, 1334; 1722, 1707; 1944, 1898
//   16 of 4096 x 2048, mean 1024: 1572, 1532; 1840, 1813; 2319, 2257            32 of 1024 x 512, 256: 120, 113; 148, 148; 174, 160
//   16 of 1024 x 1408, mean 512 (138 MB, within the cache): 229, 219; 264, 267; 340, 328
// (the backward call as a whole).  With many rows the matrix cores are the bound and the stores make no difference there (8
// groups of 4096 x 14336, mean 4096: 18939, 18920), but after non-temporal ones the update of dx by moe_gate_topk_bwd
// takes 67 us, after plain ones 46.
static bool stream_gradients(int64_t R, int groups) { return R <= 2048 * (int64_t)groups; }

// Whether the products over ragged rows go through the instances of gg_quad_kernel that request the weights of experts with a single
// row tile, and store the outputs, non-temporally.  With few rows per expert the weights are the work: outputs that stay out of
// the caches leave them to the weights that the next kernels read.  The test per tile costs where there are more rows, so it goes
// by the mean.  us, all plain; the weights alone non-temporal; weights and outputs:
//   forward, 64 experts of 2048 x 1408, mean 32: 227, 220, 214   64: 244, 241, 226   128: 282, 281, 268   192: 333, 337, 334
//     256: 387, 393, 391   512: 622, 646, 646
//     32 of 4096 x 2048, 64: 322, 306, 289   128: 365, 367, 353   192: 439, 440, 431   256: 523, 532, 533
//     8 of 4096 x 14336, 128: 644, 658, 641   192: 708, 726, 717
//   training, 64 of 2048 x 1408, 64: 847, 792, 765   128: 977, 962, 937   192: 1200, 1178, 1161   256: 1349, 1339, 1333
//     8 of 4096 x 7168, 128: 1184, 1181, 1170   192: 1309, 1289, 1287   256: 1599, 1606, 1597
//     128 of 2048 x 768, 80: 1040, 1010, 976   128: 1206, 1161, 1132   192: 1400, 1366, 1356
static bool stream_few_rows(int64_t R, int groups) { return R <= 192 * (int64_t)groups; }

// Whether a weight gradient's tiles are too short for gg_quad_kernel, which runs at least two k-stages per tile and fills its
// pipeline first.  A training pass with the gradients on gg256_kernel and on gg_quad_kernel (us; experts of 4096 x 7168 (8),
// 2048 x 1408 (64), 512 x 768 (32)), by mean rows per expert:
//   16: 822, 891; 713, 762    64: 1005, 1057; 885, 892; 190, 191    80: 1139, 1137; 953, 949    96: 1222, 1194; 1050, 1021; 199, 198
//   128: 1278, 1222; 1135, 1102; 203, 204    256: 254, 253 (the smallest)    512: 2183, 2131 (64 experts)    4096: 28203, 27583 (8)
static bool few_rows_per_tile(int64_t R, int groups) { return R < 80 * (int64_t)groups; }

// workgroups of 256 threads for that many tiles, a multiple of 64 of them; a dimension holds fewer than 2^32 threads
static dim3 f32_grid(int64_t tiles) {
    constexpr int64_t kMost = 1 << 23;
    const int64_t blocks = (tiles + 63) / 64 * 64;
    return blocks <= kMost ? dim3((unsigned)blocks) : dim3((unsigned)kMost, (unsigned)((blocks + kMost - 1) / kMost));
}

// number of bm x bm tiles (ragged M: an upper bound) where the rows belong to `groups` groups
template <bool DUAL, bool RAGK>
static int64_t f32_tiles(const GArgs& g, int64_t R, int bm, int groups) {
    const int n_out = DUAL ? bm / 2 : bm;
    const int64_t n = (g.N + n_out - 1) / n_out;
    return n * (RAGK ? (int64_t)((g.M + bm - 1) / bm) * groups : (R + bm - 1) / bm + groups);
}

// Whether a product is one for gg_f32_split_kernel, by the number of 64x64 tiles (ragged M: an upper bound), the mean rows per
// expert and the contraction.  Kernel times over those of gg_f32_kernel in 2x2 blocks, least and most of 4 to 256 experts of 128 x 128
// to 4096 x 1024:
//   more than 16 rows per expert, one matrix, tiles: up to 64 0.33 to 0.90   128 0.31 to 0.73   192 0.32 to 0.97   320 0.59 to 1.40
//     640 0.53 to 1.79 (the shorter the contraction the worse)
//   two matrices: up to 64 0.72 to 0.78   128 0.35 to 0.76   192 0.37 to 0.93   320 0.59 to 1.33.  Contractions of 2048 and more: 192
//     0.37 to 0.63, 256 0.61 and 0.62, 264 0.59 (4 experts with 32 rows), but 320 tiles all of which have rows 53 us -> 58
//   at most 16 rows per expert (a tile of 64 rows would be empty but for a quarter), more tiles than that, rows even and Zipf-skewed:
//     contractions of 128 0.74 to 1.41, of 256 0.58 to 1.15, of 512 and more 0.31 to 1.0 but for 1.11 at one row for each of 256 experts
//     and 1.10 at 16 rows for each of 4.  Where a sixteenth of the experts has all the rows, which the host cannot know, up to 1.8: with few rows
//     most workgroups of a grid made for every expert find no tile, with more the tiles are four times as many for nothing.  Forward passes,
//     64x64 tiles and this: 128 experts of 512 x 1024, 1 row on average 44, 36, 4 rows 53, 54, 16 rows 99, 119; 256 of these 62, 68, 78, 105, 168,
//     235; 128 of 1024 x 768 with 16 rows 133, 149.  (As many workgroups as the chip holds, each taking tile after tile, spares the empty ones: 256 experts
//     35, 77, 210, but 64 experts of 2048 x 1408 with 4 rows each 505 -> 555.)
//   gradients: up to 32 tiles 0.46 to 1.10   64 0.49 to 0.95   128 0.64 to 1.13 (the most: 4.4 us -> 4.9)   256 0.97 to 1.9   more
//     up to 6 (many tiles, few stages each).  dW_g stays there too: 5 -> 5 to 8.
// Its sums are in another order than those of the other fp32 kernels.  So the products over ragged rows count the experts, not the
// replica groups that their rows may be cut into: those must give the same bits.
template <bool DUAL, bool RAGK>
static bool f32_split_tiles(const GArgs& g, int64_t R) {
    const int experts = RAGK ? g.E : g.n_weights;
    const int64_t tiles = f32_tiles<DUAL, RAGK>(g, R, kF32Tile, experts);
    if (RAGK) return tiles <= 128;
    if (R <= 16 * (int64_t)experts && (int64_t)g.K * g.nseg >= 512) return true;
    if (DUAL) return tiles <= 128 || (g.K >= 2048 && tiles <= 320 && f32_tiles<DUAL, RAGK>(g, R, kF32Tile, 0) <= 192);
    return tiles <= 192;
}

template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
static void launch_f32_split(const GArgs& g, int64_t R, hipStream_t st) {
    auto kern = gg_f32_split_kernel<AT, BT, DUAL, EPI, RAGK>;
    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kF32SplitLds);
    kern<<<f32_grid(f32_tiles<DUAL, RAGK>(g, R, kF32SplitTile, g.E)), 256, kF32SplitLds, st>>>(g);
}

static void launch_f32_split_bwd(const GArgs& dx, const GArgs& dw2, const GArgs& dw13, int64_t R, hipStream_t st) {
    auto blocks = [](int64_t tiles) { return (int)((tiles + 63) / 64 * 64); };
    F32SplitBwdArgs a{dx, dw2, dw13, blocks(f32_tiles<false, false>(dx, R, kF32SplitTile, dx.E)), blocks(f32_tiles<false, true>(dw2, R, kF32SplitTile, dw2.E))};
    const int64_t all = (int64_t)a.dx_blocks + a.dw2_blocks + blocks(f32_tiles<true, true>(dw13, R, kF32SplitTile, dw13.E));
    ensure_dynamic_lds(reinterpret_cast<const void*>(&gg_f32_split_bwd_kernel), kF32SplitLds);
    gg_f32_split_bwd_kernel<<<f32_grid(all), 256, kF32SplitLds, st>>>(a);
}

template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
static void launch_f32(const GArgs& g, int64_t tiles, hipStream_t st) {
    auto kern = gg_f32_kernel<AT, BT, DUAL, EPI, RAGK>;
    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kF32Lds);
    kern<<<f32_grid(tiles), 256, kF32Lds, st>>>(g);
}

// Whether a product with B in k-row form is one for 128x128 tiles, by their number (ragged M: an upper bound) and the mean rows per
// expert.  Kernel times, 128x128 over 64x64 tiles:
//   gradients, dW2: 16 to 512 tiles 1.24 to 3.5; 1024 to 1536 0.87 to 1.20, mostly above 1; 2816 and more 0.77 to 0.94
//     dW1|dW3: 32 to 512 1.03 to 3.3; 2040 0.97 to 1.03; 2048 0.87 to 0.95; 2816 to 57344 0.75 to 0.97
//   forward, two matrices, 512 rows per expert and more: 576 to 1152 0.87 to 1.10; 1760 1.00 to 1.04; 2112 to 45408 0.86 to 0.99
//     fewer rows, 2112 to 5376 0.97 to 1.40
//   forward, one matrix, 1000 rows and more: 288 to 2304 0.92 to 1.41; 4128 to 18432 0.93 to 1.00; fewer rows 0.99 to 1.9
// (below 1 under the lines: mostly a single expert; the products with B in row form 0.95 to 2.1, above 1 in 79 of 84).  Whole passes in us, 128x128 tiles from 512 on
// in every product, 64x64 tiles alone, this rule:
//   training, 8 experts of 4096 x 14336, 512 tokens 14153, 12293, 11719; 4096 73790, 75478, 73338; 16384 276856, 293322, 278733
//     128 of 2048 x 768, 16384: 32699, 33754, 32443   16 of 4096 x 7168, 4096: 71890, 74683, 71773   8 of 1024 x 2816, 2048: 2363, 2156, 2132
template <bool DUAL, bool RAGK>
static bool f32_large_tiles(int64_t tiles, int64_t R, int groups) {
    if (RAGK) return tiles >= 2048;
    return DUAL ? tiles >= 2048 && R >= 512 * (int64_t)groups : tiles >= 4096 && R >= 1024 * (int64_t)groups;
}

// A(m,k) layout AT, B(k,n) layout BT as in the bf16 kernel.
template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
static void launch_gg(const moe_shape* s, const GArgs& g, int64_t R, hipStream_t st) {
    if (s->dtype == MOE_BF16) {
        constexpr bool fast_form = RAGK ? (AT == 1 && BT == 0) : (AT == 0);
        if constexpr (fast_form) {
            // The tile kernels keep a lane's offsets from its tile's base in 32 bits: at most 256 rows of a leading dimension
            // below 2^21 (results: 2^22) are below 2^31 bytes.  The bases are in 64 bits, so no offset asks for the bounds on R*lda
            // and N*ldb; operands that large have not been run on the tile kernels.
            const bool ok = g.lda % 8 == 0 && g.ldb % 8 == 0 && g.N >= 8 && g.lda < (1 << 21) && g.ldb < (1 << 21) && g.ldc < (1 << 22) &&
                            (uint64_t)R * (uint64_t)g.lda < (1ull << 32) && (uint64_t)g.N * (uint64_t)g.ldb < (1ull << 32) &&
                            (!RAGK || g.M >= 8);
            if constexpr (!RAGK) {
                if (ok && launch_few_rows<BT, DUAL, EPI>(g, R, st)) return;
                if (ok) {
                    auto kern = g.K % TK ? gg_quad_kernel<BT, DUAL, EPI, true>
                                : stream_few_rows(R, g.E) ? gg_quad_kernel<BT, DUAL, EPI, false, false, true>
                                                         : gg_quad_kernel<BT, DUAL, EPI, false>;
                    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kQuadLds);
                    kern<<<dim3(256), kThreads, kQuadLds, st>>>(g);  // persistent: one workgroup per CU
                    return;
                }
            } else if (ok) {
                auto go = [&](auto kern, int lds) {
                    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), lds);
                    kern<<<dim3(256), kThreads, lds, st>>>(g);
                };
                if (few_rows_per_tile(R, g.E)) go(gg256_kernel<AT, BT, DUAL, EPI, RAGK>, kGemmLds);  // (stores as stream_gradients says)
                else if (stream_gradients(R, g.E)) go(gg_quad_kernel<BT, DUAL, EPI, false, true, true>, kQuadLds);
                else go(gg_quad_kernel<BT, DUAL, EPI, false, true>, kQuadLds);
                return;
            }
        }
        dim3 grid;
        if (RAGK) grid = dim3((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, g.E);
        else grid = dim3((g.N + BN - 1) / BN, (unsigned)((R + BM - 1) / BM + g.E), 1);
        gg_bf16_kernel<AT, BT, DUAL, EPI, RAGK><<<grid, 256, 0, st>>>(g);
    } else {
        if (f32_split_tiles<DUAL, RAGK>(g, R)) {
            launch_f32_split<AT, BT, DUAL, EPI, RAGK>(g, R, st);
            return;
        }
        if constexpr (BT == 0) {
            const int64_t large = f32_tiles<DUAL, RAGK>(g, R, kF32LargeTile, g.E);
            if (f32_large_tiles<DUAL, RAGK>(large, R, g.E)) {
                gg_f32_large_kernel<AT, DUAL, EPI, RAGK><<<f32_grid(large), 256, 0, st>>>(g);
                return;
            }
        }
        launch_f32<AT, BT, DUAL, EPI, RAGK>(g, f32_tiles<DUAL, RAGK>(g, R, kF32Tile, g.E), st);
    }
}

void launch_gate_dwg_gemm(const void* x, const void* dl_hi, const void* dl_lo, const int32_t* chunk_offsets,
                          int nchunks, int d, int n_pad, float* partial, const void* zero_row, hipStream_t st) {
    GArgs g{};
    g.zero_row = zero_row;
    g.offsets = chunk_offsets; g.E = nchunks; g.M = d; g.N = n_pad; g.nseg = 2;
    g.seg[0] = {x, dl_hi, nullptr};
    g.seg[1] = {x, dl_lo, nullptr};
    g.lda = d; g.ldb = n_pad; g.strideC = (int64_t)d * n_pad;
    g.C0 = partial; g.ldc = n_pad;
    auto kern = gg256_kernel<1, 0, false, EPI_STORE_F32, true>;
    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kGemmLds);
    kern<<<dim3(256), kThreads, kGemmLds, st>>>(g);
}

// dW_g of bf16 layers: partial[c][m][n] as in launch_gate_dwg_gemm, n_out columns per row.
//
// What bounds it is reading the tokens, so they are read once (hi and lo meet the same fragments), in tiles of 128 columns of
// x by 64 experts, and there are as many chunks of tokens as it takes to fill the chip.  Four wavefronts of 32 columns each;
// 64-token stages in a ring of two, 32 KB each: x as [64 tokens][256 B] (swz_krow16), hi and lo as [64 tokens][128 B]
// (swz_few_krow), all read transposed.
//
// Measured (us, on 256x256 tiles of gg256_kernel with x read for hi and again for lo, 512 tokens a chunk -> this): 16384 tokens
// of 4096 over 8 experts 85 -> 37 (3.7 TB/s), of 2048 over 128 57 -> 35, 4099 of 1096 over 24 38 -> 9, 4096 of 512 over 32
// 33 -> 5.
constexpr int kDwgM = 128, kDwgN = 64, kDwgStage = 64 * kDwgM * 2 + 2 * 64 * kDwgN * 2, kDwgStages = 2;
constexpr int kDwgLds = kDwgStages * kDwgStage;
__global__ __launch_bounds__(256) void gate_dwg_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ hi,
                                                       const bf16_t* __restrict__ lo, const int32_t* __restrict__ chunk_offsets,
                                                       int d, int n_pad, int n_out, float* __restrict__ partial) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int m0 = blockIdx.x * kDwgM, n0 = blockIdx.y * kDwgN, c = blockIdx.z;
    const int t0 = chunk_offsets[c], tokens = chunk_offsets[c + 1] - t0, total = (tokens + 63) / 64;
    const int nb = min(kDwgN, n_out - n0) / 16;  // blocks of 16 experts
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_AS char*)smem);
    const char* zeros = reinterpret_cast<const char*>(kZeroRow) + (lane & 31) * 16;
    // this wavefront's DMA chunks: 4 of x (4 tokens each), 2 of hi and 2 of lo (8 tokens each)
    const char *xa[4], *ha[2], *la[2];
    int xq[4], hq[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        xq[i] = (wave * 4 + i) * 4 + (lane >> 4);
        const int col = min(m0 + ((lane & 15) ^ swz_krow16(xq[i])) * 8, d - 8);  // (columns past the end: any; not stored)
        xa[i] = reinterpret_cast<const char*>(x + (int64_t)(t0 + xq[i]) * d + col);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        hq[i] = (wave * 2 + i) * 8 + (lane >> 3);
        const int64_t off = (int64_t)(t0 + hq[i]) * n_pad + n0 + ((lane & 7) ^ swz_few_krow(hq[i])) * 8;
        ha[i] = reinterpret_cast<const char*>(hi + off);
        la[i] = reinterpret_cast<const char*>(lo + off);
    }
    auto issue = [&](int it) {
        const uint32_t st = lds_base + (it & 1) * kDwgStage;
        const int left = tokens - it * 64;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            dma16(xq[i] < left ? xa[i] : zeros, st + (wave * 4 + i) * 1024);
            xa[i] += (int64_t)64 * d * 2;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dma16(hq[i] < left ? ha[i] : zeros, st + 16384 + (wave * 2 + i) * 1024);
            dma16(hq[i] < left ? la[i] : zeros, st + 24576 + (wave * 2 + i) * 1024);
            ha[i] += (int64_t)64 * n_pad * 2;
            la[i] += (int64_t)64 * n_pad * 2;
        }
    };
    const int l16 = lane & 15, kg = lane >> 4, q = kg * 8 + (l16 >> 2), half = (l16 & 3) >> 1;
    auto pair = [](const char* p, int step) -> bf16x8 {
        const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)p);
        const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p + step));
        return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    f32x4v acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    if (total > 0) issue(0);
    for (int it = 0; it < total; ++it) {
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (it + 1 < total) issue(it + 1);
        const char* s = smem + (it & 1) * kDwgStage;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 a[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                a[i] = pair(s + (ks * 32 + q) * 256 + (((wave * 4 + i * 2 + half) ^ swz_krow16(q)) << 4) + (l16 & 1) * 8, 1024);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (j >= nb) break;
                const char* p = s + 16384 + (ks * 32 + q) * 128 + (((j * 2 + half) ^ swz_few_krow(q)) << 4) + (l16 & 1) * 8;
                const bf16x8 h = pair(p, 512), l = pair(p + 8192, 512);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(h, a[i], acc[i][j], 0, 0, 0);
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, a[i], acc[i][j], 0, 0, 0);
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + wave * 32 + i * 16 + l16;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j < nb && m < d) *reinterpret_cast<f32x4v*>(partial + ((int64_t)c * d + m) * n_out + n0 + j * 16 + kg * 4) = acc[i][j];
    }
}

void launch_gate_dwg(const void* x, const void* dl_hi, const void* dl_lo, const int32_t* chunk_offsets, int nchunks, int d,
                     int n_pad, int n_out, float* partial, hipStream_t st) {
    ensure_dynamic_lds(reinterpret_cast<const void*>(&gate_dwg_kernel), kDwgLds);
    gate_dwg_kernel<<<dim3((d + kDwgM - 1) / kDwgM, (n_out + kDwgN - 1) / kDwgN, nchunks), 256, kDwgLds, st>>>(
        static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(dl_hi), static_cast<const bf16_t*>(dl_lo), chunk_offsets, d,
        n_pad, n_out, partial);
}

void launch_gate_dwg_gemm_f32(const void* x, const void* dl, const int32_t* chunk_offsets, int nchunks, int d, int n_pad,
                              float* partial, hipStream_t st) {
    GArgs g{};
    g.offsets = chunk_offsets; g.E = nchunks; g.M = d; g.N = n_pad; g.nseg = 1;
    g.seg[0] = {x, dl, nullptr};
    g.lda = d; g.ldb = n_pad; g.strideC = (int64_t)d * n_pad;
    g.C0 = partial; g.ldc = n_pad;
    const int64_t tiles = (int64_t)((n_pad + 63) / 64) * ((d + 63) / 64) * nchunks;
    launch_f32<1, 0, false, EPI_STORE, true>(g, tiles, st);
}

void launch_gate_dx_gemm(const void* dl_hi, const void* dl_lo, const void* wg_pad, const int32_t* whole, int d, int n_pad,
                         void* dx, hipStream_t st) {
    GArgs g{};
    g.offsets = whole; g.E = 1; g.N = d; g.K = n_pad; g.nseg = 2;
    g.seg[0] = {dl_hi, wg_pad, nullptr};
    g.seg[1] = {dl_lo, wg_pad, nullptr};
    g.lda = n_pad; g.ldb = n_pad; g.strideB = 0;
    g.C0 = dx; g.ldc = d;
    auto kern = gg256_kernel<0, 1, false, EPI_ADD, false>;
    ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kGemmLds);
    kern<<<dim3(256), kThreads, kGemmLds, st>>>(g);
}

// Tile queues: the two wgrad launches draw their tiles (a tile costs as much as its expert has rows, so a
// fixed deal leaves workgroups idle at the end: 2-4 % of the backward pass on the skewed workloads); the
// kernels with ragged M keep the fixed order, where drawing measured no gain.
constexpr size_t kSchedBytes = kSchedWords * sizeof(uint32_t);  // tile queues of one GEMM launch
constexpr int kBwdLaunches = 2;

size_t ffn_fwd_workspace_bytes(const moe_shape* s) {
    return align_up((size_t)s->T * s->k * s->f * el_size(s), 256);  // H
}
size_t ffn_bwd_workspace_bytes(const moe_shape* s) {
    // H, dA, dB, (A, B when recomputing), expert order, a row of zeros, tile queues
    return 5 * align_up((size_t)s->T * s->k * s->f * el_size(s), 256) + 2048 + kBwdLaunches * kSchedBytes;
}


}  // namespace moe

using namespace moe;

// groups: number of row groups described by offsets (the experts themselves, or replica groups whose weights
// are those of expert expert_of_group[g])
static void run_fwd1(const moe_shape* s, const void* x_perm, const int32_t* offsets, const void* w1, const void* w3,
                     void* H, void* a_save, void* b_save, hipStream_t st, int groups = 0,
                     const int32_t* expert_of_group = nullptr, bool products = false) {
    GArgs g{};
    g.offsets = offsets; g.E = groups ? groups : s->E; g.N = s->f; g.K = s->d; g.nseg = 1;
    g.expert_of_group = expert_of_group; g.n_weights = s->E;
    g.seg[0] = {x_perm, w1, w3};
    g.lda = s->d; g.ldb = s->f; g.strideB = (int64_t)s->d * s->f;
    g.C0 = H; g.S0 = a_save; g.S1 = b_save; g.ldc = s->f; g.products = products ? 1 : 0;
    launch_gg<0, 0, true, EPI_SWIGLU, false>(s, g, (int64_t)s->T * s->k, st);
}

static moe_status ffn_fwd_impl(const char* who, const moe_shape* s, int groups, const int32_t* expert_of_group,
                               const void* x_perm, const int32_t* offsets, const void* w1, const void* w3,
                               const void* w2, void* y_perm, void* a_save, void* b_save, void* ws, size_t ws_bytes,
                               void* stream, void* h_save = nullptr) {
    // h_save: the products form (H is kept, the saved pair is P = B*silu'(A), Q = silu(A)); no workspace then
    MOE_RETURN_IF(check_shape(s, who));
    MOE_RETURN_IF(check_ptr(x_perm, "x_perm", who));
    MOE_RETURN_IF(check_ptr(offsets, "offsets", who));
    MOE_RETURN_IF(check_ptr(w1, "w1", who));
    MOE_RETURN_IF(check_ptr(w3, "w3", who));
    MOE_RETURN_IF(check_ptr(w2, "w2", who));
    MOE_RETURN_IF(check_ptr(y_perm, "y_perm", who));
    MOE_RETURN_IF(check_ptr(a_save, "a_save", who, true));
    MOE_RETURN_IF(check_ptr(b_save, "b_save", who, true));
    if (!h_save) MOE_RETURN_IF(check_ptr(ws, "ws", who));
    if ((a_save == nullptr) != (b_save == nullptr)) {
        set_error("%s: a_save and b_save must both be given or both be NULL", who);
        return MOE_ERR_INVALID_ARG;
    }
    MOE_RETURN_IF(check_device(who));
    if (!h_save && ws_bytes < ffn_fwd_workspace_bytes(s)) {
        set_error("%s: workspace %zu < %zu bytes", who, ws_bytes, ffn_fwd_workspace_bytes(s));
        return MOE_ERR_WORKSPACE_TOO_SMALL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t R = (int64_t)s->T * s->k;
    void* H = h_save ? h_save : ws;
    run_fwd1(s, x_perm, offsets, w1, w3, H, a_save, b_save, st, groups, expert_of_group, h_save != nullptr);
    GArgs g{};
    g.offsets = offsets; g.E = groups; g.N = s->d; g.K = s->f; g.nseg = 1;
    g.expert_of_group = expert_of_group; g.n_weights = s->E;
    g.seg[0] = {H, w2, nullptr};
    g.lda = s->f; g.ldb = s->d; g.strideB = (int64_t)s->f * s->d;
    g.C0 = y_perm; g.ldc = s->d;
    launch_gg<0, 0, false, EPI_STORE, false>(s, g, R, st);
    return launch_status(who);
}

extern "C" moe_status moe_grouped_ffn_fwd(const moe_shape* s, const void* x_perm, const int32_t* offsets,
                                          const void* w1, const void* w3, const void* w2, void* y_perm, void* a_save,
                                          void* b_save, void* ws, size_t ws_bytes, void* stream) {
    return ffn_fwd_impl("moe_grouped_ffn_fwd", s, s ? s->E : 0, nullptr, x_perm, offsets, w1, w3, w2, y_perm, a_save,
                        b_save, ws, ws_bytes, stream);
}

extern "C" moe_status moe_grouped_ffn_fwd_groups(const moe_shape* s, int32_t G, const int32_t* expert_of_group,
                                                 const void* x_perm, const int32_t* group_offsets, const void* w1,
                                                 const void* w3, const void* w2, void* y_perm, void* a_save,
                                                 void* b_save, void* ws, size_t ws_bytes, void* stream) {
    const char* who = "moe_grouped_ffn_fwd_groups";
    if (G < 1 || G > MOE_MAX_EXPERTS) {
        set_error("%s: G=%d must be in [1, %d]", who, G, MOE_MAX_EXPERTS);
        return MOE_ERR_INVALID_ARG;
    }
    MOE_RETURN_IF(check_ptr(expert_of_group, "expert_of_group", who));
    return ffn_fwd_impl(who, s, G, expert_of_group, x_perm, group_offsets, w1, w3, w2, y_perm, a_save, b_save, ws,
                        ws_bytes, stream);
}

// groups / expert_of_group as in ffn_fwd_impl; the weight gradients are written per group
static moe_status ffn_bwd_impl(const char* who, const moe_shape* s, int groups, const int32_t* expert_of_group,
                               const void* x_perm, const int32_t* offsets, const void* w1, const void* w3,
                               const void* w2, const void* a_save, const void* b_save, const void* dy_perm,
                               void* dx_perm, void* dw1, void* dw3, void* dw2, void* ws, size_t ws_bytes,
                               void* stream, const void* h_save = nullptr) {
    MOE_RETURN_IF(check_shape(s, who));
    MOE_RETURN_IF(check_ptr(x_perm, "x_perm", who));
    MOE_RETURN_IF(check_ptr(offsets, "offsets", who));
    MOE_RETURN_IF(check_ptr(w1, "w1", who));
    MOE_RETURN_IF(check_ptr(w3, "w3", who));
    MOE_RETURN_IF(check_ptr(w2, "w2", who));
    MOE_RETURN_IF(check_ptr(a_save, "a_save", who, true));
    MOE_RETURN_IF(check_ptr(b_save, "b_save", who, true));
    MOE_RETURN_IF(check_ptr(dy_perm, "dy_perm", who));
    MOE_RETURN_IF(check_ptr(dx_perm, "dx_perm", who));
    MOE_RETURN_IF(check_ptr(dw1, "dw1", who));
    MOE_RETURN_IF(check_ptr(dw3, "dw3", who));
    MOE_RETURN_IF(check_ptr(dw2, "dw2", who));
    MOE_RETURN_IF(check_ptr(ws, "ws", who));
    if (h_save && (!a_save || !b_save)) {
        set_error("%s: the products form needs h_save, p_save and q_save", who);
        return MOE_ERR_INVALID_ARG;
    }
    MOE_RETURN_IF(check_device(who));
    if (ws_bytes < ffn_bwd_workspace_bytes(s)) {
        set_error("%s: workspace %zu < %zu bytes", who, ws_bytes, ffn_bwd_workspace_bytes(s));
        return MOE_ERR_WORKSPACE_TOO_SMALL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t R = (int64_t)s->T * s->k;
    const size_t rf = (size_t)R * s->f * el_size(s);
    Carver cv(ws);
    void* H = cv.take(rf);  // (not used in the products form, which reads h_save)
    void* dA = cv.take(rf);
    void* dB = cv.take(rf);
    if (!a_save || !b_save) {  // expert-only recomputation: rebuild A and B (H is rewritten below anyway)
        void* A = cv.take(rf);
        void* B = cv.take(rf);
        run_fwd1(s, x_perm, offsets, w1, w3, H, A, B, st, groups, expert_of_group);
        a_save = A;
        b_save = B;
    }
    {  // dH = dYp * W2^T, then the SwiGLU derivative in the epilogue
        GArgs g{};
        g.offsets = offsets; g.E = groups; g.N = s->f; g.K = s->d; g.nseg = 1;
        g.expert_of_group = expert_of_group; g.n_weights = s->E;
        g.seg[0] = {dy_perm, w2, nullptr};
        g.lda = s->d; g.ldb = s->d; g.strideB = (int64_t)s->f * s->d;
        g.C0 = H; g.C1 = dA; g.C2 = dB; g.S0 = a_save; g.S1 = b_save; g.ldc = s->f;
        if (h_save) launch_gg<0, 1, false, EPI_DHP, false>(s, g, R, st);  // dA = dH*P, dB = dH*Q
        else launch_gg<0, 1, false, EPI_DH, false>(s, g, R, st);
    }
    GArgs gx{};  // dXp = dA * W1^T + dB * W3^T
    gx.offsets = offsets; gx.E = groups; gx.N = s->d; gx.K = s->f; gx.nseg = 2;
    gx.expert_of_group = expert_of_group; gx.n_weights = s->E;
    gx.seg[0] = {dA, w1, nullptr};
    gx.seg[1] = {dB, w3, nullptr};
    gx.lda = s->f; gx.ldb = s->f; gx.strideB = (int64_t)s->d * s->f;
    gx.C0 = dx_perm; gx.ldc = s->d;
    GArgs g2{};  // dW2[e] = H_e^T * dYp_e
    g2.offsets = offsets; g2.E = groups; g2.M = s->f; g2.N = s->d; g2.nseg = 1;
    g2.seg[0] = {h_save ? h_save : H, dy_perm, nullptr};
    g2.lda = s->f; g2.ldb = s->d; g2.strideC = (int64_t)s->f * s->d;
    g2.C0 = dw2; g2.ldc = s->d;
    GArgs g13{};  // [dW1|dW3][e] = Xp_e^T * [dA_e|dB_e]
    g13.offsets = offsets; g13.E = groups; g13.M = s->d; g13.N = s->f; g13.nseg = 1;
    g13.seg[0] = {x_perm, dA, dB};
    g13.lda = s->d; g13.ldb = s->f; g13.strideC = (int64_t)s->d * s->f;
    g13.C0 = dw1; g13.C1 = dw3; g13.ldc = s->f;
    if (s->dtype == MOE_F32 && f32_split_tiles<false, false>(gx, R) && f32_split_tiles<false, true>(g2, R) &&
        f32_split_tiles<true, true>(g13, R)) {
        // (neither the experts' order nor the tile queues: the tiles are few enough to run all at once)
        launch_f32_split_bwd(gx, g2, g13, R, st);
        return launch_status(who);
    }
    launch_gg<0, 1, false, EPI_STORE, false>(s, gx, R, st);
    int32_t* order = static_cast<int32_t*>(cv.take(1024));
    void* zero_row = cv.take(512);
    uint32_t* sched = static_cast<uint32_t*>(cv.take(kBwdLaunches * kSchedBytes));
    expert_order_kernel<<<1, 256, 0, st>>>(offsets, groups, order, static_cast<uint32_t*>(zero_row), sched,
                                           kBwdLaunches * kSchedWords);
    g2.order = g13.order = order;
    g2.zero_row = g13.zero_row = zero_row;
    g2.sched = sched;
    g13.sched = sched + kSchedWords;
    launch_gg<1, 0, false, EPI_STORE, true>(s, g2, R, st);
    launch_gg<1, 0, true, EPI_STORE2, true>(s, g13, R, st);
    return launch_status(who);
}


extern "C" moe_status moe_grouped_ffn_bwd(const moe_shape* s, const void* x_perm, const int32_t* offsets,
                                          const void* w1, const void* w3, const void* w2, const void* a_save,
                                          const void* b_save, const void* dy_perm, void* dx_perm, void* dw1, void* dw3,
                                          void* dw2, void* ws, size_t ws_bytes, void* stream) {
    return ffn_bwd_impl("moe_grouped_ffn_bwd", s, s ? s->E : 0, nullptr, x_perm, offsets, w1, w3, w2, a_save, b_save,
                        dy_perm, dx_perm, dw1, dw3, dw2, ws, ws_bytes, stream);
}

extern "C" moe_status moe_grouped_ffn_fwd_products(const moe_shape* s, const void* x_perm, const int32_t* offsets,
                                                   const void* w1, const void* w3, const void* w2, void* y_perm,
                                                   void* h_save, void* p_save, void* q_save, void* stream) {
    const char* who = "moe_grouped_ffn_fwd_products";
    MOE_RETURN_IF(check_ptr(h_save, "h_save", who));
    MOE_RETURN_IF(check_ptr(p_save, "p_save", who));
    MOE_RETURN_IF(check_ptr(q_save, "q_save", who));
    return ffn_fwd_impl(who, s, s ? s->E : 0, nullptr, x_perm, offsets, w1, w3, w2, y_perm, p_save, q_save, nullptr, 0,
                        stream, h_save);
}

extern "C" moe_status moe_grouped_ffn_bwd_products(const moe_shape* s, const void* x_perm, const int32_t* offsets,
                                                   const void* w1, const void* w3, const void* w2, const void* h_save,
                                                   const void* p_save, const void* q_save, const void* dy_perm,
                                                   void* dx_perm, void* dw1, void* dw3, void* dw2, void* ws,
                                                   size_t ws_bytes, void* stream) {
    const char* who = "moe_grouped_ffn_bwd_products";
    MOE_RETURN_IF(check_ptr(h_save, "h_save", who));
    MOE_RETURN_IF(check_ptr(p_save, "p_save", who));
    MOE_RETURN_IF(check_ptr(q_save, "q_save", who));
    return ffn_bwd_impl(who, s, s ? s->E : 0, nullptr, x_perm, offsets, w1, w3, w2, p_save, q_save, dy_perm, dx_perm,
                        dw1, dw3, dw2, ws, ws_bytes, stream, h_save);
}

extern "C" moe_status moe_grouped_ffn_bwd_groups(const moe_shape* s, int32_t G, const int32_t* expert_of_group,
                                                 const void* x_perm, const int32_t* group_offsets, const void* w1,
                                                 const void* w3, const void* w2, const void* a_save,
                                                 const void* b_save, const void* dy_perm, void* dx_perm,
                                                 void* dw1_groups, void* dw3_groups, void* dw2_groups, void* ws,
                                                 size_t ws_bytes, void* stream) {
    const char* who = "moe_grouped_ffn_bwd_groups";
    if (G < 1 || G > MOE_MAX_EXPERTS) {
        set_error("%s: G=%d must be in [1, %d]", who, G, MOE_MAX_EXPERTS);
        return MOE_ERR_INVALID_ARG;
    }
    MOE_RETURN_IF(check_ptr(expert_of_group, "expert_of_group", who));
    return ffn_bwd_impl(who, s, G, expert_of_group, x_perm, group_offsets, w1, w3, w2, a_save, b_save, dy_perm, dx_perm,
                        dw1_groups, dw3_groups, dw2_groups, ws, ws_bytes, stream);
}
