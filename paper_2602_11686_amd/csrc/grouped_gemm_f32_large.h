// Grouped fp32 GEMM in tiles of 128 x 128, for products with many of them: what the 64 x 64 tiles of grouped_gemm_f32.h lose to
// reading every operand twice as often counts there, and their better filled last round does not.  Operands in k-row form on the
// B side (forward products and weight gradients), one segment; tile walk and epilogues as in the other kernels.
//
// Bound by the matrix pipe: a stage of 16 contraction indices keeps a SIMD busy for 2048 clocks, so a plain double buffer in LDS,
// staged through registers, hides its loads.  Four wavefronts of 64 x 64, in 16 x 16 blocks of v_mfma_f32_16x16x4.
//
// LDS: an operand whose contraction index is contiguous in memory is kept as [row][16 + 4 pad]; a lane reads its
// row's four values k = 4*(lane/16) .. +3 with one ds_read_b128 (16 rows at a stride of 5 pieces: no conflict)
// and the four MFMAs of a stage take one of them each, so MFMA i contracts k = i, 4+i, 8+i, 12+i: the sums are those of the 64 x 64
// kernel, bit for bit.  An operand whose other index is contiguous is kept as [k][128 + 4]; the same four values are four
// ds_read_b32, whose lane groups start 16 banks apart (4*(128 + 4) mod 64 == 16).
//
// Measured beside the rule that takes it (f32_large_tiles): gradients 3 to 25 %, forward products of large batches 1 to 14 %.
#pragma once

namespace moe {

constexpr int kF32LargeTile = 128;

template <int FORM>  // 0: [row][k], k contiguous in memory; 1: [k][row]
struct F32Large {
    static constexpr int BM = kF32LargeTile;
    static constexpr int kK = 16;                               // contraction indices per stage
    static constexpr int kLd = FORM == 0 ? kK + 4 : BM + 4;
    static constexpr int kFloats = FORM == 0 ? BM * kLd : kK * kLd;
    static constexpr int kPieces = BM * kK / 4 / 256;           // 16-byte pieces per thread and stage
    // This thread's pieces of a stage: addresses at k = k0 of the operand's rows r0 .. (rows past r_lim: any valid one,
    // masked at the store) and the k inside the stage.  `split`: tile rows from BM/2 on come from base2.
    const float* at[kPieces];
    int kk[kPieces];
    int64_t step;  // floats from one stage to the next
    __device__ __forceinline__ void set(const float* base, const float* base2, bool split, int64_t ld, int r0, int r_lim, int k0) {
        step = FORM == 0 ? kK : kK * ld;
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int p = threadIdx.x + i * 256;
            int r = FORM == 0 ? p / (kK / 4) : (p % (BM / 4)) * 4;
            kk[i] = FORM == 0 ? (p % (kK / 4)) * 4 : p / (BM / 4);
            const bool second = split && r >= BM / 2;
            r = min(r0 + r - (second ? BM / 2 : 0), FORM == 0 ? r_lim - 1 : r_lim - 4);
            at[i] = (second ? base2 : base) + (FORM == 0 ? (int64_t)r * ld + k0 + kk[i] : (int64_t)(k0 + kk[i]) * ld + r);
        }
    }
    // the next stage, of which `left` contraction indices exist; the others read zeros (leading dimensions and extents
    // are multiples of four: a piece is inside or outside as a whole)
    __device__ __forceinline__ void load(f32x4v (&v)[kPieces], int left) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            v[i] = *reinterpret_cast<const f32x4v*>(kk[i] < left ? at[i] : reinterpret_cast<const float*>(kZeroRow));
            at[i] += step;
        }
    }
    static __device__ __forceinline__ void store(float* s, const f32x4v (&v)[kPieces]) {
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int p = threadIdx.x + i * 256;
            const int off = FORM == 0 ? p / (kK / 4) * kLd + p % (kK / 4) * 4 : p / (BM / 4) * kLd + p % (BM / 4) * 4;
            *reinterpret_cast<f32x4v*>(s + off) = v[i];
        }
    }
    // the values of tile row `row` (a lane's own) at k = 4*kg .. 4*kg+3
    static __device__ __forceinline__ f32x4v frag(const float* s, int row, int kg) {
        if constexpr (FORM == 0) return *reinterpret_cast<const f32x4v*>(s + row * kLd + kg * 4);
        f32x4v v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = s[(kg * 4 + i) * kLd + row];
        return v;
    }
};

template <int AT, bool DUAL, int EPI, bool RAGK>
__global__ __launch_bounds__(256) void gg_f32_large_kernel(const GArgs g) {
    using TA = F32Large<AT>;
    using TB = F32Large<1>;
    constexpr int BM = kF32LargeTile;
    constexpr int NB = BM / 32;          // 16x16 blocks per wavefront along each side
    constexpr int kK = TA::kK;
    __shared__ __attribute__((aligned(16))) float sA[2][TA::kFloats], sB[2][TB::kFloats];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n_out = DUAL ? BM / 2 : BM;
    const int n_tiles = (g.N + n_out - 1) / n_out;

    // ---- which tile: chunks of eight neighbouring tiles go to the XCDs in turn (the grid is a multiple of 64) ----
    // (a second grid dimension where one cannot hold the tiles: f32_grid)
    const int b0 = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    const int L = (((b0 >> 6) * 8 + (b0 & 7)) << 3) + ((b0 >> 3) & 7);
    int e, m0, m_lim, kbeg, kend, m, nt;
    if constexpr (RAGK) {
        const int m_tiles = (g.M + BM - 1) / BM, per = m_tiles * n_tiles;
        if (L >= per * g.E) return;
        e = g.order ? g.order[L / per] : L / per;  // heaviest experts first
        walk_tile(L % per, m_tiles, n_tiles, m, nt);
        m0 = m * BM;
        m_lim = g.M;
        kbeg = g.offsets[e];
        kend = g.offsets[e + 1];
    } else {
        int local, b;
        if (!find_tile<BM>(g, L, n_tiles, e, b, m_lim, local)) return;
        walk_tile(local, (m_lim - b + BM - 1) / BM, n_tiles, m, nt);
        m0 = b + m * BM;
        kbeg = 0;
        kend = g.K;
    }
    const int n0 = nt * n_out;

    const int wm = (wave >> 1) * (BM / 2), wn = wave & 1;
    const int l16 = lane & 15, kg = lane >> 4;
    auto b_row = [&](int j) {  // tile column of block j: with two matrices, blocks NB/2 .. are the second one's
        return DUAL ? (j / (NB / 2)) * (BM / 2) + wn * (BM / 4) + (j % (NB / 2)) * 16 : wn * (BM / 2) + j * 16;
    };
    f32x4v acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = (f32x4v){0.f, 0.f, 0.f, 0.f};

    const int total = (kend - kbeg + kK - 1) / kK;
    f32x4v ra[TA::kPieces], rb[TB::kPieces];
    const int64_t eoff = RAGK ? 0 : (int64_t)weight_index(g, e) * g.strideB;
    TA ta;
    TB tb;
    ta.set(static_cast<const float*>(g.seg[0].A), nullptr, false, g.lda, m0, m_lim, kbeg);
    tb.set(static_cast<const float*>(g.seg[0].B) + eoff, DUAL ? static_cast<const float*>(g.seg[0].B2) + eoff : nullptr, DUAL,
           g.ldb, n0, g.N, kbeg);
    auto gload = [&](int it) {
        const int left = kend - kbeg - it * kK;
        ta.load(ra, left);
        tb.load(rb, left);
    };
    if (total > 0) {
        gload(0);
        TA::store(sA[0], ra);
        TB::store(sB[0], rb);
    }
    __syncthreads();
    for (int it = 0; it < total; ++it) {
        const bool more = it + 1 < total;
        if (more) gload(it + 1);
        const float* a_s = sA[it & 1];
        const float* b_s = sB[it & 1];
        f32x4v a[NB], b[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) a[i] = TA::frag(a_s, wm + i * 16 + l16, kg);
#pragma unroll
        for (int j = 0; j < NB; ++j) b[j] = TB::frag(b_s, b_row(j) + l16, kg);
        // (B first: blocks are accumulated transposed, a lane then holds four consecutive columns of one row)
#pragma unroll
        for (int z = 0; z < 4; ++z)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][z], a[i][z], acc[i][j], 0, 0, 0);
        if (more) {
            TA::store(sA[(it + 1) & 1], ra);
            TB::store(sB[(it + 1) & 1], rb);
        }
        __syncthreads();
    }
    const int64_t cbase = RAGK ? (int64_t)e * g.strideC : 0;
    constexpr int NJ4 = DUAL ? NB / 2 : NB;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NJ4; ++j) {
            const int row = m0 + wm + i * 16 + l16, col = n0 + b_row(j) + kg * 4;
            if (row < m_lim && col < g.N)
                epilogue_x4<float, EPI>(g, cbase + (int64_t)row * g.ldc + col, acc[i][j], acc[i][DUAL ? j + NB / 2 : j]);
        }
}

}  // namespace moe
