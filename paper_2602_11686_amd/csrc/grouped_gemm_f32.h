// Grouped fp32 GEMM on the fp32 MFMAs: fp32 operands, products and sums, at twice the rate of the scalar FMA units.
// Operand forms, tile walk and epilogues as in the bf16 kernels.  (Products with very many tiles: grouped_gemm_f32_large.h.)
//
// What bounds it is the matrix pipe (154 TFLOP/s in a loop of 16x16x4 MFMAs alone, 139 at the 2.1 GHz that the power limit
// leaves a whole kernel), and before that the last tiles: few experts of 64 to 1000 rows make few tiles.  So a workgroup of
// four wavefronts owns a tile of 64 x 64 only, and a ring of three LDS stages of 32 contraction indices (48 KB, three
// workgroups per unit), filled by DMA two stages ahead.
//
// A wavefront computes 32 x 32: as one block in 32x32x2 MFMAs in the forward products (WIDE), as 2 x 2 blocks in 16x16x4 in the
// others.  MFMA z of 16 contraction indices contracts z, 4+z, 8+z, 12+z, MFMAs 2z and 2z+1 of the wide form z, 4+z and 8+z,
// 12+z: the sums are the same bit for bit.  Kernels of whole training passes, us, 2 x 2 blocks and one block (tokens, experts, sizes):
//   forward, W1|W3 and W2: 2048, 8 of 1024 x 2816 503, 499 and 282, 276; 4096, 8 of 768 x 1024 249, 244 and 135, 134; W2 of 4096, 4 of
//     2048 x 5632 1699, 1656; of 16384, 8 of 1024 x 2816 1652, 1616
//   dgrad, W2 and W1|W3: the same 260, 271 and 529, 535; 142, 149 and 254, 257; 1642, 1675 and 3278, 3402; 1700, 1780 and 3213, 3327;
//     16384 tokens, 128 of 2048 x 768 3668, 3835 and 7080, 7321
//   gradients: 243, 244 (W2, the first); 127, 127 and 235, 241 (the second); 1675, 1707 (W2, the last); only W2 of 8192, 8 of 512 x 1024
//     the other way, 175, 169
// Whole passes under load, us, 2 x 2 blocks everywhere, one block everywhere, this: 2048, 8 of 1024 x 2816 2135, 2142, 2135; 4096, 4 of
// 2048 x 5632 14553, 14880, 14550; 16384, 128 of 2048 x 768 32870, 34310, 32950; 16384, 8 of 1024 x 2816 14760, 15180, 14820.
//
// Measured, training passes (us; 128x128 or 64x64 tiles staged through registers, 16 indices per stage -> 2 x 2 blocks): 2048 tokens, 8
// experts of 1024 x 2816 2368 -> 2157; 4096 tokens, 4 of 2048 x 5632 8428 -> 7870; 512 tokens, 8 of 1024 x 2816 970 -> 816;
// 2000 tokens, 24 of 516 x 1036 925 -> 798; forward of 64 tokens, 64 of 2048 x 1408 1230 -> 665, of 8 tokens, 8 of
// 1024 x 2816 205 -> 142.  80 to 110 TFLOP/s.  Tried: 64 x 128 tiles (-4 to +1.5 %), 128 x 128 with two stages (0 to -18 %), two
// or four stages (-2 to +1, -3 to -6 %), fragments of the next half stage read under the MFMAs of this one (0).  What the DMA costs, from
// copies with pieces left out: without requests in the loop 1882 of 2123 us, without LDS reads 2102, without barriers too 1862.
//
// LDS: an operand whose contraction index is contiguous in memory ("row form") lies as [64 rows][128 B], the 16-byte piece
// p of row r in slot p ^ ((r >> 1) & 7); a lane reads four consecutive k of its row at once.  An operand whose other index is
// contiguous ("k-row form") lies as [32 k-rows][256 B], piece p of k-row q in slot p ^ swz(q).  2 x 2 blocks: a lane reads W neighbouring
// columns of a k-row at once, one for each of W blocks: block j of those holds columns W*n + j, n = 0 .. 15.  One block: half a
// wavefront reads 32 columns of a k-row, the other half those of the k-row four further on, from the other half of the banks (two
// matrices, 16 columns of each: from the other two quarters).
#pragma once

namespace moe {

constexpr int kF32Tile = 64, kF32K = 32, kF32Stages = 3;
constexpr int kF32Operand = kF32Tile * kF32K * 4;              // bytes of one operand's stage
constexpr int kF32Lds = kF32Stages * 2 * kF32Operand;

// WIDE: a block of 32 x 32 per wavefront, otherwise 2 x 2 blocks of 16 x 16.
template <bool WIDE, bool DUAL>
__device__ __forceinline__ int swz_f32(int q) { return WIDE ? (DUAL ? 4 : 8) * ((q >> 2) & 1) : 8 * ((q >> 2) & 1) + 4 * ((q >> 3) & 1); }

// This wavefront's DMA chunks (1 KB) of one operand's stages.
template <int FORM, bool WIDE, bool DUAL>  // 0: row form; 1: k-row form
struct F32Issue {
    static constexpr int kChunks = kF32Operand / 4096;  // per wavefront and stage
    static constexpr int kRowPieces = FORM == 0 ? 8 : kF32Tile / 4;
    const char* at[kChunks];  // this lane's pieces of the next stage
    int kk[kChunks];          // their contraction index inside the stage
    int64_t step;             // bytes from one stage to the next
    // rows (or columns) r0 .. of `base`, those from r_lim on: any valid ones (masked at the store); `split`: from tile column
    // 32 on they are those of base2
    __device__ __forceinline__ void set(const float* base, const float* base2, bool split, int64_t ld, int r0, int r_lim, int k0) {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        step = (FORM == 0 ? kF32K : kF32K * ld) * 4;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const int p = (wave * kChunks + i) * 64 + lane, line = p / kRowPieces, slot = p % kRowPieces;
            int r;
            if constexpr (FORM == 0) {
                r = line;
                kk[i] = (slot ^ swz_rows(line)) * 4;
            } else {
                r = (slot ^ swz_f32<WIDE, DUAL>(line)) * 4;
                kk[i] = line;
            }
            const bool second = split && r >= kF32Tile / 2;
            r = min(r0 + r - (second ? kF32Tile / 2 : 0), FORM == 0 ? r_lim - 1 : r_lim - 4);
            const float* b = second ? base2 : base;
            at[i] = reinterpret_cast<const char*>(b + (FORM == 0 ? (int64_t)r * ld + k0 + kk[i] : (int64_t)(k0 + kk[i]) * ld + r));
        }
    }
    // the next stage, of which `left` contraction indices exist; the others read zeros (leading dimensions and extents are
    // multiples of four: a piece is inside or outside as a whole)
    __device__ __forceinline__ void issue(uint32_t lds_wave, int left) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            dma16(kk[i] < left ? at[i] : reinterpret_cast<const char*>(kZeroRow) + (threadIdx.x & 31) * 16, lds_wave + i * 1024);
            at[i] += step;
        }
    }
};

template <int W>
__device__ __forceinline__ void lds_floats(const char* p, float (&v)[W]) {
    if constexpr (W == 1) v[0] = *reinterpret_cast<const float*>(p);
    else if constexpr (W == 2) { const f32x2v x = *reinterpret_cast<const f32x2v*>(p); v[0] = x[0]; v[1] = x[1]; }
    else { const f32x4v x = *reinterpret_cast<const f32x4v*>(p); for (int j = 0; j < 4; ++j) v[j] = x[j]; }
}

template <bool WIDE> struct F32Acc { using type = f32x16; };
template <> struct F32Acc<false> { using type = f32x4v; };

template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
__global__ __launch_bounds__(256, 2) void gg_f32_kernel(const GArgs g) {
    static_assert(!(DUAL && BT == 1), "two B matrices are taken in k-row form only");
    constexpr bool WIDE = AT == 0 && BT == 0;
    using TA = F32Issue<AT, WIDE, false>;
    using TB = F32Issue<BT == 0 ? 1 : 0, WIDE, DUAL>;
    constexpr int BM = kF32Tile, S = kF32Stages;
    constexpr int NB = WIDE ? 1 : 2;               // blocks per wavefront along each side
    constexpr int WB = WIDE || DUAL ? 1 : 2;       // blocks that share a read of B in k-row form
    constexpr int kOperand = kF32Operand, kStage = 2 * kOperand;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
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

    // ---- issue side ----
    const int nk = (kend - kbeg + kF32K - 1) / kF32K, total = nk * g.nseg;
    const int64_t eoff = RAGK ? 0 : (int64_t)weight_index(g, e) * g.strideB;
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_AS char*)smem);
    TA ta;
    TB tb;
    auto segment = [&](int sg) {
        ta.set(static_cast<const float*>(g.seg[sg].A), nullptr, false, g.lda, m0, m_lim, kbeg);
        tb.set(static_cast<const float*>(g.seg[sg].B) + eoff, DUAL ? static_cast<const float*>(g.seg[sg].B2) + eoff : nullptr,
               DUAL, g.ldb, n0, g.N, kbeg);
    };
    auto issue = [&](int it, int buf) {
        if (it == nk) segment(1);
        const int left = kend - kbeg - (it >= nk ? it - nk : it) * kF32K;
        const uint32_t st = lds_base + buf * kStage + wave * (TA::kChunks * 1024);
        ta.issue(st, left);
        tb.issue(st + kOperand, left);
    };
    segment(0);

    // ---- compute side ----
    const int wm = wave >> 1, wn = wave & 1, ln = lane & (WIDE ? 31 : 15), kg = lane / (WIDE ? 32 : 16);
    typename F32Acc<WIDE>::type acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < (WIDE ? 16 : 4); ++r) acc[i][j][r] = 0.f;
    // WIDE: v[p][z] is this lane's row or column `line` at k = 16*h + 8*p + 4*kg + z.  Otherwise v[j][z] is block j's value at
    // k = 16*h + 4*kg + z, of the rows or columns from `line` on, W blocks sharing a read (DUAL: half the blocks are the second matrix's).
    auto frags = [&](auto form, auto width, auto dual, const char* s, int line, int h, float (&v)[2][4]) {
        constexpr int W = decltype(width)::value;
        if constexpr (WIDE) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                if constexpr (decltype(form)::value == 0) {
                    lds_floats<4>(s + line * 128 + (((h * 4 + p * 2 + kg) ^ swz_rows(ln)) << 4), v[p]);  // (swz_rows repeats every 16 rows)
                } else {
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const int k = h * 16 + p * 8 + kg * 4 + z;
                        v[p][z] = *reinterpret_cast<const float*>(s + k * (BM * 4) + (((line >> 2) ^ swz_f32<true, decltype(dual)::value>(kg * 4)) << 4) + (line & 3) * 4);
                    }
                }
            }
        } else if constexpr (decltype(form)::value == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                lds_floats<4>(s + (line + j * 16 + ln) * 128 + (((h * 4 + kg) ^ swz_rows(ln)) << 4), v[j]);
        } else {
#pragma unroll
            for (int z = 0; z < 4; ++z)
#pragma unroll
                for (int q = 0; q < 2 / W; ++q) {
                    const int col = q * (BM / 2) + line + ln * W, k = kg * 4 + z;
                    float x[W];
                    lds_floats<W>(s + (h * 16 + k) * (BM * 4) + (((col >> 2) ^ swz_f32<false, false>(k)) << 4) + (col & 3) * 4, x);
#pragma unroll
                    for (int j = 0; j < W; ++j) v[q * W + j][z] = x[j];
                }
        }
    };
    // (WIDE, two matrices: 16 columns of each)
    const int a_line = wm * 32 + (WIDE ? ln : 0);
    const int b_line = !WIDE ? wn * 16 * WB : DUAL ? (ln >> 4) * (BM / 2) + wn * 16 + (ln & 15) : wn * 32 + ln;
    auto compute = [&](int buf) {
        const char* sa = smem + buf * kStage;
        const char* sb = sa + kOperand;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            float a[2][4], b[2][4];
            frags(IntTag<AT>{}, IntTag<2>{}, IntTag<0>{}, sa, a_line, h, a);
            frags(IntTag<BT == 0 ? 1 : 0>{}, IntTag<WB>{}, IntTag<DUAL>{}, sb, b_line, h, b);
            // (B first: blocks are accumulated transposed)
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                if constexpr (WIDE) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[p][z], a[p][z], acc[0][0], 0, 0, 0);
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][z], a[i][z], acc[i][j], 0, 0, 0);
                }
            }
        }
    };
    for (int s = 0; s < S - 1 && s < total; ++s) issue(s, s);
    int cur = 0, fill = S - 1;  // ring positions of the stage computed and of the one requested next
    for (int it = 0; it < total; ++it) {
        // stage `it` has landed (behind it up to S-2 stages are in flight) and this wavefront's LDS reads of the buffer that is
        // refilled below have returned; the barrier says so for all wavefronts
        if (it + S - 1 <= total) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * 2 * TA::kChunks) : "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (it + S - 1 < total) issue(it + S - 1, fill);
        compute(cur);
        cur = cur + 1 == S ? 0 : cur + 1;
        fill = fill + 1 == S ? 0 : fill + 1;
    }

    // ---- epilogue: a lane holds, of each of its rows, quads of four consecutive columns ----
    const int64_t cbase = RAGK ? (int64_t)e * g.strideC : 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int row = m0 + wm * 32 + (WIDE ? ln : AT == 0 ? i * 16 + ln : ln * 2 + i);
        auto quad = [&](int q, int t) {  // matrix q, quad t
            f32x4v v;
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                if constexpr (WIDE) v[z] = acc[0][0][(q * 2 + t) * 4 + z];
                else if constexpr (BT == 1) v[z] = acc[i][t][z];
                else v[z] = acc[i][q * WB + (4 * t + z) % WB][(4 * t + z) / WB];
            }
            return v;
        };
        constexpr int NQ = WIDE ? (DUAL ? 2 : 4) : WB;
#pragma unroll
        for (int t = 0; t < NQ; ++t) {
            int col = n0;
            if constexpr (WIDE) col += wn * (DUAL ? 16 : 32) + t * 8 + kg * 4;
            else col += wn * 16 * WB + (BT == 1 ? t * 16 + kg * 4 : kg * 4 * WB + t * 4);
            if (row < m_lim && col < g.N)
                epilogue_x4<float, EPI>(g, cbase + (int64_t)row * g.ldc + col, quad(0, t), quad(DUAL ? 1 : 0, t));
        }
    }
}

}  // namespace moe
