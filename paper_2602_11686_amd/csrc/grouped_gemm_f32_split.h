// Grouped fp32 GEMM for products with few tiles: the wavefronts of a workgroup share a 32 x 32 tile and split its contraction.
// Operand forms, tile walk and epilogues as in grouped_gemm_f32.h; MFMAs 16x16x4, in 2 x 2 blocks.
//
// What bounds a product that leaves units idle is the chain of one tile: 1024 clocks of MFMAs per wavefront and stage of 32
// contraction indices (32 16x16x4 or 16 32x32x2), one memory latency at the start, and a barrier per stage.  Here wavefront w contracts the slabs
// w, w+4, w+8, ... of 32 indices on its own, from a ring of two slabs (16 KB) that only it fills and reads: a quarter of the
// chain, no barrier before the end, and 256 indices requested at once.  The four sums meet in LDS, added in the order of the
// wavefronts.  A tile a quarter as large is four times the workgroups, at twice the operand traffic per FLOP: with enough tiles
// the 64 x 64 kernel is the faster one (f32_split_tiles has the line).
//
// Measured, kernels of a training pass in launch order (us; 64 x 64 tiles in 2 x 2 blocks -> this): 256 tokens, 8 experts of 128 x 256 8.0, 9.6, 9.3, 14.6,
// 6.8, 6.8 -> 6.7, 5.2, 6.0, 6.9, 4.6, 6.1.  Whole passes: forward of 8 tokens, 8 experts of 1024 x 2816 151 -> 88, of 64 tokens, 64 of
// 2048 x 1408 720 -> 540; training, 64 tokens, 8 of 1024 x 2816 411 -> 282, 2048 tokens, 4 of 256 x 512 239 -> 220.  Against 64 bits
// four sums of a quarter each are closer than one (y of the first two 1.3e-6 -> 6.4e-7, 1.4e-6 -> 6.9e-7).
//
// LDS: row form slabs [32 rows][128 B], the 16-byte piece p of row r in slot p ^ ((r >> 1) & 7).  k-row form slabs [32 lines][128 B],
// line k ^ ((k >> 2) & 1) holds k-row k, piece p in slot p ^ 4 * ((k >> 3) & 1): the four k-rows that a read touches (k, k+4, k+8,
// k+12) alternate between the two halves of the banks, and where 16 columns are read between the quarters.
#pragma once

namespace moe {

constexpr int kF32SplitTile = 32, kF32SplitStages = 2;
constexpr int kF32Slab = kF32SplitTile * kF32K * 4;                     // bytes of one operand's slab
constexpr int kF32SplitWave = kF32SplitStages * 2 * kF32Slab;           // a wavefront's ring
constexpr int kF32SplitLds = 4 * kF32SplitWave;

// A wavefront's requests of one operand's slabs.
template <int FORM>  // 0: row form; 1: k-row form
struct F32SlabIssue {
    static constexpr int kChunks = kF32Slab / 1024;
    const char* at[kChunks];  // this lane's pieces of the next slab
    int kk[kChunks];          // their contraction index inside the slab
    int64_t step;             // bytes from one slab of this wavefront to the next
    // as F32Issue::set; `split`: from tile column 16 on they are those of base2
    __device__ __forceinline__ void set(const float* base, const float* base2, bool split, int64_t ld, int r0, int r_lim, int k0) {
        const int lane = threadIdx.x & 63;
        step = 4 * (FORM == 0 ? kF32K : kF32K * ld) * 4;
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            const int p = i * 64 + lane, line = p >> 3, slot = p & 7;
            int r;
            if constexpr (FORM == 0) {
                r = line;
                kk[i] = (slot ^ swz_rows(line)) * 4;
            } else {
                kk[i] = line ^ ((line >> 2) & 1);
                r = (slot ^ (4 * ((line >> 3) & 1))) * 4;
            }
            const bool second = split && r >= kF32SplitTile / 2;
            r = min(r0 + r - (second ? kF32SplitTile / 2 : 0), FORM == 0 ? r_lim - 1 : r_lim - 4);
            const float* b = second ? base2 : base;
            at[i] = reinterpret_cast<const char*>(b + (FORM == 0 ? (int64_t)r * ld + k0 + kk[i] : (int64_t)(k0 + kk[i]) * ld + r));
        }
    }
    __device__ __forceinline__ void issue(uint32_t lds, int left) {
#pragma unroll
        for (int i = 0; i < kChunks; ++i) {
            dma16(kk[i] < left ? at[i] : reinterpret_cast<const char*>(kZeroRow) + (threadIdx.x & 31) * 16, lds + i * 1024);
            at[i] += step;
        }
    }
};

// One workgroup's tile: workgroup b0 of the product.
template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
__device__ __forceinline__ void f32_split_tile(const GArgs& g, int b0, char* smem) {
    static_assert(!(DUAL && BT == 1), "two B matrices are taken in k-row form only");
    using TA = F32SlabIssue<AT>;
    using TB = F32SlabIssue<BT == 0 ? 1 : 0>;
    constexpr int BM = kF32SplitTile, S = kF32SplitStages;
    constexpr int WB = DUAL ? 1 : 2;  // blocks that share a read of B in k-row form
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_out = DUAL ? BM / 2 : BM;
    const int n_tiles = (g.N + n_out - 1) / n_out;

    // ---- which tile (as in gg_f32_kernel; a product has a multiple of 64 workgroups) ----
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

    // ---- issue side: slab j of this wavefront is slab wave + 4*j of the tile ----
    const int nk = (kend - kbeg + kF32K - 1) / kF32K, slabs = nk * g.nseg;
    const int total = wave < slabs ? (slabs - wave + 3) / 4 : 0;
    const int64_t eoff = RAGK ? 0 : (int64_t)weight_index(g, e) * g.strideB;
    char* const ring = smem + wave * kF32SplitWave;
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_AS char*)ring);
    TA ta;
    TB tb;
    int seg = -1;
    auto issue = [&](int j, int buf) {
        const int slab = wave + 4 * j, sg = slab >= nk ? 1 : 0, k0 = kbeg + (slab - sg * nk) * kF32K;
        if (sg != seg) {
            seg = sg;
            ta.set(static_cast<const float*>(g.seg[sg].A), nullptr, false, g.lda, m0, m_lim, k0);
            tb.set(static_cast<const float*>(g.seg[sg].B) + eoff, DUAL ? static_cast<const float*>(g.seg[sg].B2) + eoff : nullptr,
                   DUAL, g.ldb, n0, g.N, k0);
        }
        ta.issue(lds_wave + buf * 2 * kF32Slab, kend - k0);
        tb.issue(lds_wave + buf * 2 * kF32Slab + kF32Slab, kend - k0);
    };

    // ---- compute side ----
    const int l16 = lane & 15, kg = lane >> 4;
    f32x4v acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    // v[j][z]: block j's value at k = 16*h + 4*kg + z
    auto frags = [&](auto form, auto width, const char* s, int h, float (&v)[2][4]) {
        constexpr int W = decltype(width)::value;
        if constexpr (decltype(form)::value == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j)
                lds_floats<4>(s + (j * 16 + l16) * 128 + (((h * 4 + kg) ^ swz_rows(l16)) << 4), v[j]);  // (swz_rows repeats every 16 rows)
        } else {
#pragma unroll
            for (int z = 0; z < 4; ++z)
#pragma unroll
                for (int q = 0; q < 2 / W; ++q) {  // (DUAL: q is the matrix)
                    const int col = q * 16 + l16 * W, line = (h * 16 + kg * 4 + z) ^ (kg & 1);
                    float x[W];
                    lds_floats<W>(s + line * 128 + (((col >> 2) ^ (4 * (kg >> 1))) << 4) + (col & 3) * 4, x);
#pragma unroll
                    for (int j = 0; j < W; ++j) v[q * W + j][z] = x[j];
                }
        }
    };
    for (int j = 0; j < S && j < total; ++j) issue(j, j);
    for (int it = 0; it < total; ++it) {
        const int buf = it & 1;
        // slab `it` has landed, the one behind it may be in flight (nobody else touches this wavefront's ring)
        if (it + 1 < total) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * TA::kChunks) : "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const char* sa = ring + buf * 2 * kF32Slab;
        float a[2][2][4], b[2][2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            frags(IntTag<AT>{}, IntTag<2>{}, sa, h, a[h]);
            frags(IntTag<BT == 0 ? 1 : 0>{}, IntTag<WB>{}, sa + kF32Slab, h, b[h]);
        }
        if (it + S < total) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the reads of this slab have returned: it may be refilled
            issue(it + S, buf);
        }
        // (B first: blocks are accumulated transposed)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int z = 0; z < 4; ++z)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[h][j][z], a[h][i][z], acc[i][j], 0, 0, 0);
    }

    // ---- the four sums: quads of four consecutive columns of a row (DUAL: [matrix][row block], else [row block][quad]) ----
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        f32x4v v;
        if constexpr (BT == 1) {
            v = acc[u >> 1][u & 1];
        } else {
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                if constexpr (DUAL) v[z] = acc[u & 1][u >> 1][z];
                else v[z] = acc[u >> 1][z % 2][2 * (u & 1) + z / 2];
            }
        }
        *reinterpret_cast<f32x4v*>(ring + u * 1024 + lane * 16) = v;
    }
    __syncthreads();
    auto sum = [&](int u) {
        const char* p = smem + u * 1024 + lane * 16;
        f32x4v v = *reinterpret_cast<const f32x4v*>(p);
#pragma unroll
        for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const f32x4v*>(p + w * kF32SplitWave);
        return v;
    };
    if (DUAL && wave >= 2) return;
    const int i = DUAL ? wave : wave >> 1, t = DUAL ? 0 : wave & 1;
    const int row = m0 + (AT == 0 ? i * 16 + l16 : l16 * 2 + i);
    const int col = n0 + (BT == 1 ? t * 16 + kg * 4 : kg * 4 * WB + t * 4);
    if (row < m_lim && col < g.N) {
        const f32x4v v0 = sum(wave), v1 = DUAL ? sum(2 + wave) : v0;
        epilogue_x4<float, EPI>(g, (RAGK ? (int64_t)e * g.strideC : 0) + (int64_t)row * g.ldc + col, v0, v1);
    }
}

template <int AT, int BT, bool DUAL, int EPI, bool RAGK>
__global__ __launch_bounds__(256) void gg_f32_split_kernel(const GArgs g) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    f32_split_tile<AT, BT, DUAL, EPI, RAGK>(g, (int)(blockIdx.y * gridDim.x + blockIdx.x), smem);
}

// The three products behind dH, which need nothing of one another, in one launch: as launches of their own each leaves most
// of the chip idle and pays its start and its end.  The rows' gradient first, its contraction is the longest.  256 tokens, 8
// experts of 128 x 256 (us): four launches (the experts' order among them) of 6.9, 1.6, 4.6, 6.1 -> 10.2; the training pass, bound by
// the host's launches, 89 -> 80.
struct F32SplitBwdArgs {
    GArgs dx, dw2, dw13;
    int dx_blocks, dw2_blocks;
};
__global__ __launch_bounds__(256) void gg_f32_split_bwd_kernel(const F32SplitBwdArgs a) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (b < a.dx_blocks) f32_split_tile<0, 1, false, EPI_STORE, false>(a.dx, b, smem);
    else if (b < a.dx_blocks + a.dw2_blocks) f32_split_tile<1, 0, false, EPI_STORE, true>(a.dw2, b - a.dx_blocks, smem);
    else f32_split_tile<1, 0, true, EPI_STORE2, true>(a.dw13, b - a.dx_blocks - a.dw2_blocks, smem);
}

}  // namespace moe
