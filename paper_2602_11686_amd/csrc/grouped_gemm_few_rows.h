// Grouped bf16 GEMM for experts with few rows (decode steps, short batches): the weights are the work.
//
//   C[m,n] = sum_k A(m,k) * B(k,n) per expert, ragged M, the operand forms and epilogues of gg_quad_kernel
//
// What bounds it is how fast the weights arrive from HBM, so the tile is chosen for loads in flight: a workgroup
// of four wavefronts owns BM rows x 64 columns (per B matrix, or two column blocks of 64: NB = 2) and streams its B
// columns in 64-wide k-stages through a ring of S LDS buffers, filled by DMA S-1 stages ahead, and the number of tiles is
// several times the number of units where gg_quad_kernel has too few 256-wide ones.  Every B request takes whole 128-byte
// lines.  Workgroups per unit and weights in flight on it (gg_quad_kernel: two stages of 32 KB), by instance <BM, NB, S>:
//   <64,2,3> 2, 64 KB    <64,1,3> 3, 48 KB    <128,2,2> 2, 32 KB    <128,1,3> 2, 32 KB    <128,2,3> 1, 32 KB
// Weights are requested non-temporally where one row tile uses them.  An expert's second row tile runs beside the first
// on the same XCD, but finds such lines in its L2 only in part (bytes fetched past L2 over the weights' own: 96 rows in
// tiles of 64 1.6, 200 rows in tiles of 128 2.0): with several row tiles the requests are plain (us, W1|W3 and both dgrads;
// 2048 rows over 64 experts of 2048 x 1408, Zipf-skewed: 165 -> 150, 240 -> 218; 4096 rows on 16 of 128 experts of
// 2048 x 768: 80 -> 67, 148 -> 115).  Two loops, because the test inside one costs 64 tokens of 128 experts 1 %.
// (Replica groups: the test is the group's own.  Plain requests where another group has the expert, whole passes in us: 64 groups
// of 8 experts of 4096 x 2048, 16 and 32 rows per group 1665 -> 1567, 1712 -> 1634; 32 of 16, 16 rows 915 -> 884; but 128 of 64
// experts of 2048 x 1408, 16 and 32 rows 1258 -> 1270, 1323 -> 1361.)
//
// LDS: row form (K contiguous; A, and B in the dgrad products) as [64 or BM rows][128 B], read with ds_read_b128;
// k-row form (N contiguous; B forward) as [64 k-rows][128 B], read with the transposing ds_read_b64_tr_b16.  The
// 16-byte piece p of row r sits in slot p ^ swz(r), applied on the global side of the DMA; the rows that one LDS
// read touches then fall into different banks.
//
// MFMA 16x16x32, B first: a lane holds four consecutive columns of one row.  Wavefront w computes columns
// 16w .. 16w+15 of every column block for all rows of the tile; 16-row blocks past the expert's rows are skipped.
//
// Measured (BM 64, NB 2, S 3; the weights of the live experts over the time): 8 tokens, 2 of 8 experts of
// 4096 x 14336: W1|W3 370 -> 302 us (5.5 TB/s), W2 300 -> 136 us (6.0 TB/s; a read-only kernel reaches 6.3, 7.1 with
// non-temporal loads); 64 tokens, 8 of 128 experts of 2048 x 768: 159 -> 117 us and 84 -> 62 us.  With plain weight
// loads these are 335, 155, 133 and 70 us.  Two stages instead of three: 332 and 198 us at 8 tokens.
#pragma once

namespace moe {

constexpr int kFewThreads = 256;

template <int BM, int NB, int S>
constexpr int few_rows_lds() { return S * (BM * 128 + NB * 8192); }

__device__ __forceinline__ int swz_few_krow(int q) { return 2 * (((q >> 1) & 1) | (((q >> 3) & 1) << 1)); }

// dma16 for what is read once: non-temporal
__device__ __forceinline__ void dma16_stream(const void* gsrc, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" ::"s"(lds_addr), "v"(gsrc) : "memory", "m0");
}

template <int BT, bool DUAL, int EPI, int BM, int NB, int S>
__global__ __launch_bounds__(kFewThreads) void gg_few_rows_kernel(const GArgs g) {
    static_assert(!(DUAL && (BT == 1 || NB != 2)), "two B matrices: one column block of each, k-row form");
    constexpr int MI = BM / 16;
    constexpr int kABytes = BM * 128, kStage = kABytes + NB * 8192;
    constexpr int CA = BM / 32, CB = 2 * NB;  // DMA instructions per wavefront and stage
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_out = DUAL ? 64 : 64 * NB;
    const int n_tiles = (g.N + n_out - 1) / n_out;
    // chunks of eight consecutive tiles go to the XCDs in turn (the grid is a multiple of 64); the row tiles of
    // one column tile are consecutive
    const int L = (((int)(blockIdx.x >> 6) * 8 + (int)(blockIdx.x & 7)) << 3) + (int)((blockIdx.x >> 3) & 7);
    int e, m0, m_lim, local;
    if (!find_tile<BM>(g, L, n_tiles, e, m0, m_lim, local)) return;
    const int m_tiles = (m_lim - m0 + BM - 1) / BM;
    const int n0 = (local / m_tiles) * n_out;
    m0 += (local % m_tiles) * BM;
    const int rows = m_lim - m0;

    // ---- issue side: this wavefront's pieces of a stage ----
    const int64_t woff = (int64_t)weight_index(g, e) * g.strideB;
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_AS char*)smem);
    const int nk = (g.K + 63) / 64, total = nk * g.nseg;
    const char* zeros = reinterpret_cast<const char*>(kZeroRow) + (lane & 31) * 16;
    int64_t a_off[CA], b_off[CB];  // byte offsets of this lane's pieces from the segment's matrices, at k = 0
    int a_k[CA], b_k[CB];          // their k inside the stage
#pragma unroll
    for (int i = 0; i < CA; ++i) {
        const int r = (wave * CA + i) * 8 + (lane >> 3);
        a_k[i] = ((lane & 7) ^ swz_rows(r)) * 8;
        a_off[i] = ((int64_t)(m0 + min(r, rows - 1)) * g.lda + a_k[i]) * 2;  // (rows past the end: any; masked at the store)
    }
#pragma unroll
    for (int i = 0; i < CB; ++i) {
        const int c = wave * CB + i, h = c >> 3, r = (c & 7) * 8 + (lane >> 3);
        const int nb = n0 + (DUAL ? 0 : h * 64);
        if constexpr (BT == 1) {
            b_k[i] = ((lane & 7) ^ swz_rows(r)) * 8;
            b_off[i] = (woff + (int64_t)min(nb + r, g.N - 1) * g.ldb + b_k[i]) * 2;
        } else {
            b_k[i] = r;
            b_off[i] = (woff + (int64_t)r * g.ldb + min(nb + ((lane & 7) ^ swz_few_krow(r)) * 8, g.N - 8)) * 2;
        }
    }
    const int b_mat = DUAL ? wave >> 1 : 0;  // (CB = 4 chunks per wavefront: half h = wave/2)
    auto issue = [&](auto stream, int stage, int buf) {
        const int sg = stage >= nk ? 1 : 0, k0 = (stage - sg * nk) * 64, left = g.K - k0;
        const uint32_t st = lds_base + buf * kStage;
        const char* Ab = static_cast<const char*>(g.seg[sg].A) + (int64_t)k0 * 2;
        const char* Bb = static_cast<const char*>(b_mat ? g.seg[sg].B2 : g.seg[sg].B) + (int64_t)k0 * (BT == 1 ? 1 : g.ldb) * 2;
#pragma unroll
        for (int i = 0; i < CA; ++i)
            dma16(a_k[i] < left ? Ab + a_off[i] : zeros, st + (wave * CA + i) * 1024);
#pragma unroll
        for (int i = 0; i < CB; ++i) {
            const void* from = b_k[i] < left ? Bb + b_off[i] : zeros;
            if constexpr (decltype(stream)::value) dma16_stream(from, st + kABytes + (wave * CB + i) * 1024);
            else dma16(from, st + kABytes + (wave * CB + i) * 1024);
        }
    };

    // ---- compute side ----
    const int l16 = lane & 15, kg = lane >> 4;
    const int tr_q = kg * 8 + (l16 >> 2);  // + 32*ks + 4*t: neither changes the swizzle
    int b_rd;
    if constexpr (BT == 1) b_rd = (wave * 16 + l16) * 128;
    else b_rd = tr_q * 128 + (((wave * 2 + ((l16 & 3) >> 1)) ^ swz_few_krow(tr_q)) << 4) + (l16 & 1) * 8;
    f32x4v acc[MI][NB];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int h = 0; h < NB; ++h) acc[i][h] = (f32x4v){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](int buf) {
        const char* sa = smem + buf * kStage;
        const char* sb = sa + kABytes;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 b[NB];
            const int piece = ((ks * 4 + kg) ^ swz_rows(l16)) << 4;  // (swz_rows repeats every 16 rows)
#pragma unroll
            for (int h = 0; h < NB; ++h) {
                if constexpr (BT == 1) {
                    b[h] = *reinterpret_cast<const bf16x8*>(sb + h * 8192 + b_rd + piece);
                } else {
                    const char* p = sb + h * 8192 + b_rd + ks * 4096;
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)p);
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p + 512));
                    b[h] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                }
            }
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                if (i * 16 >= rows) break;
                const bf16x8 a = *reinterpret_cast<const bf16x8*>(sa + (i * 16 + l16) * 128 + piece);
#pragma unroll
                for (int h = 0; h < NB; ++h) acc[i][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[h], a, acc[i][h], 0, 0, 0);
            }
        }
    };
    auto run = [&](auto stream) {
        for (int s = 0; s < S - 1 && s < total; ++s) issue(stream, s, s);
        int cur = 0, fill = S - 1;  // ring positions of the stage computed and of the one requested next
        for (int it = 0; it < total; ++it) {
            // stage `it` has landed (behind it up to S-2 stages are in flight) and this wavefront's LDS reads of the buffer
            // that is refilled below have returned; the barrier says so for all wavefronts
            if (it + S - 1 <= total) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S - 2) * (CA + CB)) : "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
            __syncthreads();
            if (it + S - 1 < total) issue(stream, it + S - 1, fill);
            compute(cur);
            cur = cur + 1 == S ? 0 : cur + 1;
            fill = fill + 1 == S ? 0 : fill + 1;
        }
    };
    if (m_tiles == 1) run(IntTag<1>{});
    else run(IntTag<0>{});

    // ---- epilogue: four consecutive columns of one row per lane, stored directly ----
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        if (i * 16 >= rows) break;
        const int r = i * 16 + l16;
#pragma unroll
        for (int h = 0; h < (DUAL ? 1 : NB); ++h) {
            const int col = n0 + h * 64 + wave * 16 + kg * 4;
            if (r < rows && col < g.N)
                epilogue_x4<bf16_t, EPI>(g, (int64_t)(m0 + r) * g.ldc + col, acc[i][h], acc[i][DUAL ? 1 : h]);
        }
    }
}

}  // namespace moe
