// Grouped bf16 GEMM over ragged row counts, 256x256x64 tiles computed quadrant by quadrant.
//
// One template covers the six products of the expert FFN (6*H*H' FLOPs per routed token forward, twice that backward;
// paper section 3.1):
//
//   RAGK == false: the ragged dimension is M (the rows of one expert)
//       A  [rows][K]  K contiguous                 (Xp, H, dYp, dA, dB)
//       B  BT == 0: [K][N]  N contiguous           (forward: W1, W3 [d][f], W2 [f][d])
//          BT == 1: [N][K]  K contiguous           (dgrad:   W2 as [f][d], W1/W3 as [d][f])
//   RAGK == true: the ragged dimension is the contraction (wgrad), BT == 0
//       A  [rows][M]  M contiguous                 (Xp, H)
//       B  [rows][N]  N contiguous                 (dA|dB, dYp)
//       C_e [M][N] = sum over the rows of expert e;  an expert without rows gets zeros.
//
// What bounds a loop with one barrier per k-stage is that barrier: the 64 DMA instructions of a stage can only be
// requested behind it, in a burst, and have to land before the next one.  Here a stage's tile is computed as four quadrants of
// 128 x 128, so that its four operand halves (A0, B0, B1, A1: 128 rows or columns each, 16 KB) fall free one after the
// other, and the halves of the stage after next are requested into them one by one:
//
//   phase 1  A0 x B0, fragments of B1 are read         request A1 of stage t+1
//   -- barrier X: A1 of stage t has landed; A0, B0 of stage t are free
//   phase 2  A0 x B1, fragments of A1 are read         request A0 of stage t+2
//   phase 3  A1 x B1                                   request B0 of stage t+2
//   -- barrier Y: A0, B0, B1 of stage t+1 have landed; A1, B1 of stage t are free
//   phase 4  A1 x B0, fragments of A0, B0 of stage t+1 request B1 of stage t+2
//
// Two DMA instructions per wavefront and phase, every half has a whole stage to land, and the waits count (vmcnt 8 and
// 6), so that the queue of requests never drains, not between tiles either: requests run along the workgroup's
// list of tiles two stages ahead of the MFMAs, and the first stages of the next tile arrive under the last stages and the
// epilogue of this one.  A fragment register is read anew right behind the last MFMA that takes it.
//
// 8 wavefronts, 2 x 4; a wavefront computes 64 x 32 of each quadrant (rows 128*qm + 64*wm, columns 128*qn + 32*wn),
// accumulated transposed (B is the first operand).  128 accumulators and 64 fragment registers per lane.
//
// The MFMAs are 16x16x32.  On large products the power limit sets the shader clock, so a product takes as long as
// the energy of its operations: an MFMA-only loop over normally distributed operands holds 2080 TFLOP/s in
// 16x16x32 and 1810 in 32x32x16 (zeros: 2450 in both).  One accumulation per 32 contraction indices instead of two.
//
// Measured, 32768 rows over 8 experts of 4096 x 14336 (us; one barrier per stage and 32x32x16 -> this): forward 1
// 6500 -> 6070, forward 2 3210 -> 2930, dgrad 1 3620 -> 3220, dgrad 2 6500 -> 5990, 1270 to 1310 TFLOP/s without the epilogue
// of dgrad 1.  The four phases alone, still in 32x32x16: 6590, 3210, 3580, 6500 (with zeros as operands 5510, 2190, 3190,
// 4270 against 5940, 2680, 3470, 5380: 9 to 26 % fewer clocks, at a lower clock).  With the weight gradients here too a
// training pass of these sizes takes 27580 us instead of 28200, 16 experts of 4096 x 2048 over 32 groups 2854 instead of 3001.
//
// LDS: row form halves [128 rows][128 B], the 16-byte piece p of row r in slot p ^ ((r >> 1) & 7); k-row form halves
// [64 k-rows][256 B], swz_krow16 (DUAL: B0 is the first matrix, B1 the second).  The two stage buffers lie on both sides of
// 16 KB of their own for the epilogue's staging, each with its A1 next to it: the staging area is those 16 KB and the A1
// that is not requested yet.
#pragma once

namespace moe {

constexpr int kQHalf = 16384;
// byte offsets of A0, B0, B1 of a stage buffer from its base; A1 lies behind them (buffer 0) or before them (buffer 1)
constexpr int kQA0 = 0, kQB0 = kQHalf, kQB1 = 2 * kQHalf;
constexpr int kQBase0 = 0, kQA1of0 = 3 * kQHalf;
constexpr int kQA1of1 = 5 * kQHalf, kQBase1 = 6 * kQHalf;   // (16 KB between the two A1 halves)
constexpr int kQStaging0 = 3 * kQHalf, kQStaging1 = 4 * kQHalf;
constexpr int kQTableOff = 9 * kQHalf;
constexpr int kQList = 512;                                  // entries of the ring of tiles, built 256 at a time
constexpr int kQListOff = kQTableOff + ((2 * (MOE_MAX_EXPERTS + 1) * 4 + 15) & ~15);
constexpr int kQUsersOff = kQListOff + kQList * 16;
constexpr int kQuadLds = kQUsersOff + MOE_MAX_EXPERTS * 4;
static_assert(kQuadLds <= kLdsBytes, "fits the unit's LDS");

// 256-byte k-rows read transposed for 16x16x32 MFMAs: half a wavefront reads a pair of 16-byte pieces of the k-rows q, q+1, q+2,
// q+3 and q+8 .. q+11, which this spreads over all 64 banks
__device__ __forceinline__ int swz_krow16(int q) { return 2 * ((q & 3) | (((q >> 3) & 1) << 2)); }

// dma16_s for what is read once: non-temporal
__device__ __forceinline__ void dma16_s_stream(const void* sbase, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_addr), "v"(voff), "s"(sbase)
                 : "memory", "m0");
}

// KREST: K is no multiple of 64 (the last stage of a segment reads zeros past it); an instance of its own.
//
// RAGK: the contraction is ragged (AT == 1: A in k-row form, BT == 0).
//
// STREAM: what is read or written once is requested and stored non-temporally (an instance of its own: of two stores behind a
// test at run time the compiler makes one plain store).  Ragged K: C.  Ragged M: all outputs, but those of the derivative
// epilogues, and the weights of experts with a single row tile, which nobody else reads.  (Replica groups: weights
// are nobody else's where no other group with rows has the expert.  Taken for a group's own whenever the group has one tile,
// passes over 32 groups of 16 experts of 4096 x 2048, 128 groups of 64 of 2048 x 1408 and 64 groups of 8 of 4096 x 2048 took 1266,
// 1846 and 2054 us at 128, 128 and 64 rows per group, and now take 1183, 1803 and 1837.)
template <int BT, bool DUAL, int EPI, bool KREST, bool RAGK = false, bool STREAM = false>
__global__ __launch_bounds__(kThreads) void gg_quad_kernel(const GArgs g) {
    static_assert(!(DUAL && BT == 1), "two B matrices are taken in k-row form only");
    static_assert(RAGK ? BT == 0 && !KREST && (EPI == EPI_STORE || EPI == EPI_STORE2) : EPI != EPI_STORE2 && !(KREST && STREAM), "forms");
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    int32_t* t_off = reinterpret_cast<int32_t*>(smem + kQTableOff);  // [E+1] rows of each expert
    int32_t* t_pref = t_off + MOE_MAX_EXPERTS + 1;                   // [E+1] tiles before expert e
    // the workgroup's tiles: index of the weights (-1: no more tiles), m0, m_lim (STREAM: negated where nobody else reads the
    // weights), n0; ragged K: expert, m0, its first row, n0
    int4* list = reinterpret_cast<int4*>(smem + kQListOff);
    int32_t* users = reinterpret_cast<int32_t*>(smem + kQUsersOff);  // [experts] groups with rows that have the expert
    const bool count_users = STREAM && !RAGK && g.expert_of_group;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave >> 2, wn = wave & 3;
    const int n_out = DUAL ? TN / 2 : TN;     // output columns per tile
    const int n_tiles = (g.N + n_out - 1) / n_out;
    const int m_tiles_k = (g.M + TM - 1) / TM;  // ragged K

    // ---- rows of each expert and the number of tiles before it ----
    for (int i = threadIdx.x; i <= g.E; i += kThreads) t_off[i] = g.offsets[i];
    if (count_users && threadIdx.x < MOE_MAX_EXPERTS) users[threadIdx.x] = 0;
    __syncthreads();
    if (count_users && threadIdx.x < g.E && t_off[threadIdx.x + 1] > t_off[threadIdx.x]) atomicAdd(&users[weight_index(g, threadIdx.x)], 1);
    if (wave == 0) {  // exclusive scan of the per-expert tile counts: 4 experts per lane, then across lanes
        int c[4], sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = lane * 4 + u;
            c[u] = e < g.E ? (RAGK ? m_tiles_k : (t_off[e + 1] - t_off[e] + TM - 1) / TM) * n_tiles : 0;
            sum += c[u];
        }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(incl, d, 64);
            if (lane >= d) incl += o;
        }
        int run = incl - sum;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = lane * 4 + u;
            if (e <= g.E) t_pref[e] = run;
            run += c[u];
        }
        if (lane == 63) t_pref[MOE_MAX_EXPERTS] = run;  // (E == MOE_MAX_EXPERTS: the total belongs to "lane 64")
    }
    __syncthreads();
    // When the last round of tiles fills at most half of the workgroups, its tiles are cut into their upper and lower
    // 128 rows (tiles split_from + 2i and + 2i + 1), so that the round costs a 128-row tile's time.
    int total_tiles = t_pref[g.E], split_from = total_tiles;
    if constexpr (!RAGK) {
        const int left = total_tiles % (int)gridDim.x;
        if (left > 0 && 2 * left <= (int)gridDim.x) {
            split_from = total_tiles - left;
            total_tiles += left;
        }
    }
    // Logical tile L -> entry `pos` of the ring.  (The lower half of a cut tile of at most 128 rows is empty; it belongs to
    // the last round, so it ends the workgroup's list.)
    auto build_entry = [&](int pos, int L) {
        int4 d = {-1, 0, 0, 0};
        if (L < total_tiles) {
            int m, nt;
            if constexpr (RAGK) {
                const int per = m_tiles_k * n_tiles, oi = L / per;
                d.x = g.order[oi];  // heaviest experts first
                walk_tile(L - oi * per, m_tiles_k, n_tiles, m, nt);
                d.y = m * TM;
                d.z = t_off[d.x];
                d.w = nt * n_out;
            } else {
                int part = -1;
                if (L >= split_from) {
                    part = (L - split_from) & 1;
                    L = split_from + ((L - split_from) >> 1);
                }
                int lo = 0, hi = g.E - 1;  // the expert whose tiles hold L: the last one with t_pref <= L
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (t_pref[mid] <= L) lo = mid;
                    else hi = mid - 1;
                }
                const int b = t_off[lo], en = t_off[lo + 1];
                walk_tile(L - t_pref[lo], (en - b + TM - 1) / TM, n_tiles, m, nt);
                d.y = b + m * TM;
                d.z = en;
                if (part >= 0) {
                    d.y += part * (TM / 2);
                    d.z = min(en, d.y + TM / 2);
                }
                d.w = nt * n_out;
                if (d.y < d.z) d.x = weight_index(g, lo);
                if (STREAM && en - b <= (part < 0 ? TM : TM / 2) && !(count_users && users[weight_index(g, lo)] > 1)) d.z = -d.z;
            }
        }
        list[pos & (kQList - 1)] = d;
    };
    // Ragged M: the fixed order logical_tile(blockIdx.x + pos * gridDim.x).  Ragged K, where a tile costs as much as its
    // expert has rows: the first two tiles in that order, the others drawn two tiles ahead from queues.  The logical
    // order is cut into blocks of 32, block b belongs to XCD b % 8; entry c of queue x is tile ((c / 32) * 8 + x) * 32 + c % 32;
    // a workgroup draws from its XCD's queue, then from the others.
    if (!RAGK || threadIdx.x < 2) build_entry(threadIdx.x, logical_tile(blockIdx.x + threadIdx.x * gridDim.x));
    __syncthreads();
    const int xcd = blockIdx.x & 7;
    int qx = 0;  // (wavefront 0) queues found empty so far; the current one is that of XCD (xcd + qx) % 8
    auto queue_counter = [&](int x) { return g.sched + ((xcd + x) & 7) * kSchedStride; };
    auto tile_of_draw = [&](int x, int c) { return ((((c + 64) >> 5) * 8 + ((xcd + x) & 7)) << 5) + (c & 31); };
    auto draw = [&]() -> int {
        return qx < 8 && lane == 0 ? (int)__hip_atomic_fetch_add(queue_counter(qx), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    };
    // (wavefront 0) draw `c` of the current queue, or of the next one that has any, becomes entry `pos`
    auto place_draw = [&](int pos, int c) {
        int L = total_tiles;
        while (qx < 8) {
            c = __builtin_amdgcn_readfirstlane(c);
            L = tile_of_draw(qx, c);
            if (L < total_tiles) break;
            bool live = false;  // one look at all counters
            if (lane > qx && lane < 8)
                live = tile_of_draw(lane, (int)__hip_atomic_load(queue_counter(lane), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < total_tiles;
            const uint64_t m = __ballot(live);
            qx = m ? __builtin_ctzll(m) : 8;
            c = draw();
        }
        if (lane == 0) build_entry(pos, qx < 8 ? L : total_tiles);
    };
    struct Tile {
        int w, m0, m_lim, n0;  // w: index of the weights, or of the result
        int row0, rows;        // ragged K: the expert's
        bool alone;            // the weights are read by this tile only
    };
    auto tile_at = [&](int pos) -> Tile {
        const int4 d = list[pos & (kQList - 1)];
        Tile t{__builtin_amdgcn_readfirstlane(d.x), __builtin_amdgcn_readfirstlane(d.y), __builtin_amdgcn_readfirstlane(d.z),
               __builtin_amdgcn_readfirstlane(d.w), 0, 0, false};
        if constexpr (RAGK) {
            t.row0 = t.m_lim;
            t.rows = t.w < 0 ? 0 : __builtin_amdgcn_readfirstlane(t_off[t.w + 1]) - t.row0;
            t.m_lim = g.M;
        } else if constexpr (STREAM) {
            t.alone = t.m_lim < 0;
            t.m_lim = t.alone ? -t.m_lim : t.m_lim;
        }
        return t;
    };

    // ================= issue side: a cursor over the stages of the workgroup's tiles =================
    // A half is 16 chunks of 1 KB, two per wavefront: chunk 2*wave + u.  Row form: rows 8c .. 8c+7, lane -> row 8c + lane/8,
    // slot lane%8.  k-row form: k-rows 4c .. 4c+3, lane -> k-row 4c + lane/16, slot lane%16.
    const int64_t lda = g.lda, ldb = g.ldb;
    const uint32_t lds_wave = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_AS char*)smem + wave * 2048);
    const int nk = RAGK ? 0 : (g.K + TK - 1) / TK;  // k-stages per segment
    // k-stages of a tile.  Ragged K: at least two, so that the cursor, two stages ahead, is never two tiles ahead (what lies
    // past an expert's rows reads zeros, all of it where an expert has no rows)
    auto stages_of = [&](const Tile& t) { return RAGK ? max(2, (t.rows + TK - 1) / TK) : nk * g.nseg; };
    uint32_t a_off[4], b_off[4];  // byte offsets of this lane's pieces (half, chunk) from the tile's bases at k = 0
    const char* sA[2];
    const char* sB[2];            // per segment; DUAL: per matrix
    int ipos = 0, istage = 0, ibuf = 0, itotal = 0, irows = 0;
    bool ialone = false;
    auto cursor_to = [&](const Tile& t) {
        if (t.w < 0) return;  // past the last tile: its first stages once more, which nobody reads
        itotal = stages_of(t);
        irows = t.rows;
        ialone = t.alone;
        const int64_t eoff = RAGK ? (int64_t)t.row0 * ldb : (int64_t)t.w * g.strideB;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int q = s < g.nseg ? s : 0;
            sA[s] = reinterpret_cast<const char*>(static_cast<const bf16_t*>(g.seg[q].A) + (RAGK ? (int64_t)t.row0 * lda + t.m0 : (int64_t)t.m0 * lda));
            const bf16_t* b = static_cast<const bf16_t*>(DUAL && s ? g.seg[0].B2 : g.seg[q].B) + eoff;
            sB[s] = reinterpret_cast<const char*>(BT == 1 ? b + (int64_t)t.n0 * ldb : b + t.n0);
        }
        int ln = lane;
        asm volatile("" : "+v"(ln));  // (what follows is computed per tile and not kept through the main loop)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int c = wave * 2 + u;
                if constexpr (RAGK) {
                    const int q = c * 4 + (ln >> 4);
                    int col = h * 128 + ((ln & 15) ^ swz_krow16(q)) * 8;
                    col = t.m0 + col < g.M ? col : g.M - 8 - t.m0;
                    a_off[2 * h + u] = ((uint32_t)q * (uint32_t)lda + (uint32_t)col) * 2;
                } else {
                    const int r = h * 128 + c * 8 + (ln >> 3), last = t.m_lim - 1 - t.m0;
                    const int rl = r < last ? r : last;  // rows past the expert's end: any valid row (masked at the store)
                    a_off[2 * h + u] = ((uint32_t)rl * (uint32_t)lda + ((ln & 7) ^ swz_rows(r)) * 8) * 2;
                }
                if constexpr (BT == 1) {
                    const int r = h * 128 + c * 8 + (ln >> 3), last = g.N - 1 - t.n0;
                    const int rl = r < last ? r : last;
                    b_off[2 * h + u] = ((uint32_t)rl * (uint32_t)ldb + ((ln & 7) ^ swz_rows(r)) * 8) * 2;
                } else {
                    const int q = c * 4 + (ln >> 4);
                    int col = (DUAL ? 0 : h * 128) + ((ln & 15) ^ swz_krow16(q)) * 8;
                    col = t.n0 + col < g.N ? col : g.N - 8 - t.n0;  // columns past the end: any valid ones
                    b_off[2 * h + u] = ((uint32_t)q * (uint32_t)ldb + (uint32_t)col) * 2;
                }
            }
    };
    // Half `h` of operand A / B at the cursor, chunk u of this wavefront's two.
    auto k_row = [&](int u) { return (wave * 2 + u) * 4 + (lane >> 4); };  // k-row form: this lane's in the stage
    auto zeros = [&]() { return reinterpret_cast<const char*>(kZeroRow) + (lane & 31) * 16; };
    auto issue_a = [&](int h, int u) {
        if constexpr (RAGK) {
            const char* base = sA[0] + (int64_t)istage * TK * lda * 2;
            const uint32_t to = lds_wave + (h ? (ibuf ? kQA1of1 : kQA1of0) : (ibuf ? kQBase1 : kQBase0) + kQA0) + u * 1024;
            const int left = irows - istage * TK;
            if (left >= TK) dma16_s(base, a_off[2 * h + u], to);
            else dma16(k_row(u) < left ? base + a_off[2 * h + u] : zeros(), to);
            return;
        }
        const int sg = istage >= nk ? 1 : 0, k0 = (istage - sg * nk) * TK;
        const char* base = (sg ? sA[1] : sA[0]) + (int64_t)k0 * 2;
        const uint32_t to = lds_wave + (h ? (ibuf ? kQA1of1 : kQA1of0) : (ibuf ? kQBase1 : kQBase0) + kQA0) + u * 1024;
        if (!KREST || k0 + TK <= g.K) {
            dma16_s(base, a_off[2 * h + u], to);
        } else {  // (K is a multiple of 8: a 16-byte piece is inside or outside as a whole)
            const int r = (wave * 2 + u) * 8 + (lane >> 3);
            dma16(((lane & 7) ^ swz_rows(r)) * 8 < g.K - k0 ? base + a_off[2 * h + u] : zeros(), to);
        }
    };
    auto issue_b = [&](int h, int u) {
        if constexpr (RAGK) {
            const char* base = (DUAL ? sB[h] : sB[0]) + (int64_t)istage * TK * ldb * 2;
            const uint32_t to = lds_wave + (ibuf ? kQBase1 : kQBase0) + (h ? kQB1 : kQB0) + u * 1024;
            const int left = irows - istage * TK;
            if (left >= TK) dma16_s(base, b_off[2 * h + u], to);
            else dma16(k_row(u) < left ? base + b_off[2 * h + u] : zeros(), to);
            return;
        }
        const int sg = istage >= nk ? 1 : 0, k0 = (istage - sg * nk) * TK;
        const char* base = (DUAL ? sB[h] : sg ? sB[1] : sB[0]) + (BT == 1 ? (int64_t)k0 * 2 : (int64_t)k0 * ldb * 2);
        const uint32_t to = lds_wave + (ibuf ? kQBase1 : kQBase0) + (h ? kQB1 : kQB0) + u * 1024;
        if (!KREST || k0 + TK <= g.K) {
            if (STREAM && ialone) dma16_s_stream(base, b_off[2 * h + u], to);
            else dma16_s(base, b_off[2 * h + u], to);
        } else {
            const int r = (wave * 2 + u) * 8 + (lane >> 3);
            const int k = BT == 1 ? ((lane & 7) ^ swz_rows(r)) * 8 : k_row(u);
            dma16(k < g.K - k0 ? base + b_off[2 * h + u] : zeros(), to);
        }
    };
    auto advance = [&]() {  // behind the request of A1, a stage's last
        ibuf ^= 1;
        if (++istage == itotal) {
            istage = 0;
            cursor_to(tile_at(++ipos));
        }
    };

    // ================= compute side =================
    const int l16 = lane & 15, kg = lane >> 4;
    const int tr_krow = kg * 8 + (l16 >> 2);          // + ks*32 + t*4: neither changes the swizzle
    const int sw = swz_rows(l16);                     // (repeats every 16 rows)
    const int a_rd = (wm * 64 + l16) * 128 + ((kg ^ sw) << 4);  // + i*16 rows; ks flips bit 2 of the piece
    const int b_rd = (wn * 32 + l16) * 128 + ((kg ^ sw) << 4);
    auto read_tr = [&](const char* half, int col, int ks) -> bf16x8 {  // 16 columns from `col` on
        const char* p = half + tr_krow * 256 + ((((col >> 3) + ((l16 & 3) >> 1)) ^ swz_krow16(tr_krow)) << 4) + (l16 & 1) * 8 + ks * 8192;
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)p);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS_AS bf16x4*)(p + 1024));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto read_a = [&](const char* half, int i, int ks) -> bf16x8 {
        if constexpr (RAGK) return read_tr(half, wm * 64 + i * 16, ks);
        return *reinterpret_cast<const bf16x8*>(half + (a_rd ^ (ks << 6)) + i * 2048);
    };
    auto read_b = [&](const char* half, int j, int ks) -> bf16x8 {
        if constexpr (BT == 1) return *reinterpret_cast<const bf16x8*>(half + (b_rd ^ (ks << 6)) + j * 2048);
        else return read_tr(half, wn * 32 + j * 16, ks);
    };
    auto barrier = [&]() {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    int buf = 0;  // the stage buffer of the tile's first stage
    int pos = 0;  // the tile's entry
    // One tile, of at most 128 rows (HALF) or more.  (The accumulators live in here: shared by both forms they are copied.)
    auto run_tile = [&](auto half_tag, const Tile& t) {
        constexpr bool kHalf = decltype(half_tag)::value != 0;
        f32x4v acc[kHalf ? 4 : 8][4];  // 16 x 16 blocks: rows 4*qm + i, columns 2*qn + j
        bf16x8 fa[4][2], fb[2][2][2];  // [row block of the quadrant][k-step], [column half][column block][k-step]
        // Row block i of quadrant (qm, qn), k-step ks; the pin keeps it between the reads and requests around it.
        auto mma = [&](int qm, int qn, int ks, int i) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                f32x4v& c = acc[4 * qm + i][2 * qn + j];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[qn][j][ks], fa[i][ks], c, 0, 0, 0);
            }
            asm volatile("" : "+v"(acc[4 * qm + i][2 * qn]), "+v"(acc[4 * qm + i][2 * qn + 1])::"memory");
        };
        // A quadrant: eight steps of two MFMAs, `between(ks, i)` behind each
        auto quadrant = [&](int qm, int qn, auto between) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    mma(qm, qn, ks, i);
                    between(ks, i);
                }
        };
        // Fragments of A0 and B0 of the next stage, read behind the last MFMAs that take what they replace.
        auto read_next = [&](const char* nxt, int ks, int i) {
            fa[i][ks] = read_a(nxt + kQA0, i, ks);
            if (i == 3) {
#pragma unroll
                for (int j = 0; j < 2; ++j) fb[0][j][ks] = read_b(nxt + kQB0, j, ks);
            }
        };
        auto stage = [&]() {
            const char* cur = smem + (buf ? kQBase1 : kQBase0);
            const char* a1 = smem + (buf ? kQA1of1 : kQA1of0);
            const char* nxt = smem + (buf ? kQBase0 : kQBase1);
            quadrant(0, 0, [&](int ks, int i) {
                if (i < 2) fb[1][i][ks] = read_b(cur + kQB1, i, ks);
                if (i == 3) issue_a(1, ks);
            });
            advance();
            if constexpr (kHalf) {
                // the two quadrants of A0 alone (A1 is requested and never read).  A0, B0 of the next stage have landed, B1 and A1
                // of it are pending; A0, B0 of this one are free
                asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
                barrier();
                quadrant(0, 1, [&](int ks, int i) {
                    read_next(nxt, ks, i);
                    if (i % 2) {
                        if (ks == 0) issue_a(0, i / 2);
                        else issue_b(0, i / 2);
                    }
                });
                // B1 of the next stage has landed; B1 of this one is free
                asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
                barrier();
                issue_b(1, 0);
                issue_b(1, 1);
            } else {
                asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
                barrier();
                quadrant(0, 1, [&](int ks, int i) {
                    fa[i][ks] = read_a(a1, i, ks);
                    if (i == 3) issue_a(0, ks);
                });
                quadrant(1, 1, [&](int ks, int i) {
                    if (i == 3) issue_b(0, ks);
                });
                asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
                barrier();
                quadrant(1, 0, [&](int ks, int i) {
                    read_next(nxt, ks, i);
                    if (i == 3) issue_b(1, ks);
                });
            }
            buf ^= 1;
        };

        // ---- epilogue of one tile.  A lane holds four consecutive columns of one row: of block (4*qm + i, 2*qn + j) row
        // 128*qm + 64*wm + 16*i + lane%16, columns 128*qn + 32*wn + 16*j + 4*(lane/16) .. +3 (DUAL: qn is the matrix).
        // They go through LDS 64 rows x 128 columns at a time (two row blocks of each wavefront, p = 2*qm + i/2), so that global
        // memory sees 16-byte accesses along rows.
        auto epilogue = [&](const Tile& t, char* stg) {
            // (derived afresh from an opaque copy of the thread's index: recomputed per tile instead of living in registers
            // through the main loop)
            int tid = threadIdx.x;
            asm volatile("" : "+v"(tid));
            const int lane = tid & 63, wave = tid >> 6;
            const int wm = wave >> 2, wn = wave & 3, l16 = lane & 15, kg = lane >> 4;
            const int64_t tile_base = (RAGK ? (int64_t)t.w * g.strideC : 0) + (int64_t)t.m0 * g.ldc + t.n0;
            uint32_t ldc_u = (uint32_t)g.ldc;  // (opaque per tile, or the store offsets are computed once and kept in scratch)
            asm volatile("" : "+s"(ldc_u));
            auto tile_row = [&](int p, int sr) { return (p >> 1) * 128 + (sr >> 5) * 64 + (p & 1) * 32 + (sr & 31); };
            const int sr_w = wm * 32 + l16;  // the staging row this lane writes of the pair's first row block
            if constexpr (EPI == EPI_DH || EPI == EPI_DHP) {
                // dH in fp32 through LDS; then 8 columns per thread: read A, B, write H = silu(A)*B, dA = dH*B*silu'(A),
                // dB = dH*silu(A).  EPI_DHP: the saved pair is P = B*silu'(A), Q = silu(A), dA = dH*P, dB = dH*Q.  Staging rows
                // are 512 B, 16-byte pieces at piece ^ row%32.  The arithmetic bounds this epilogue, so the saved operands of
                // pass q+1 are requested at the top of pass q into a second set of registers.  Every lane loads (dead
                // items from a clamped address) and consumes what it loaded; only the stores are predicated.
                constexpr int IPT = 64 * 16 / kThreads;  // 8-column items per thread and pass
                const int last_row = t.m_lim - 1 - t.m0, last_col = g.N - 8 - t.n0;
                u32x4 pre0[2][IPT], pre1[2][IPT];
                auto load_pass = [&](int q, u32x4 (&p0)[IPT], u32x4 (&p1)[IPT]) {
#pragma unroll
                    for (int u = 0; u < IPT; ++u) {
                        const int item = tid + u * kThreads;
                        const int trow = tile_row(q >> 1, item >> 4), tcol = (q & 1) * 128 + (item & 15) * 8;
                        const int lrow = trow < last_row ? trow : last_row, lcol = tcol < last_col ? tcol : last_col;
                        const uint32_t off = (uint32_t)lrow * ldc_u + (uint32_t)lcol;
                        p0[u] = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(g.S0) + tile_base + off);
                        p1[u] = *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(g.S1) + tile_base + off);
                    }
                };
                {
                    constexpr int NP = kHalf ? 4 : 8;  // pass q: pair of row blocks q/2, column half q%2
                    load_pass(0, pre0[0], pre1[0]);
                    __builtin_amdgcn_sched_barrier(0);  // the loads of pass 0 stay in front of those of pass 1
#pragma unroll
                    for (int q = 0; q < NP; ++q) {
                        const int i = q >> 1, p = q & 1;
                        const bool more = q + 1 < NP;
                        if (more) load_pass(q + 1, pre0[(q + 1) & 1], pre1[(q + 1) & 1]);
#pragma unroll
                        for (int u = 0; u < 2; ++u)
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                const int sr = sr_w + u * 16, piece = (wn * 8 + j * 4 + kg) ^ (sr & 31);
                                *reinterpret_cast<f32x4v*>(stg + sr * 512 + piece * 16) = acc[2 * i + u][2 * p + j];
                            }
                        __syncthreads();
                        // the loads of pass q (builtins, so that the compiler's own bookkeeping of pending loads agrees)
                        if (more) __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
                        else __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0)
#pragma unroll
                        for (int u = 0; u < IPT; ++u) {
                            const int item = tid + u * kThreads;
                            const int sr = item >> 4, cg = item & 15, sw = sr & 31;
                            const int trow = tile_row(i, sr), tcol = p * 128 + cg * 8;
                            const bool live = t.m0 + trow < t.m_lim && t.n0 + tcol < g.N;
                            const uint32_t off = (uint32_t)trow * ldc_u + (uint32_t)tcol;
                            const f32x4v d0 = *reinterpret_cast<const f32x4v*>(stg + sr * 512 + ((2 * cg) ^ sw) * 16);
                            const f32x4v d1 = *reinterpret_cast<const f32x4v*>(stg + sr * 512 + ((2 * cg + 1) ^ sw) * 16);
                            const float dh[8] = {d0[0], d0[1], d0[2], d0[3], d1[0], d1[1], d1[2], d1[3]};
                            const u32x4 av = pre0[q & 1][u], bv = pre1[q & 1][u];
                            u32x4 oh, oa, ob;
#pragma unroll
                            for (int z4 = 0; z4 < 4; ++z4) {
                                float hh[2], da[2], db[2];
#pragma unroll
                                for (int z = 0; z < 2; ++z) {
                                    const float A = __uint_as_float(z ? (av[z4] & 0xFFFF0000u) : (av[z4] << 16));
                                    const float B = __uint_as_float(z ? (bv[z4] & 0xFFFF0000u) : (bv[z4] << 16));
                                    if constexpr (EPI == EPI_DHP) {
                                        da[z] = dh[2 * z4 + z] * A;
                                        db[z] = dh[2 * z4 + z] * B;
                                    } else {
                                        const float sg = sigmoid_f(A);          // one exp and one reciprocal per element
                                        const float sA = A * sg;                // silu(A)
                                        const float gr = sg + sA * (1.0f - sg); // silu'(A) = s (1 + A (1 - s))
                                        hh[z] = sA * B;
                                        da[z] = dh[2 * z4 + z] * B * gr;
                                        db[z] = dh[2 * z4 + z] * sA;
                                    }
                                }
                                if constexpr (EPI == EPI_DH) oh[z4] = pack_bf16x2(hh[0], hh[1]);
                                oa[z4] = pack_bf16x2(da[0], da[1]);
                                ob[z4] = pack_bf16x2(db[0], db[1]);
                            }
                            if (live) {
                                if constexpr (EPI == EPI_DH) *reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C0) + tile_base + off) = oh;
                                *reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C1) + tile_base + off) = oa;
                                *reinterpret_cast<u32x4*>(static_cast<bf16_t*>(g.C2) + tile_base + off) = ob;
                            }
                        }
                        __syncthreads();
                    }
                }
            } else {
                // bf16: a pass fills one of two 16 KB areas with 64 rows of 256 B (16-byte pieces at piece ^ row%16) and leaves
                // as 16 bytes per lane along rows.  The areas take the passes in turn, so one barrier per pass is enough: a
                // wavefront that writes pass p+2 has passed the barrier of pass p+1, which every wavefront reaches only
                // after it has read pass p.
                constexpr int ITEMS = 64 * 16 / kThreads;
                int pn = 0;
                auto pass = [&](int i, auto value, bf16_t* dst, int col0) {
                    char* sb = stg + (pn++ & 1) * 16384;
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            const f32x4v v = value(2 * i + u, j);
                            u32x2 o;
                            o[0] = pack_bf16x2(v[0], v[1]);
                            o[1] = pack_bf16x2(v[2], v[3]);
                            *reinterpret_cast<u32x2*>(sb + (sr_w + u * 16) * 256 + (((wn * 4 + j * 2 + (kg >> 1)) ^ l16) << 4) + (kg & 1) * 8) = o;
                        }
                    __syncthreads();
                    u32x4 v[ITEMS];
#pragma unroll
                    for (int u = 0; u < ITEMS; ++u) {
                        const int item = tid + u * kThreads, sr = item >> 4, pc = item & 15;
                        v[u] = *reinterpret_cast<const u32x4*>(sb + sr * 256 + ((pc ^ (sr & 15)) << 4));
                    }
#pragma unroll
                    for (int u = 0; u < ITEMS; ++u) {
                        const int item = tid + u * kThreads;
                        const int trow = tile_row(i, item >> 4), tcol = col0 + (item & 15) * 8;
                        // (offsets inside a tile fit 32 bits: at most 256 rows of ldc < 2^22 elements)
                        if (t.m0 + trow < t.m_lim && t.n0 + tcol < g.N) {
                            u32x4* to = reinterpret_cast<u32x4*>(dst + tile_base + ((uint32_t)trow * ldc_u + (uint32_t)tcol));
                            if constexpr (STREAM) __builtin_nontemporal_store(v[u], to);
                            else *to = v[u];
                        }
                    }
                };
#pragma unroll
                for (int i = 0; i < (kHalf ? 2 : 4); ++i) {
                    if constexpr (EPI == EPI_SWIGLU) {
                        auto each = [&](auto f) {  // f(a, b) over the four columns
                            return [&, f](int r, int j) {
                                f32x4v v;
#pragma unroll
                                for (int z = 0; z < 4; ++z) v[z] = f(acc[r][j][z], acc[r][2 + j][z]);
                                return v;
                            };
                        };
                        pass(i, each([](float a, float b) { return silu_f(a) * b; }), static_cast<bf16_t*>(g.C0), 0);
                        if (g.S0) {
                            bf16_t* s0 = const_cast<bf16_t*>(static_cast<const bf16_t*>(g.S0));
                            bf16_t* s1 = const_cast<bf16_t*>(static_cast<const bf16_t*>(g.S1));
                            if (g.products) {  // P = b * silu'(a), Q = silu(a)
                                pass(i, each([](float a, float b) {
                                    const float sg = sigmoid_f(a), sA = a * sg;
                                    return b * (sg + sA * (1.0f - sg));
                                }), s0, 0);
                                pass(i, each([](float a, float) { return a * sigmoid_f(a); }), s1, 0);
                            } else {
                                pass(i, each([](float a, float) { return a; }), s0, 0);
                                pass(i, each([](float, float b) { return b; }), s1, 0);
                            }
                        }
                    } else {
                        pass(i, [&](int r, int j) { return acc[r][j]; }, static_cast<bf16_t*>(g.C0), 0);
                        if constexpr (DUAL) pass(i, [&](int r, int j) { return acc[r][2 + j]; }, static_cast<bf16_t*>(g.C1), 0);
                        else pass(i, [&](int r, int j) { return acc[r][2 + j]; }, static_cast<bf16_t*>(g.C0), 128);
                    }
                }
            }
        };

#pragma unroll
        for (int i = 0; i < (kHalf ? 4 : 8); ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = (f32x4v){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) read_next(smem + (buf ? kQBase1 : kQBase0), ks, i);
        const int total = stages_of(t);
        for (int it = 0; it < total; ++it) stage();
        int drawn = 0;
        if constexpr (RAGK)
            if (wave == 0) drawn = draw();  // (arrives under the epilogue)
        // (buf: the buffer of the next tile's first stage; the A1 half that is free is the other one's)
        epilogue(t, smem + (buf ? kQStaging0 : kQStaging1));
        if constexpr (RAGK)
            if (wave == 0) place_draw(pos + 2, drawn);
        // the staging area has been read: the A1 half under it may be requested (ragged K: and the drawn entry is in the list).
        // (The derivative epilogues' last pass ends so.)
        if constexpr (EPI != EPI_DH && EPI != EPI_DHP) __syncthreads();
    };

    // ================= the tiles of this workgroup =================
    Tile t = tile_at(0);
    if (t.w < 0) return;
    cursor_to(t);
    // what the stages before the first would have requested: stage 0, and A0, B0, B1 of stage 1
    auto issue_first = [&]() {
        issue_a(0, 0); issue_a(0, 1);
        issue_b(0, 0); issue_b(0, 1);
        issue_b(1, 0); issue_b(1, 1);
    };
    issue_first();
    issue_a(1, 0); issue_a(1, 1);
    advance();
    issue_first();
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // A0, B0, B1 of stage 0
    barrier();
    for (;;) {
        if (t.m_lim - t.m0 <= TM / 2) run_tile(IntTag<1>{}, t);
        else run_tile(IntTag<0>{}, t);
        ++pos;
        if (!RAGK && (pos & 255) == 128 && pos > 256) {  // the half of the ring that no cursor is in
            const int next = (pos & ~255) + 256 + threadIdx.x;
            if (threadIdx.x < 256) build_entry(next, logical_tile(blockIdx.x + next * gridDim.x));
            __syncthreads();
        }
        t = tile_at(pos);
        if (t.w < 0) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (nothing may land in LDS that is no longer this workgroup's)
}

}  // namespace moe
