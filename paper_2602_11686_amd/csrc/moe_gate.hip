// Gate of the MoE layer: moe_gate_topk and moe_gate_topk_bwd.
//
// g(x) = Softmax(TopK(x * W_g)) (paper, Preliminary section).  Logits are
// accumulated in fp32 from exact products of the stored values, a per-expert
// bias is added, and the k largest are picked by a wavefront: every lane holds
// the logits of the experts (lane, lane+64, ...), k rounds of a 64-lane
// arg-max (value descending, expert index ascending on ties) pick the slots in
// order, and the softmax runs over the k picked values only.
#include "moe_internal.h"

namespace moe {

// What moe_gate_topk cannot do without (bf16 with d a multiple of 256: the packed gate weight).
static inline size_t gate_needed_bytes(const moe_shape* s) { return align_up((size_t)MOE_MAX_EXPERTS * s->d * 2, 256); }

// ---- short batches: the hidden dimension split over workgroups --------------------------------------------
constexpr int kGateF32Tokens = 16, kGateF32Waves = 8;
static inline int gate_tiles16(int E) { const int n = (E + 15) / 16; return n <= 1 ? 1 : n <= 2 ? 2 : n <= 4 ? 4 : n <= 8 ? 8 : 16; }
// the gate weight in blocks of 16 experts x 16 k-values
static inline size_t gate_pack16_bytes(const moe_shape* s) { return (size_t)((s->d + 15) / 16) * 16 * gate_tiles16(s->E) * 16 * 2; }
static inline bool gate_packed(const moe_shape* s) { return s->dtype == MOE_BF16 && s->d % 256 == 0; }
// Workgroups per token tile: enough for every compute unit, at least 16 values of the hidden dimension per wavefront.  With
// more than 128 experts a workgroup's partial sums (128 KB) leave no room for a second one on its unit, and the few past
// 256 would make a second round (us, whole, rounded up, down; 900 tokens of 4096 x 256: 108, 139, 101; 700 of 8192 x 256:
// 202, 259, 168).  From 33 experts on that costs more than it gives too, where the slices come out even (960 of
// 4096 x 64: 27, 28, 24), but not where they do not (900 of 2056 x 128: 27 and 30, 666 whole; 2000 of 4104 x 8: 20 and 26).
static inline int gate_splits(const moe_shape* s) {
    const int tiles = (s->T + kGateF32Tokens - 1) / kGateF32Tokens;
    const bool one_round = s->E > 128 || (s->E > 32 && gate_packed(s));
    const int want = one_round ? (tiles < 256 ? 256 / tiles : 1) : (256 + tiles - 1) / tiles;
    const int most = (s->d + 16 * kGateF32Waves - 1) / (16 * kGateF32Waves);
    const int n = want < most ? want : most;
    return n < 32 ? n : 32;
}
// Up to how many tokens: a token tile of the kernels that contract the whole hidden dimension takes its 6 to 70 us however few tiles
// there are.  us, whole (with the packing of the weight) and split, 8, 512, 1024, 2048 tokens:
//   bf16 MFMAs: 2048 x 64 experts 8.8, 7.1   10.1, 8.7   10.4, 12.0   10.7, 16.6    4096 x 128 20, 11   22, 17   23, 26   23, 40
//     4096 x 8 8.2, 6.4   10.0, 8.3   10.2, 13.3   10.4, 20.6    2048 x 256 25, 18   28, 28   28, 48   28, 82
//   fp32 MFMAs: fp32, 2048 x 128 34, 9   39, 13   39, 19   40, 27, at 4096 tokens (never split) 43; 1024 x 8 5.6, 5.1   7.0, 5.9   7.0, 7.1   7.4, 7.5
//     bf16, 1096 x 24 15, 7   15, 8   15, 10   16, 14;   2056 x 128 68, 11   66, 15   65, 20   63, 28
// So from some 600 tokens on the bf16 MFMAs would be faster whole.  They are split up to 1024 all the same: the two ways add in different
// orders, so moving the line moves the logits of those batches in their last bits, and now and then a pick among near equals.
static inline size_t gate_split_bytes(const moe_shape* s) {
    return s->T <= (gate_packed(s) ? 1024 : 2048) && gate_splits(s) > 1 ? (size_t)gate_splits(s) * s->T * gate_tiles16(s->E) * 16 * sizeof(float) : 0;
}
size_t gate_workspace_bytes(const moe_shape* s) {
    size_t n = gate_needed_bytes(s);
    for (const size_t b : {align_up(gate_split_bytes(s), 256), align_up(gate_pack16_bytes(s), 256)}) n = n > b ? n : b;
    return n;
}

// ---- bf16 forward on the matrix cores ------------------------------------------------------
// One workgroup = 16 or 32 tokens; each of its wavefronts contracts a part of the hidden dimension for all tokens and all experts,
// with operands straight from global memory: for a 16x16x32 MFMA a lane reads 16 bytes of its token's row, two lanes 32 contiguous
// bytes, and the next MFMA takes the other halves of those lines.  The partial sums meet in LDS and are added in a fixed order,
// then each wavefront runs the top-k of its share of the tokens.
//
// The order of the sums is that of 32x32x16 MFMAs whose lanes hold k and k+32 (which k-values a step takes, how many parts there
// are): logits, and with them the picks among near equals, are the same bit for bit as from those.
//
// What bounds it is reading the tokens and, per workgroup, the whole gate weight (7 to 12 TB/s of both out of L2), and up to some
// 4000 tokens the chain of one workgroup.  Measured (the whole call with the packing of the weight, us; 32 tokens in
// 32x32x16 MFMAs, whose lanes read pieces of 16 bytes 64 bytes apart -> this): 1777 x 4096, 16 experts 19 -> 11; 4096 x 4096, 16 22 -> 13;
// 2048 x 2048, 64 19 -> 11; 8192 x 2048, 64 21 -> 18; 4096 x 2048, 128 45 -> 20; 16384 x 2048, 128 56 -> 47; 16384 x 4096, 8 42 -> 33
// (4.0 TB/s); 16384 x 2048, 160 137 -> 88; 16384 x 6144, 32 58 -> 54, 65536 200 -> 181 (a unit's tokens and weights requested together: 59, 207).
typedef __bf16 gbf16x8 __attribute__((ext_vector_type(8)));
typedef float gf32x4 __attribute__((ext_vector_type(4)));

// The gate weight in the order the MFMA lanes of gate_topk_mfma_kernel consume it ("fragment-major"): the
// 64 lanes x 8 values of one B operand are 1 KB of consecutive memory, so that every operand load of a
// wavefront is one fully coalesced 1 KB read (a plain transposed copy makes each lane read 16 bytes of a
// different row).  Block index: (k-step, expert tile j); inside a block lane (l16, kg) holds expert j*16 + l16 and, of the
// 64-wide chunk step/2, k = (kg%2)*32 + (step%2)*16 + (kg/2)*8 + 0..7.  Experts past E are zero.  A thread writes the 16 bytes of
// one lane (one value each: some 2 us more).
__global__ __launch_bounds__(256) void gate_pack_wg_kernel(const bf16_t* __restrict__ wg, bf16_t* __restrict__ wfrag, int d, int E, int NT) {
    const int64_t n = (int64_t)(d / 32) * NT * 64;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int lane = (int)(i & 63), blk = (int)(i >> 6), kg = lane >> 4;
        const int step = blk / NT, e = (blk - step * NT) * 16 + (lane & 15);
        const int k = (step >> 1) * 64 + (kg & 1) * 32 + ((step & 1) * 2 + (kg >> 1)) * 8;
        bf16_t v[8];
#pragma unroll
        for (int z = 0; z < 8; ++z) v[z] = e < E ? wg[(size_t)(k + z) * E + e] : (bf16_t)0;
        uint4 o;
        o.x = v[0] | (uint32_t)v[1] << 16; o.y = v[2] | (uint32_t)v[3] << 16;
        o.z = v[4] | (uint32_t)v[5] << 16; o.w = v[6] | (uint32_t)v[7] << 16;
        *reinterpret_cast<uint4*>(wfrag + i * 8) = o;
    }
}

template <int N>
struct GateTag {
    static constexpr int value = N;
};

// Maximum over the 64 lanes, returned wave-uniform: DPP row shifts build the maximum of each
// row of 16 in its last lane, two row broadcasts carry it to lane 63.
__device__ __forceinline__ float wave_max_f32(float v) {
#define MOE_DPP_MAX(ctrl, rmask)                                                                              \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v),            \
                                                                       __builtin_bit_cast(int, v), ctrl, rmask, 0xf, false)))
    MOE_DPP_MAX(0x111, 0xf);  // row_shr:1
    MOE_DPP_MAX(0x112, 0xf);  // row_shr:2
    MOE_DPP_MAX(0x114, 0xf);  // row_shr:4
    MOE_DPP_MAX(0x118, 0xf);  // row_shr:8
    MOE_DPP_MAX(0x142, 0xa);  // row_bcast:15 into rows 1 and 3
    MOE_DPP_MAX(0x143, 0xc);  // row_bcast:31 into rows 2 and 3
#undef MOE_DPP_MAX
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// What follows the contraction, in one workgroup of NW wavefronts: part [NP][MT][EP] holds the partial logits of MT
// tokens, added in a fixed order; then top-k and softmax.  A wavefront finishes MT/NW tokens.  part is reused for
// the picked logits ([MT][MOE_MAX_EXPERTS]).
template <int EP, int NP, int NW, int MT>
__device__ __forceinline__ void gate_finish(float* part, const float* __restrict__ bias, int32_t* __restrict__ ids,
                                            float* __restrict__ wout, float* __restrict__ logits_out, int t0, int Tn,
                                            int E, int k) {
    constexpr int TPW = MT / NW;         // tokens finished by each wavefront
    constexpr int NE = (EP + 63) / 64;   // experts per lane
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // wave w finishes tokens TPW*w .. TPW*w + TPW-1; lane owns experts lane, lane+64, ...
    float vals[TPW][NE];
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int row = wave * TPW + i;
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const int e = lane + 64 * j;
            float v = -INFINITY;
            if (e < E) {
                v = part[row * EP + e];
#pragma unroll
                for (int q = 1; q < NP; ++q) v += part[(q * MT + row) * EP + e];  // fixed order
                v += bias ? bias[e] : 0.f;
            }
            vals[i][j] = v;
        }
    }
    __syncthreads();  // partial sums consumed; LDS is reused for the picked logits
    // top-k of the wave's tokens, all their arg-max reductions of a round in flight together
    float* sel = part + wave * TPW * MOE_MAX_EXPERTS;  // [TPW][k]
    if (logits_out) {
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            const int t = t0 + wave * TPW + i;
#pragma unroll
            for (int j = 0; j < NE; ++j)
                if (t < Tn && lane + 64 * j < E) logits_out[(size_t)t * E + lane + 64 * j] = vals[i][j];
        }
    }
    for (int s = 0; s < k; ++s) {
#pragma unroll
        for (int i = 0; i < TPW; ++i) {
            float lv = vals[i][0];
#pragma unroll
            for (int j = 1; j < NE; ++j) lv = fmaxf(lv, vals[i][j]);
            const float m = wave_max_f32(lv);  // uniform
            // lowest expert index holding the maximum: experts are laid out e = lane + 64*j
            int be = -1;
#pragma unroll
            for (int j = NE - 1; j >= 0; --j) {
                const uint64_t bal = __ballot(vals[i][j] == m);
                if (bal) be = 64 * j + __builtin_ctzll(bal);
            }
            if ((unsigned)be >= (unsigned)E) be = 0;  // nothing but NaN left: an index in range all the same
            if ((be & 63) == lane) {
#pragma unroll
                for (int j = 0; j < NE; ++j)
                    if (be == lane + 64 * j) vals[i][j] = -INFINITY;
            }
            const int t = t0 + wave * TPW + i;
            if (lane == 0 && t < Tn) {
                ids[(size_t)t * k + s] = be;
                sel[i * MOE_MAX_EXPERTS + s] = m;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
        const int t = t0 + wave * TPW + i;
        if (t >= Tn) continue;
        const float* sl = sel + i * MOE_MAX_EXPERTS;
        const float m0 = sl[0];
        float z = 0.f;
        for (int s = 0; s < k; ++s) z += __expf(sl[s] - m0);
        for (int s = lane; s < k; s += 64) wout[(size_t)t * k + s] = __expf(sl[s] - m0) / z;
    }
}

// NT expert tiles of 16, MB token tiles of 16, NW wavefronts.  A wavefront goes through its part in pairs of chunks of U units, a unit
// is a k-step and G of the expert tiles; the operands of one chunk are requested before the MFMAs of the other.
template <int NT, int MB, int NW>
__global__ __launch_bounds__(NW * 64) void gate_topk_mfma_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wfrag,
                                                             const float* __restrict__ bias, int32_t* __restrict__ ids,
                                                             float* __restrict__ wout, float* __restrict__ logits_out,
                                                             int Tn, int d, int E, int k) {
    extern __shared__ float part[];  // [NW][MT][EP] partial logits, then the picked logits [MT][MOE_MAX_EXPERTS]
    constexpr int EP = NT * 16, MT = MB * 16, G = NT < 8 ? NT : 8, H = NT / G;
    constexpr int U = NT <= 2 ? 2 : 1;
    constexpr int kSteps = 2 * U / H;  // k-steps of a pair
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const int l16 = lane & 15, kg = lane >> 4;
    const int64_t first = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * MT;
    if (first >= Tn) return;
    const int t0 = (int)first;
    const int ns = d / (32 * NW), pairs = (ns + kSteps - 1) / kSteps;  // of this wavefront's part of the hidden dimension
    const int k_lane = wave * ns * 32 + (kg & 1) * 32 + (kg >> 1) * 8;
    const bf16_t* xa[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) xa[i] = x + (size_t)min(t0 + i * 16 + l16, Tn - 1) * d;
    const bf16_t* wb = wfrag + (size_t)wave * ns * NT * 512 + lane * 8;

    gf32x4 acc[MB][NT];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (gf32x4){0.f, 0.f, 0.f, 0.f};
    gbf16x8 a[2][U][MB], b[2][U][G];
    auto step_of = [&](int p, int c, int u) { return p * kSteps + (c * U + u) / H; };
    // (past the end: any valid addresses, mma leaves them out)
    auto load = [&](int p, auto c_tag) {
        constexpr int c = decltype(c_tag)::value;
        // (all units of a row one after the other: they are halves of the same lines)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int step = min(step_of(p, c, u), ns - 1), kk = k_lane + (step >> 1) * 64 + (step & 1) * 16;
                a[c][u][i] = *reinterpret_cast<const gbf16x8*>(xa[i] + kk);
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int step = min(step_of(p, c, u), ns - 1), h = (c * U + u) % H;
#pragma unroll
            for (int j = 0; j < G; ++j) b[c][u][j] = *reinterpret_cast<const gbf16x8*>(wb + ((size_t)step * NT + h * G + j) * 512);
        }
    };
    auto mma = [&](int p, auto c_tag) {
        constexpr int c = decltype(c_tag)::value;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int step = step_of(p, c, u);
            const int h = (c * U + u) % H;
            if (step >= ns) break;
#pragma unroll
            for (int j = 0; j < G; ++j)
#pragma unroll
                for (int i = 0; i < MB; ++i)
                    acc[i][h * G + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[c][u][i], b[c][u][j], acc[i][h * G + j], 0, 0, 0);
        }
    };
    load(0, GateTag<0>{});
    for (int p = 0; p < pairs; ++p) {
        load(p, GateTag<1>{});
        mma(p, GateTag<0>{});
        if (p + 1 < pairs) load(p + 1, GateTag<0>{});
        mma(p, GateTag<1>{});
    }
    // partial sums -> LDS (accumulator layout: col = lane%16, row = 4*(lane/16) + r)
    float* mine = part + (size_t)wave * MT * EP;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) mine[(i * 16 + kg * 4 + r) * EP + j * 16 + l16] = acc[i][j][r];
    __syncthreads();
    gate_finish<EP, NW, NW, MT>(part, bias, ids, wout, logits_out, t0, Tn, E, k);
}

// Tokens per workgroup: 32 read the weight half as often from L2, 16 fill the chip twice as well.  The whole call in us, 16 tokens
// and 32: 17 to 32 experts, 4096 x 4096 14, 18, 6000 x 6144 33, 30, 8192 x 6144 36, 31, 8192 x 4096 26, 23, 16384 x 6144 63, 53; 64 experts,
// 2048 x 2048 11, 14, 8192 x 2048 18.9, 18.0, 16384 x 4096 58, 48; 128 experts of 2048, 8192 28, 34, 12000 39, 45, 16384 49, 47, of 6144, 16384 120, 92; up to 16 experts
// 1777 x 4096 11, 17, 8192 x 4096 22.7, 22.7, 16384 x 4096 36, 34; more than 128 experts 4096 x 2048 29, 43, 16384 x 2048 91, 93.
// Wavefronts: 8 where every part is whole 64-wide chunks, 4 from 128 padded experts on (their partial sums leave room for fewer
// workgroups on a unit).
static void launch_gate_topk_mfma(const moe_shape* s, const bf16_t* x, const bf16_t* w_gate, const float* bias, int32_t* ids, float* w,
                                  float* logits, bf16_t* wfrag, hipStream_t st) {
    const int NT = gate_tiles16(s->E);
    const int64_t pieces = (int64_t)(s->d / 32) * NT * 64;
    gate_pack_wg_kernel<<<(unsigned)((pieces + 255) / 256 < 2048 ? (pieces + 255) / 256 : 2048), 256, 0, st>>>(w_gate, wfrag, s->d, s->E, NT);
    auto go = [&](auto kern, int mt, int nw) {
        size_t lds = (size_t)nw * mt * NT * 16 * sizeof(float);                                           // partial logits
        if (lds < (size_t)mt * MOE_MAX_EXPERTS * sizeof(float)) lds = (size_t)mt * MOE_MAX_EXPERTS * sizeof(float);
        ensure_dynamic_lds(reinterpret_cast<const void*>(kern), 4 * 32 * MOE_MAX_EXPERTS * sizeof(float));
        constexpr int64_t kMost = 1 << 20;
        const int64_t blocks = ((int64_t)s->T + mt - 1) / mt;
        const dim3 grid = blocks <= kMost ? dim3((unsigned)blocks) : dim3((unsigned)kMost, (unsigned)((blocks + kMost - 1) / kMost));
        kern<<<grid, nw * 64, lds, st>>>(x, wfrag, bias, ids, w, logits, s->T, s->d, s->E, s->k);
    };
    const bool many = s->T >= (NT == 8 ? 16384 : 8192), eight = s->d % 512 == 0;
#define MOE_GATE_LAUNCH(N, W)                             \
    if (many) go(gate_topk_mfma_kernel<N, 2, W>, 32, W);  \
    else go(gate_topk_mfma_kernel<N, 1, W>, 16, W);
    if (NT == 1 && eight) { MOE_GATE_LAUNCH(1, 8) }
    else if (NT == 1) { MOE_GATE_LAUNCH(1, 4) }
    else if (NT == 2 && eight) { MOE_GATE_LAUNCH(2, 8) }
    else if (NT == 2) { MOE_GATE_LAUNCH(2, 4) }
    else if (NT == 4 && eight) { MOE_GATE_LAUNCH(4, 8) }
    else if (NT == 4) { MOE_GATE_LAUNCH(4, 4) }
    else if (NT == 8) { MOE_GATE_LAUNCH(8, 4) }
    else go(gate_topk_mfma_kernel<16, 1, 4>, 16, 4);
#undef MOE_GATE_LAUNCH
}

// ---- fp32, and bf16 with a hidden dimension that the kernel above does not split evenly ------------------
// v_mfma_f32_16x16x4: one workgroup = 16 tokens, eight wavefronts with an eighth of the hidden dimension each, operands
// straight from global memory (a lane reads four consecutive values of its token's row, and the same four rows of
// its expert's column).  The matrix pipe has little to do here; the chain of dependent loads is what costs, so a
// wavefront requests U 16-wide pieces before it uses the first.  bf16 values are widened, which is exact.
// Measured against one lane per expert and a serial walk of the hidden dimension (us): fp32, 2048 tokens x 1024, 8
// experts 200 -> 7; fp32, 256 x 128, 8 experts 33 -> 4; bf16, 4099 x 1096, 24 experts 300 -> 26.
__device__ __forceinline__ gf32x4 gate_load4(const float* p) { return *reinterpret_cast<const gf32x4*>(p); }
__device__ __forceinline__ gf32x4 gate_load4(const bf16_t* p) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    return (gf32x4){__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u), __uint_as_float(u.y << 16),
                    __uint_as_float(u.y & 0xFFFF0000u)};
}

// PACKED: the gate weight (bf16) in the order the lanes consume it: block (16 k-values, expert tile j), lane (l16, kg) holds expert
// j*16 + l16, k = 4*kg .. +3.  One load of 8 bytes per lane and block instead of four of 2 bytes.
// Experts past E and k past d are zero.
__global__ __launch_bounds__(256) void gate_pack16_wg_kernel(const bf16_t* __restrict__ wg, bf16_t* __restrict__ wfrag, int d, int E, int NT) {
    const int64_t n = (int64_t)((d + 15) / 16) * NT * 64;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const int lane = (int)(i & 63), blk = (int)(i >> 6), step = blk / NT;
        const int e = (blk - step * NT) * 16 + (lane & 15), k = step * 16 + (lane >> 4) * 4;
        bf16_t v[4];
#pragma unroll
        for (int z = 0; z < 4; ++z) v[z] = e < E && k < d ? wg[(size_t)(k + z) * E + e] : (bf16_t)0;  // (d is a multiple of four)
        *reinterpret_cast<uint2*>(wfrag + i * 4) = make_uint2(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16);
    }
}

// SPLIT: blockIdx.y picks a slice of the hidden dimension; the sums over the slice go to `slices`
// ([gridDim.y][Tn][NT*16]) and gate_split_finish_kernel does the rest.
//
// ROWS: E fills the expert tiles.  Tile j's column l16 is expert l16*NT + j, so that a lane reads its NT experts of a k-row at once
// (plain: of 64 experts four loads of 2 bytes 32 bytes apart).  The whole call, us: 64 x 2048, 128 experts 11.5 -> 10.6; 512 x 2048, 64
// 10.0 -> 8.6; 1024 x 2048, 64 15.8 -> 12.3; 1024 x 2048, 128 27.1 -> 17.9; 1000 x 4096, 32 21.3 -> 15.7; 300 x 1096, 256 18.2 -> 18.8 (so not
// there).  The same bits.  Against PACKED: gate_pack_pays.
enum { GATE_PLAIN = 0, GATE_PACKED = 1, GATE_ROWS = 2 };
template <class T, int NT, bool SPLIT, int WFORM>  // NT expert tiles of 16
__global__ __launch_bounds__(kGateF32Waves * 64) void gate_topk_f32_kernel(
    const T* __restrict__ x, const T* __restrict__ wg, const float* __restrict__ bias, int32_t* __restrict__ ids,
    float* __restrict__ wout, float* __restrict__ logits_out, float* __restrict__ slices, int Tn, int d, int E, int k) {
    extern __shared__ float part[];  // [waves][16][NT*16] partial logits, then the picked logits
    constexpr int NW = kGateF32Waves, MT = kGateF32Tokens, EP = NT * 16;
    constexpr int U = NT <= 2 ? 4 : NT <= 4 ? 2 : 1;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int l16 = lane & 15, kg = lane >> 4;
    // (a third grid dimension where the first cannot hold the tokens)
    const int64_t first = ((int64_t)blockIdx.z * gridDim.x + blockIdx.x) * MT;
    if (first >= Tn) return;
    const int t0 = (int)first;
    const int trow = min(t0 + l16, Tn - 1);
    const int nw = NW * (SPLIT ? (int)gridDim.y : 1), w = SPLIT ? (int)blockIdx.y * NW + wave : wave;
    const int kq = (d + 16 * nw - 1) / (16 * nw) * 16;
    const int kb = min(w * kq, d), ke = min(kb + kq, d);
    gf32x4 acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[j] = (gf32x4){0.f, 0.f, 0.f, 0.f};
    for (int c = kb; c < ke; c += 16 * U) {
        gf32x4 a[U];
        float b[U][NT][4];
        struct alignas(NT * sizeof(T) < 16 ? NT * sizeof(T) : 16) Row { T v[NT]; };
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int kk = c + u * 16 + kg * 4;  // (d is a multiple of four: four values are inside or outside together)
            const bool in = kk < ke;
            a[u] = (gf32x4){0.f, 0.f, 0.f, 0.f};
            if (in) a[u] = gate_load4(x + (size_t)trow * d + kk);
            if constexpr (WFORM == GATE_ROWS) {
                Row row[4] = {};
#pragma unroll
                for (int z = 0; z < 4; ++z)
                    if (in) row[z] = *reinterpret_cast<const Row*>(wg + (size_t)(kk + z) * EP + l16 * NT);
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int z = 0; z < 4; ++z) b[u][j][z] = Elem<T>::load(&row[z].v[j]);
                continue;
            }
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                const int e = j * 16 + l16;
                if constexpr (WFORM == GATE_PACKED) {
                    gf32x4 v = {0.f, 0.f, 0.f, 0.f};
                    if (in) v = gate_load4(wg + ((size_t)(c / 16 + u) * NT + j) * 256 + lane * 4);
#pragma unroll
                    for (int z = 0; z < 4; ++z) b[u][j][z] = v[z];
                    continue;
                }
#pragma unroll
                for (int z = 0; z < 4; ++z) b[u][j][z] = in && e < E ? Elem<T>::load(wg + (size_t)(kk + z) * E + e) : 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int z = 0; z < 4; ++z)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][z], b[u][j][z], acc[j], 0, 0, 0);
    }
    // accumulator layout: col = lane%16, row = 4*(lane/16) + r
    float* mine = part + (size_t)wave * MT * EP;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(kg * 4 + r) * EP + (WFORM == GATE_ROWS ? l16 * NT + j : j * 16 + l16)] = acc[j][r];
    __syncthreads();
    if constexpr (SPLIT) {
        for (int i = threadIdx.x; i < MT * EP; i += NW * 64) {
            float v = part[i];
#pragma unroll
            for (int q = 1; q < NW; ++q) v += part[q * MT * EP + i];  // fixed order
            if (t0 + i / EP < Tn) slices[((size_t)blockIdx.y * Tn + t0) * EP + i] = v;
        }
    } else {
        gate_finish<EP, NW, NW, MT>(part, bias, ids, wout, logits_out, t0, Tn, E, k);
    }
}

// the slices' sums of four tokens, added in slice order, then top-k and softmax (one wavefront per token)
template <int NT>
__global__ __launch_bounds__(256) void gate_split_finish_kernel(const float* __restrict__ slices, int nslices,
                                                                const float* __restrict__ bias, int32_t* __restrict__ ids,
                                                                float* __restrict__ wout, float* __restrict__ logits_out,
                                                                int Tn, int E, int k) {
    constexpr int EP = NT * 16, MT = 4;
    __shared__ float part[MT * MOE_MAX_EXPERTS];
    const int t0 = blockIdx.x * MT;
    for (int i = threadIdx.x; i < MT * EP; i += 256) {
        const int t = min(t0 + i / EP, Tn - 1);
        float v = 0.f;
#pragma unroll 8
        for (int q = 0; q < nslices; ++q) v += slices[((size_t)q * Tn + t) * EP + i % EP];
        part[i] = v;
    }
    __syncthreads();
    gate_finish<EP, 1, 4, MT>(part, bias, ids, wout, logits_out, t0, Tn, E, k);
}

// Whether the bf16 weight is packed for gate_topk_f32_kernel when the hidden dimension is not split.  Packing is a launch of 2 to 3 us, and what
// it saves grows with the hidden dimension and the tokens; the packed form goes over all of the expert tiles that an instance has, the plain one
// skips those without experts (65 to 80 experts fill 5 of 8).  The whole call in us, plain and packed (tokens x d, experts):
//   one tile: 2049 x 520, 8 7.3, 8.3   4096 x 520 8.3, 8.8   16384 x 520 16.7, 16.2   2049 x 648, 16 8.2, 8.6   3000 x 648 9.2,
//     9.0   2049 x 776, 8 9.2, 9.2   2049 x 904, 12 11.4, 9.8   16384 x 2056 53, 40
//   all of 2, 4, 8 or 16 (or 15): 2049 x 520, 17 10.6, 10.6, 28 10.8, 10.7, 120 25.2, 22.9, 255 49, 39   4099 x 1096, 24 24.3, 18.8
//   7 of 8, 11 to 14 of 16: 2049 x 520, 100 22.4, 23.1, 176 38.6, 39.8   3000 x 520, 100 23.1, 22.8   2049 x 1000, 176 62, 55
//   3 of 4, 6 of 8: 2049 x 776, 48 17.7, 18.4   4096 x 520, 40 14.5, 15.6   2049 x 904, 96 33.2, 31.2   6000 x 520, 96 29.4, 28.8
//   5 of 8: 8192 x 776, 72 36.5, 39.4   2049 x 2056, 72 55, 62   4096 x 2056, 72 64, 63   12000 x 776, 72 69, 67   16384 x 520, 65 55, 52
//   9 or 10 of 16: 4096 x 520, 144 34.9, 40.1   2049 x 1496, 129 75, 82   2049 x 2056, 160 119, 117   6000 x 520, 129 68, 64
// As many experts as the tiles hold (GATE_ROWS needs no packing): 2049 x 520, 32 8.0, 10.7   16384 x 2056, 64 75, 111, 128 132, 175   8200 wide, 128
// 2049 154, 223; but of 32 experts from some 3000 on: 4096 x 3080 33.9, 32.9   2049 x 4104 42.6, 41.0   8192 x 6152 104, 94   (16384 x 4104 131, 133).
static bool gate_pack_pays(const moe_shape* s) {
    const int NT = gate_tiles16(s->E), live = (s->E + 15) / 16;
    if (s->d <= 512) return false;
    if (s->E == NT * 16 && NT > 1 && NT < 16) return NT == 2 && s->d > 3072;
    if (NT == 1) return s->d > 768 || s->T > 8192 || (s->d > 640 && s->T > 2900);
    if (8 * live > 7 * NT) return true;
    if (NT == 8 && live == 5) return (int64_t)s->d * s->T > 7600000;
    if (NT == 16 && live <= 10) return s->d > 2048 || s->T > 4096;
    if (4 * live == 3 * NT && NT < 16) return s->d > 896 || s->T > 4096;
    return (int64_t)s->d * s->T > 1200000;
}

template <class T>
static void launch_gate_topk_f32(const moe_shape* s, const T* x, const T* wg, const float* bias, int32_t* ids, float* w,
                                 float* logits, float* slices, T* wfrag, hipStream_t st) {
    auto go = [&](auto nt_tag) {
        constexpr int NT = decltype(nt_tag)::value;
        size_t lds = (size_t)kGateF32Waves * kGateF32Tokens * NT * 16 * sizeof(float);
        if (lds < (size_t)kGateF32Tokens * MOE_MAX_EXPERTS * sizeof(float)) lds = (size_t)kGateF32Tokens * MOE_MAX_EXPERTS * sizeof(float);
        const unsigned tiles = (unsigned)(((int64_t)s->T + kGateF32Tokens - 1) / kGateF32Tokens), most = 1 << 22;
        const dim3 grid(tiles < most ? tiles : most, slices ? gate_splits(s) : 1, (tiles + most - 1) / most);
        auto kern = slices ? gate_topk_f32_kernel<T, NT, true, GATE_PLAIN> : gate_topk_f32_kernel<T, NT, false, GATE_PLAIN>;
        if constexpr (NT > 1 && NT < 16 && sizeof(T) == 2) {
            if (s->E == NT * 16) kern = slices ? gate_topk_f32_kernel<T, NT, true, GATE_ROWS> : gate_topk_f32_kernel<T, NT, false, GATE_ROWS>;
        }
        const T* w_in = wg;
        if constexpr (sizeof(T) == 2) {
            if (wfrag && !slices && gate_pack_pays(s)) {
                const int64_t blocks = ((int64_t)((s->d + 15) / 16) * NT * 64 + 255) / 256;
                gate_pack16_wg_kernel<<<(unsigned)(blocks < 2048 ? blocks : 2048), 256, 0, st>>>(wg, wfrag, s->d, s->E, NT);
                kern = gate_topk_f32_kernel<T, NT, false, GATE_PACKED>;
                w_in = wfrag;
            }
        }
        ensure_dynamic_lds(reinterpret_cast<const void*>(kern), kGateF32Waves * kGateF32Tokens * MOE_MAX_EXPERTS * 4);
        kern<<<grid, kGateF32Waves * 64, lds, st>>>(x, w_in, bias, ids, w, logits, slices, s->T, s->d, s->E, s->k);
        if (slices)
            gate_split_finish_kernel<NT><<<(s->T + 3) / 4, 256, 0, st>>>(slices, (int)grid.y, bias, ids, w, logits, s->T, s->E, s->k);
    };
    switch (gate_tiles16(s->E)) {
        case 1: go(GateTag<1>{}); break;
        case 2: go(GateTag<2>{}); break;
        case 4: go(GateTag<4>{}); break;
        case 8: go(GateTag<8>{}); break;
        default: go(GateTag<16>{}); break;
    }
}

// ---- backward -----------------------------------------------------------------------

// The gate weight as the dx update reads it, by `blocks` workgroups of 256 threads of which this is number `block`.
// wgT[e][c] = w_gate[c][e] as fp32 (a contiguous read)
template <class T>
__device__ __forceinline__ void gate_transpose(const T* __restrict__ wg, float* __restrict__ wgT, int d, int E, int64_t block,
                                               int blocks) {
    const int64_t n = (int64_t)d * E;
    for (int64_t i = block * 256 + threadIdx.x; i < n; i += (int64_t)blocks * 256) {
        const int e = (int)(i / d), c = (int)(i - (int64_t)e * d);
        wgT[i] = Elem<T>::load(wg + (size_t)c * E + e);
    }
}

// wg_pad[c][j] = w_gate[c][j] for j < E, zero up to n_pad: a [N][K] operand with whole k-stages
__device__ __forceinline__ void gate_pad(const bf16_t* __restrict__ wg, bf16_t* __restrict__ wg_pad, int d, int E, int n_pad,
                                         int64_t block, int blocks) {
    const int64_t n = (int64_t)d * n_pad;
    for (int64_t i = block * 256 + threadIdx.x; i < n; i += (int64_t)blocks * 256) {
        const int c = (int)(i / n_pad), j = (int)(i - (int64_t)c * n_pad);
        wg_pad[i] = j < E ? wg[(size_t)c * E + j] : (bf16_t)0;
    }
}

// dx[t,c] += sum_s dl[t,s] * wgT[ids[t,s]][c]      (4 columns per thread)
// 16 bytes of dx per thread (8 bf16 / 4 fp32 columns); KT > 0: k at compile time, the k gate-weight rows are
// requested together with the dx piece.  d is a multiple of the vector width (checked with the shape).
template <class T, int VEC, int KT>
__global__ __launch_bounds__(256) void gate_bwd_dx_kernel(T* __restrict__ dx, const float* __restrict__ wgT,
                                                          const int32_t* __restrict__ ids,
                                                          const float* __restrict__ dl, int Tn, int d, int k) {
    const int q = d / VEC;
    const int64_t total = (int64_t)Tn * q;
    constexpr int KU = KT > 0 ? KT : 1;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int t = (int)(i / q), c = (int)(i - (int64_t)t * q) * VEC;
        T raw[VEC];
        static_assert(VEC * sizeof(T) == 16, "one 16-byte piece per thread");
        *reinterpret_cast<uint4*>(raw) = *reinterpret_cast<const uint4*>(dx + (size_t)t * d + c);
        float a[VEC];
#pragma unroll
        for (int j = 0; j < VEC; ++j) a[j] = Elem<T>::load(raw + j);
        if constexpr (KT > 0) {
            float g[KU], wv[KU][VEC];
#pragma unroll
            for (int s = 0; s < KU; ++s) {
                g[s] = dl[(size_t)t * KU + s];
                const float* row = wgT + (size_t)ids[(size_t)t * KU + s] * d + c;
#pragma unroll
                for (int j = 0; j < VEC; j += 4) {
                    const float4 v4 = *reinterpret_cast<const float4*>(row + j);
                    wv[s][j] = v4.x; wv[s][j + 1] = v4.y; wv[s][j + 2] = v4.z; wv[s][j + 3] = v4.w;
                }
            }
#pragma unroll
            for (int s = 0; s < KU; ++s)
#pragma unroll
                for (int j = 0; j < VEC; ++j) a[j] = fmaf(g[s], wv[s][j], a[j]);
        } else {
            for (int s = 0; s < k; ++s) {
                const float g = dl[(size_t)t * k + s];
                const float* row = wgT + (size_t)ids[(size_t)t * k + s] * d + c;
#pragma unroll
                for (int j = 0; j < VEC; ++j) a[j] = fmaf(g, row[j], a[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < VEC; ++j) Elem<T>::store(raw + j, a[j]);
        *reinterpret_cast<uint4*>(dx + (size_t)t * d + c) = *reinterpret_cast<const uint4*>(raw);
    }
}

template <class T>
static void launch_gate_bwd_dx(T* dx, const float* wgT, const int32_t* ids, const float* dl, int Tn, int d, int k,
                               hipStream_t st) {
    constexpr int VEC = 16 / sizeof(T);
    const int64_t items = (int64_t)Tn * (d / VEC);
    const int grid = (int)((items + 255) / 256 > 4096 ? 4096 : (items + 255) / 256);
    if (k == 1) gate_bwd_dx_kernel<T, VEC, 1><<<grid, 256, 0, st>>>(dx, wgT, ids, dl, Tn, d, k);
    else if (k == 2) gate_bwd_dx_kernel<T, VEC, 2><<<grid, 256, 0, st>>>(dx, wgT, ids, dl, Tn, d, k);
    else if (k == 4) gate_bwd_dx_kernel<T, VEC, 4><<<grid, 256, 0, st>>>(dx, wgT, ids, dl, Tn, d, k);
    else gate_bwd_dx_kernel<T, VEC, 0><<<grid, 256, 0, st>>>(dx, wgT, ids, dl, Tn, d, k);
}

// ---- dW_g through the grouped GEMM -----------------------------------------------------------
// dL is written out densely (bf16 layers: as two bf16 matrices hi + lo, the pair carries 16 mantissa bits
// of the fp32 value), tokens are cut into chunks, each chunk's X^T * dL is a product of its own,
// and the chunk partials are added in chunk order.
// The product runs on gate_dwg_kernel, but for very many tokens of few columns and many experts on the grouped GEMM: the dense dL
// is the most of what there is to read then, and is read once per 256 columns of x instead of once per 128.
// The whole call, gate_dwg_kernel over the grouped GEMM:
//   tokens                                 65536     131072     262144     524288       2^20
//   65 to 128 experts, d 192 to 1024                0.85-0.97  0.92-1.01  0.94-1.04  0.96-1.07
//   129 to 192 experts, d 192 to 768    0.76-0.96   0.92-1.01  0.99-1.11  1.02-1.16  1.05-1.07
//                       d 1024          0.87-0.90   0.87-0.91  0.96-0.98  1.00-1.01
//   193 to 256 experts, d 192 to 768    0.79-1.01   0.97-1.08  1.05-1.22  1.07-1.28  1.12-1.14
//                       d 1024          0.94-0.96   0.92-0.95  1.02-1.05  1.09-1.13
//   more than 128, d 128                0.74-0.82   0.93-0.95  0.97-0.98  0.97-1.00  0.99-1.01
//                  d 2048 and more      0.82-0.90   0.81-0.90  0.89-0.96  0.97-0.99
// and fewer tokens down to 0.5 (4100 tokens of 1024, 193 experts: 92 -> 45 us).  64 experts and fewer: 0.83 to 0.92.
static inline bool dwg_tokens_once(const moe_shape* s) {
    const bool few_columns = s->d > 128 && s->d <= 1024;
    return !(few_columns && (s->E > 192 ? s->T >= 1 << 17 : s->E > 128 && s->T > 1 << 18));
}
// 512 tokens (or more for very long batches: the GEMM's group table holds MOE_MAX_EXPERTS groups); gate_dwg_kernel: halved
// while its 128 x 64 tiles of all chunks are too few to give every compute unit two
static inline int mma_chunk_tokens(const moe_shape* s) {
    const int need = (s->T + MOE_MAX_EXPERTS - 1) / MOE_MAX_EXPERTS;
    int c = need <= 512 ? 512 : (need + 63) / 64 * 64;
    const int64_t tiles = (int64_t)((s->d + 127) / 128) * ((s->E + 63) / 64);
    while (dwg_tokens_once(s) && c > 64 && c % 128 == 0 && (s->T + c - 1) / c * tiles < 512) c /= 2;
    return c;
}
// fp32: 256 tokens, halved while the 64x64 tiles of all chunks are too few to give every compute unit two
static inline int f32_chunk_tokens(const moe_shape* s) {
    const int64_t tiles = (int64_t)((s->d + 63) / 64) * ((s->E + 63) / 64);
    int c = 256;
    while (c > 32 && (s->T + c - 1) / c * tiles < 512) c /= 2;
    return c;
}
static inline int f32_chunks(const moe_shape* s) { const int c = f32_chunk_tokens(s); return (s->T + c - 1) / c; }
static inline int pad4(int v) { return (v + 3) / 4 * 4; }
static inline int mma_chunks(const moe_shape* s) { const int c = mma_chunk_tokens(s); return (s->T + c - 1) / c; }
static inline int pad16(int v) { return (v + 15) / 16 * 16; }
static inline int pad64(int v) { return (v + 63) / 64 * 64; }  // the dense dL is a K operand: whole 64-wide k-stages

// workgroups in a grid whose first dimension stays below 2^32 threads
static dim3 token_grid(int64_t blocks) {
    constexpr int64_t kMost = 1 << 22;
    return blocks <= kMost ? dim3((unsigned)blocks) : dim3((unsigned)kMost, (unsigned)((blocks + kMost - 1) / kMost));
}

// one wavefront per token: dl[t,s] (fp32, for the dx update) and the dense rows, dl[t,s] = w_s (dw_s - sum_j w_j dw_j);
// D = bf16_t: hi and lo, D = float: hi is the value itself.  It also writes what else the products after it need: the chunks'
// token ranges, a row of zeros, the token range as a single group (in a launch of their own 1.4 us of the 11 that one
// fp32 token takes), and, in kWeightBlocks workgroups behind those of the tokens, the gate weight: padded to n_pad columns
// (wg_pad) or transposed (wgT), whichever is given (a launch of their own: 2 to 5 us).
constexpr int kWeightBlocks = 256;
template <class D>
__global__ __launch_bounds__(256) void gate_dl_dense_kernel(const int32_t* __restrict__ ids, const float* __restrict__ w,
                                                            const float* __restrict__ dw, float* __restrict__ dl,
                                                            D* __restrict__ hi, D* __restrict__ lo, int Tn,
                                                            int k, int n_pad, int32_t* __restrict__ chunk_off, int nchunks,
                                                            int chunk_tokens, uint32_t* __restrict__ zero_row,
                                                            int32_t* __restrict__ whole, const D* __restrict__ w_gate,
                                                            float* __restrict__ wgT, bf16_t* __restrict__ wg_pad, int d, int E) {
    const int lane = threadIdx.x & 63;
    const int64_t block = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;
    const int64_t weight_block = block - ((int64_t)Tn + 3) / 4;
    if (weight_block >= 0 && weight_block < kWeightBlocks) {
        if constexpr (sizeof(D) == 2) {
            if (wg_pad) gate_pad(w_gate, wg_pad, d, E, n_pad, weight_block, kWeightBlocks);
        }
        if (wgT) gate_transpose(w_gate, wgT, d, E, weight_block, kWeightBlocks);
    }
    const int64_t t = block * 4 + (threadIdx.x >> 6);
    const int64_t i = block * 256 + threadIdx.x;  // (at least 256 threads, and 64 for every chunk)
    if (i < 128) zero_row[i] = 0u;
    if (i < 2) whole[i] = (int)i * Tn;
    if (i <= nchunks) chunk_off[i] = (int)min(i * chunk_tokens, (int64_t)Tn);
    if (t >= Tn) return;
    // (lane s holds slot s of the token, 64 slots at a time; the others get them from its registers: loaded again for every 64 experts
    // one slot after the other they cost 19 us for 16384 tokens' top-8 of 128, this 13)
    const size_t at = (size_t)t * k;
    auto slot = [&](int s0, int& id, float& ws, float& ds) {
        const bool in = s0 + lane < k;
        id = in ? ids[at + s0 + lane] : -1;
        ws = in ? w[at + s0 + lane] : 0.f;
        ds = in ? dw[at + s0 + lane] : 0.f;
    };
    auto from = [](float v, int s) { return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), s)); };
    int id0;
    float w0, d0, dot = 0.f;
    slot(0, id0, w0, d0);
    for (int s0 = 0; s0 < k; s0 += 64) {
        int id = id0;
        float ws = w0, ds = d0;
        if (s0 > 0) slot(s0, id, ws, ds);
        for (int s = 0; s < 64 && s0 + s < k; ++s) dot += from(ws, s) * from(ds, s);
    }
    float v[MOE_MAX_EXPERTS / 64] = {};  // of experts lane, lane + 64, ...
    for (int s0 = 0; s0 < k; s0 += 64) {
        int id = id0;
        float ws = w0, ds = d0;
        if (s0 > 0) slot(s0, id, ws, ds);
        const float g = ws * (ds - dot);
        if (s0 + lane < k) dl[at + s0 + lane] = g;
        for (int s = 0; s < 64 && s0 + s < k; ++s) {
            const int e = __builtin_amdgcn_readlane(id, s) - lane;
            const float gs = from(g, s);
#pragma unroll
            for (int j = 0; j < MOE_MAX_EXPERTS / 64; ++j) v[j] = e == 64 * j ? gs : v[j];
        }
    }
#pragma unroll
    for (int j = 0; j < MOE_MAX_EXPERTS / 64; ++j) {
        const int e = lane + 64 * j;
        if (e >= n_pad) break;
        if constexpr (sizeof(D) == 2) {
            const bf16_t h = f32_to_bf16(v[j]);
            hi[(size_t)t * n_pad + e] = h;
            lo[(size_t)t * n_pad + e] = f32_to_bf16(v[j] - bf16_to_f32(h));
        } else {
            hi[(size_t)t * n_pad + e] = v[j];
        }
    }
}

// dw_gate[c][e] = sum over chunks (in chunk order) of partial[chunk][c][e]
__global__ void gate_bwd_dwg_reduce_kernel(const float* __restrict__ partial, float* __restrict__ dwg, int nchunks,
                                               int d, int E, int n_pad) {
    const int64_t n = (int64_t)d * E;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i / E), e = (int)(i - (int64_t)c * E);
        float a = 0.f;
        int ch = 0;
        for (; ch + 8 <= nchunks; ch += 8) {  // eight loads in flight, added in chunk order
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = partial[((size_t)(ch + u) * d + c) * n_pad + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) a += v[u];
        }
        for (; ch < nchunks; ++ch) a += partial[((size_t)ch * d + c) * n_pad + e];
        dwg[i] = a;
    }
}

size_t gate_bwd_workspace_bytes(const moe_shape* s) {
    size_t b = align_up((size_t)pad64(s->E) * s->d * 4, 256);          // wgT (fp32), or the padded bf16 gate weight
    b += align_up((size_t)s->T * s->k * 4, 256);                       // dl
    const bool f32 = s->dtype == MOE_F32;
    const int nch = f32 ? f32_chunks(s) : mma_chunks(s);
    b += align_up((size_t)nch * s->d * (f32 ? pad4(s->E) : pad64(s->E)) * 4, 256);  // partial sums
    b += 2 * align_up((size_t)s->T * pad64(s->E) * 2, 256);             // dense dL, hi and lo (or fp32)
    b += align_up((size_t)(nch + 1) * 4, 256) + 512 + 256;  // token chunk offsets, a row of zeros, {0, T}
    return b;
}

}  // namespace moe

using namespace moe;

extern "C" moe_status moe_gate_topk(const moe_shape* s, const void* x, const void* w_gate, const float* bias,
                                    int32_t* topk_ids, float* topk_w, float* logits_out, void* ws, size_t ws_bytes,
                                    void* stream) {
    const char* who = "moe_gate_topk";
    MOE_RETURN_IF(check_shape(s, who));
    MOE_RETURN_IF(check_ptr(x, "x", who));
    MOE_RETURN_IF(check_ptr(w_gate, "w_gate", who));
    MOE_RETURN_IF(check_ptr(bias, "bias", who, true));
    MOE_RETURN_IF(check_ptr(topk_ids, "topk_ids", who));
    MOE_RETURN_IF(check_ptr(topk_w, "topk_w", who));
    MOE_RETURN_IF(check_ptr(logits_out, "logits_out", who, true));
    hipStream_t st = static_cast<hipStream_t>(stream);
    const bool packed = gate_packed(s);
    if (packed) {
        MOE_RETURN_IF(check_ptr(ws, "ws", who));
        if (ws_bytes < gate_needed_bytes(s)) {
            set_error("%s: workspace %zu < %zu bytes", who, ws_bytes, gate_needed_bytes(s));
            return MOE_ERR_WORKSPACE_TOO_SMALL;
        }
    }
    // (a caller may bring less workspace than moe_workspace_bytes says, or none where it is not needed)
    const size_t split = gate_split_bytes(s);
    float* slices = split && ws && aligned16(ws) && ws_bytes >= split ? static_cast<float*>(ws) : nullptr;
    if (packed && !slices) {
        launch_gate_topk_mfma(s, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w_gate), bias, topk_ids, topk_w, logits_out,
                              static_cast<bf16_t*>(ws), st);
        return launch_status(who);
    }
    if (s->dtype == MOE_BF16)
        launch_gate_topk_f32(s, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w_gate), bias, topk_ids, topk_w,
                             logits_out, slices, ws && aligned16(ws) && ws_bytes >= gate_pack16_bytes(s) ? static_cast<bf16_t*>(ws) : nullptr, st);
    else
        launch_gate_topk_f32(s, static_cast<const float*>(x), static_cast<const float*>(w_gate), bias, topk_ids, topk_w,
                             logits_out, slices, static_cast<float*>(nullptr), st);
    return launch_status(who);
}

template <class T>
static moe_status gate_bwd_launch(const moe_shape* s, const T* x, const T* w_gate, const int32_t* ids,
                                  const float* w, const float* dw, T* dx, float* dwg, void* ws, hipStream_t st) {
    Carver cv(ws);
    float* wgT = static_cast<float*>(cv.take((size_t)pad64(s->E) * s->d * 4));  // fp32 transpose, or the padded bf16 copy
    float* dl = static_cast<float*>(cv.take((size_t)s->T * s->k * 4));
    const bool f32 = sizeof(T) == 4;
    const int n_pad = f32 ? pad4(s->E) : pad64(s->E), nch = f32 ? f32_chunks(s) : mma_chunks(s);
    const int n_out = !f32 && dwg_tokens_once(s) ? pad16(s->E) : n_pad;  // columns of the partial sums
    float* partial = static_cast<float*>(cv.take((size_t)nch * s->d * n_pad * 4));
    T* hi = static_cast<T*>(cv.take((size_t)s->T * n_pad * sizeof(T)));
    T* lo = f32 ? nullptr : static_cast<T*>(cv.take((size_t)s->T * n_pad * sizeof(T)));
    int32_t* coff = static_cast<int32_t*>(cv.take((size_t)(nch + 1) * 4));
    uint32_t* zero_row = static_cast<uint32_t*>(cv.take(512));
    int32_t* whole = static_cast<int32_t*>(cv.take(256));
    const bool dx_gemm = dx && !f32 && s->k >= 4;
    bf16_t* wg_pad = dx_gemm ? reinterpret_cast<bf16_t*>(wgT) : nullptr;
    gate_dl_dense_kernel<T><<<token_grid(((int64_t)s->T + 3) / 4 + (dx ? kWeightBlocks : 0)), 256, 0, st>>>(
        ids, w, dw, dl, hi, lo, s->T, s->k, n_pad, coff, nch, f32 ? f32_chunk_tokens(s) : mma_chunk_tokens(s), zero_row, whole,
        w_gate, dx && !dx_gemm ? wgT : nullptr, wg_pad, s->d, s->E);
    if (dx_gemm) {
        // dx += dL * W_g^T as a GEMM over the dense (hi + lo) dL: reads and writes dx once; the gate
        // weight stays in bf16 (padded to whole k-stages in the space of the fp32 transpose).  The
        // gather form below reads k rows of the fp32 gate weight per token from L2, which is what
        // costs from k = 4 on (measured: k = 8: 54 us against 89 us; k = 2: 93 us against 87 us).
        launch_gate_dx_gemm(hi, lo, wg_pad, whole, s->d, n_pad, dx, st);
    } else if (dx) {
        launch_gate_bwd_dx<T>(dx, wgT, ids, dl, s->T, s->d, s->k, st);
    }
    // (fp32, 256 tokens x 128: 112 us with one thread per column and a serial walk of the tokens, 4 us here;
    // 2048 tokens x 1024: 134 us and 7 us)
    if (f32) launch_gate_dwg_gemm_f32(x, hi, coff, nch, s->d, n_pad, partial, st);
    else if (dwg_tokens_once(s)) launch_gate_dwg(x, hi, lo, coff, nch, s->d, n_pad, n_out, partial, st);
    else launch_gate_dwg_gemm(x, hi, lo, coff, nch, s->d, n_pad, partial, zero_row, st);
    gate_bwd_dwg_reduce_kernel<<<256, 256, 0, st>>>(partial, dwg, nch, s->d, s->E, n_out);
    return launch_status("moe_gate_topk_bwd");
}

extern "C" moe_status moe_gate_topk_bwd(const moe_shape* s, const void* x, const void* w_gate,
                                        const int32_t* topk_ids, const float* topk_w, const float* dtopk_w,
                                        void* dx_inout, float* dw_gate, void* ws, size_t ws_bytes, void* stream) {
    const char* who = "moe_gate_topk_bwd";
    MOE_RETURN_IF(check_shape(s, who));
    MOE_RETURN_IF(check_ptr(x, "x", who));
    MOE_RETURN_IF(check_ptr(w_gate, "w_gate", who));
    MOE_RETURN_IF(check_ptr(topk_ids, "topk_ids", who));
    MOE_RETURN_IF(check_ptr(topk_w, "topk_w", who));
    MOE_RETURN_IF(check_ptr(dtopk_w, "dtopk_w", who));
    MOE_RETURN_IF(check_ptr(dx_inout, "dx_inout", who, true));
    MOE_RETURN_IF(check_ptr(dw_gate, "dw_gate", who));
    MOE_RETURN_IF(check_ptr(ws, "ws", who));
    if (s->dtype == MOE_BF16 && s->d % 8 == 0) MOE_RETURN_IF(check_device(who));  // (this path runs the grouped GEMM)
    if (ws_bytes < gate_bwd_workspace_bytes(s)) {
        set_error("%s: workspace %zu < %zu bytes", who, ws_bytes, gate_bwd_workspace_bytes(s));
        return MOE_ERR_WORKSPACE_TOO_SMALL;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (s->dtype == MOE_BF16)
        return gate_bwd_launch<bf16_t>(s, static_cast<const bf16_t*>(x), static_cast<const bf16_t*>(w_gate), topk_ids,
                                       topk_w, dtopk_w, static_cast<bf16_t*>(dx_inout), dw_gate, ws, st);
    return gate_bwd_launch<float>(s, static_cast<const float*>(x), static_cast<const float*>(w_gate), topk_ids, topk_w,
                                  dtopk_w, static_cast<float*>(dx_inout), dw_gate, ws, st);
}
