// FSEP parameter layout (paper section 3.1, executor): shard, unshard, reshard for the buffers of N
// ranks held in one device's memory.  Pure data movement in 16-byte pieces, with non-temporal accesses.
#include "moe_internal.h"
#include "moe_fsep.h"
#include <algorithm>

namespace moe {

typedef uint32_t fu32x4 __attribute__((ext_vector_type(4)));
constexpr int kFsepMaxSlots = 4096;

// (once per training run: the 64-bit division per piece stays)
__global__ __launch_bounds__(256) void fsep_shard_kernel(const fu32x4* __restrict__ experts, fu32x4* __restrict__ shards,
                                                         int N, int E, int64_t chunk_p) {
    // output piece v = ((n*E + e)*chunk_p + o)  <-  experts[(e*N + n)*chunk_p + o]
    const int64_t total = (int64_t)N * E * chunk_p;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < total; v += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = v / chunk_p, o = v - row * chunk_p;
        const int n = (int)(row / E), e = (int)(row - (int64_t)n * E);
        __builtin_nontemporal_store(__builtin_nontemporal_load(&experts[((int64_t)e * N + n) * chunk_p + o]), &shards[v]);
    }
}

// Unshard is done slot after slot or expert after expert, reshard expert after expert.  What bounds them is HBM (64 experts of
// 3 x 2048 x 1408 in bf16, 8 ranks of 16 slots: 614 and 554 us, 5.4 and 6.0 TB/s), and for exchanges of a few MB the chain of
// dependent loads and, expert after expert, finding the slots again in every workgroup: with a 64-bit division per
// piece and slots looked up 64 at a time by one wavefront, 4096 experts on 32 ranks of 128 slots at 1 KB a shard took
// 777 and 948 us; 46 and 59 now, and 2.3 us instead of 3.3 for 64 experts on 8 ranks of 8 at 112 bytes a shard.
//
// By expert: an expert's pieces are cut into units of 256 x U, one per workgroup (the loop over units is for
// grids past the launch limit).  Where a unit starts among the chunks is one 64-bit division; from there a piece finds its
// chunk by a comparison, or, with chunks shorter than a unit, a 32-bit division.
// One piece per thread where four would leave compute units without a workgroup.
static bool fsep_narrow(int64_t rows, int64_t row_pieces) { return rows * ((row_pieces + 1023) / 1024) < 256; }

// Chunk and place in it of the piece `t` behind place o0 of chunk row0, t < span (the pieces of a unit)
struct ChunkPlace {
    int64_t row, o;
};
__device__ __forceinline__ ChunkPlace chunk_place(int64_t row0, int64_t o0, uint32_t t, int64_t chunk_p, uint32_t span) {
    if (chunk_p >= span) {
        const int64_t o = o0 + t;
        return o < chunk_p ? ChunkPlace{row0, o} : ChunkPlace{row0 + 1, o - chunk_p};
    }
    const uint32_t o = (uint32_t)o0 + t, r = o / (uint32_t)chunk_p;
    return {row0 + r, (int64_t)(o - r * (uint32_t)chunk_p)};
}

// The slots hosting e in ascending order (e == E: those that host no expert).  Up to 64 slots are the bits of a mask, which every
// wavefront forms by itself; more are listed in LDS, where the wavefronts look through a quarter of them each, four
// requests in flight per lane.
struct SlotList {
    int32_t slots[kFsepMaxSlots];
    int32_t counts[4];
    static __device__ __forceinline__ bool hosts(int h, int e, int E) { return e < E ? h == e : (h < 0 || h >= E); }
    // every thread calls it; returns how many there are
    __device__ __forceinline__ int collect(const int32_t* __restrict__ hosted, int n, int e, int E, uint64_t& mask) {
        const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
        if (n <= 64) {
            mask = __ballot(lane < n && hosts(hosted[lane < n ? lane : 0], e, E));
            return __popcll(mask);
        }
        __syncthreads();  // (the slots of the previous unit are no longer read)
        const int steps = (n + 255) / 256, begin = wave * steps * 64;  // <= 16 steps
        uint32_t hits = 0;  // bit i: this lane's slot of step i
        int cnt = 0;
        for (int i0 = 0; i0 < steps; i0 += 4) {
            int h[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = begin + (i0 + u) * 64 + lane;
                h[u] = hosted[q < n ? q : n - 1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int q = begin + (i0 + u) * 64 + lane;
                const bool hit = i0 + u < steps && q < n && hosts(h[u], e, E);
                hits |= (uint32_t)hit << (i0 + u);
                cnt += __popcll(__ballot(hit));
            }
        }
        if (lane == 0) counts[wave] = cnt;
        __syncthreads();
        int pos = 0;
        for (int w = 0; w < wave; ++w) pos += counts[w];
        for (int i = 0; i < steps; ++i) {
            const bool hit = (hits >> i) & 1;
            const uint64_t m = __ballot(hit);
            if (hit) slots[pos + __popcll(m & ((1ull << lane) - 1ull))] = begin + i * 64 + lane;
            pos += __popcll(m);
        }
        __syncthreads();
        return counts[0] + counts[1] + counts[2] + counts[3];
    }
    // the s-th of them (asked for in turn)
    __device__ __forceinline__ int at(int s, int n, uint64_t& mask) const {
        if (n > 64) return slots[s];
        const int q = __builtin_ctzll(mask);
        mask &= mask - 1;
        return q;
    }
};

// restored[slot][n] <- shards[n][hosted[slot]], slot after slot, one piece per thread; slots without an expert become zeros.
// Fewer than 2^32 pieces.
__global__ __launch_bounds__(256) void fsep_unshard_slots_kernel(const fu32x4* __restrict__ shards,
                                                                 const int32_t* __restrict__ hosted,
                                                                 fu32x4* __restrict__ restored, uint32_t N, int E,
                                                                 int64_t pieces, uint32_t chunk_p) {
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < pieces; v += (int64_t)gridDim.x * 256) {
        const uint32_t row = (uint32_t)v / chunk_p, o = (uint32_t)v - row * chunk_p;
        const uint32_t slot = row / N, n = row - slot * N;
        const int e = hosted[slot];
        fu32x4 val = {0u, 0u, 0u, 0u};
        if (e >= 0 && e < E) val = __builtin_nontemporal_load(&shards[((int64_t)n * E + e) * chunk_p + o]);
        __builtin_nontemporal_store(val, &restored[v]);
    }
}

// the same, expert after expert (e == E: the slots without one): each shard read once and stored to every slot that hosts it
template <int U>
__global__ __launch_bounds__(256) void fsep_unshard_experts_kernel(const fu32x4* __restrict__ shards,
                                                                   const int32_t* __restrict__ hosted,
                                                                   fu32x4* __restrict__ restored, int N, int E, int C,
                                                                   int64_t chunk_p) {
    __shared__ SlotList list;
    const int64_t pieces = N * chunk_p, per = (pieces + 256 * U - 1) / (256 * U);  // of one expert
    for (int64_t unit = blockIdx.x; unit < ((int64_t)E + 1) * per; unit += gridDim.x) {
        const int e = (int)(unit / per);
        const int64_t v0 = (unit - e * per) * (256 * U), n0 = v0 / chunk_p, o0 = v0 - n0 * chunk_p;
        fu32x4 val[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {  // (in flight while the slots are looked up)
            const uint32_t t = u * 256 + threadIdx.x;
            val[u] = (fu32x4){0u, 0u, 0u, 0u};
            if (e < E && v0 + t < pieces) {
                const ChunkPlace c = chunk_place(n0, o0, t, chunk_p, 256 * U);
                val[u] = __builtin_nontemporal_load(&shards[(c.row * E + e) * chunk_p + c.o]);
            }
        }
        uint64_t mask = 0;
        const int cnt = list.collect(hosted, N * C, e, E, mask);
        for (int s = 0; s < cnt; ++s) {
            fu32x4* dst = restored + list.at(s, N * C, mask) * pieces;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t v = v0 + u * 256 + threadIdx.x;
                if (v < pieces) __builtin_nontemporal_store(val[u], &dst[v]);
            }
        }
    }
}

// grad_shards[n][e] <- sum over the slots that host e of grads[slot][n], in fp32 and in ascending slot order
template <class T, int U>
__global__ __launch_bounds__(256) void fsep_reshard_kernel(const fu32x4* __restrict__ grads,
                                                           const int32_t* __restrict__ hosted,
                                                           fu32x4* __restrict__ grad_shards, int N, int E, int C,
                                                           int64_t chunk_p) {
    __shared__ SlotList list;
    constexpr int VALS = 16 / sizeof(T);
    constexpr int SB = 8 / U;  // slots whose pieces are requested together
    const int64_t pieces = N * chunk_p, per = (pieces + 256 * U - 1) / (256 * U);  // of one expert
    for (int64_t unit = blockIdx.x; unit < E * per; unit += gridDim.x) {
        const int e = (int)(unit / per);
        const int64_t v0 = (unit - e * per) * (256 * U), n0 = v0 / chunk_p, o0 = v0 - n0 * chunk_p;
        uint64_t mask = 0;
        const int cnt = list.collect(hosted, N * C, e, E, mask);
        float acc[U][VALS];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int z = 0; z < VALS; ++z) acc[u][z] = 0.f;
        for (int s0 = 0; s0 < cnt; s0 += SB) {
            fu32x4 g[SB][U];
#pragma unroll
            for (int b = 0; b < SB; ++b) {
                if (s0 + b >= cnt) break;
                const fu32x4* src = grads + list.at(s0 + b, N * C, mask) * pieces;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    g[b][u] = __builtin_nontemporal_load(&src[min(v0 + u * 256 + threadIdx.x, pieces - 1)]);
            }
#pragma unroll
            for (int b = 0; b < SB; ++b) {
                if (s0 + b >= cnt) break;
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        if constexpr (sizeof(T) == 2) {
                            acc[u][2 * z] += __uint_as_float(g[b][u][z] << 16);
                            acc[u][2 * z + 1] += __uint_as_float(g[b][u][z] & 0xFFFF0000u);
                        } else {
                            acc[u][z] += __uint_as_float(g[b][u][z]);
                        }
                    }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t t = u * 256 + threadIdx.x;
            if (v0 + t >= pieces) break;
            fu32x4 out;
#pragma unroll
            for (int z = 0; z < 4; ++z) {
                if constexpr (sizeof(T) == 2) out[z] = pack_bf16x2(acc[u][2 * z], acc[u][2 * z + 1]);
                else out[z] = __float_as_uint(acc[u][z]);
            }
            const ChunkPlace c = chunk_place(n0, o0, t, chunk_p, 256 * U);
            __builtin_nontemporal_store(out, &grad_shards[(c.row * E + e) * chunk_p + c.o]);
        }
    }
}

static moe_status fsep_check(const char* who, int32_t N, int32_t E, int32_t C, int64_t psi, int32_t dtype) {
    if (dtype != MOE_F32 && dtype != MOE_BF16) {
        set_error("%s: dtype %d is neither MOE_F32 nor MOE_BF16", who, dtype);
        return MOE_ERR_INVALID_ARG;
    }
    const int64_t per_piece = dtype == MOE_BF16 ? 8 : 4;
    if (N < 1 || E < 1 || C < 1 || (int64_t)N * C > kFsepMaxSlots || psi < 1 || psi % (per_piece * N) != 0) {
        set_error("%s: N=%d E=%d C=%d psi=%lld: all >= 1, N*C <= %d, psi a multiple of %lld*N", who, N, E, C,
                  (long long)psi, kFsepMaxSlots, (long long)per_piece);
        return MOE_ERR_INVALID_ARG;
    }
    return MOE_OK;
}

// workgroups of 256 threads for that many: the kernels loop past what a launch can hold
static unsigned fsep_big_grid(int64_t workgroups) { return (unsigned)std::min<int64_t>(workgroups, 1 << 22); }

static int fsep_grid(int64_t pieces) {
    int64_t g = (pieces + 255) / 256;
    return (int)(g > 256 * 16 ? 256 * 16 : (g < 1 ? 1 : g));
}

}  // namespace moe

using namespace moe;

extern "C" moe_status moe_fsep_shard(int32_t N, int32_t E, int64_t psi, int32_t dtype, const void* experts, void* shards,
                                     void* stream) {
    const char* who = "moe_fsep_shard";
    MOE_RETURN_IF(fsep_check(who, N, E, 1, psi, dtype));
    MOE_RETURN_IF(check_ptr(experts, "experts", who));
    MOE_RETURN_IF(check_ptr(shards, "shards", who));
    const int64_t chunk_p = psi / N / (dtype == MOE_BF16 ? 8 : 4);
    fsep_shard_kernel<<<fsep_grid((int64_t)N * E * chunk_p), 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const fu32x4*>(experts), static_cast<fu32x4*>(shards), N, E, chunk_p);
    return launch_status(who);
}

extern "C" moe_status moe_fsep_unshard(int32_t N, int32_t E, int32_t C, int64_t psi, int32_t dtype, const void* shards,
                                       const int32_t* hosted, void* restored, void* stream) {
    const char* who = "moe_fsep_unshard";
    MOE_RETURN_IF(fsep_check(who, N, E, C, psi, dtype));
    MOE_RETURN_IF(check_ptr(shards, "shards", who));
    MOE_RETURN_IF(check_ptr(hosted, "hosted", who));
    MOE_RETURN_IF(check_ptr(restored, "restored", who));
    const int64_t chunk_p = psi / N / (dtype == MOE_BF16 ? 8 : 4);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const fu32x4* from = static_cast<const fu32x4*>(shards);
    fu32x4* to = static_cast<fu32x4*>(restored);
    // By expert where the copies of an expert are worth collecting its slots: half as many slots again as experts, from 16 MB
    // on, and enough distinct pieces for the workgroups.  bf16, slots / experts (us, by slot and by expert): 8 ranks of 8 slots,
    // 64 experts, 1 MB a shard: 173 and 197; of 12 slots: 264 and 250; of 16 slots: 398 and 299; of 16 slots, 16 KB a shard:
    // 8.0 and 6.0; 3 KB a shard: 3.1 and 3.8; 4096 experts on 32 ranks of 128 slots, 1 KB a shard: 46 and 56.
    const int64_t pieces = (int64_t)N * C * N * chunk_p;
    const bool by_expert = (2 * (int64_t)N * C >= 3 * (int64_t)E && pieces >= (1 << 20) && E * N * chunk_p >= (1 << 15)) ||
                           pieces >= (int64_t)1 << 32;
    if (by_expert) {
        const bool narrow = fsep_narrow((int64_t)E + 1, N * chunk_p);
        const int span = narrow ? 256 : 1024;
        auto kern = narrow ? fsep_unshard_experts_kernel<1> : fsep_unshard_experts_kernel<4>;
        kern<<<fsep_big_grid(((int64_t)E + 1) * ((N * chunk_p + span - 1) / span)), 256, 0, st>>>(from, hosted, to, N, E, C, chunk_p);
    } else {
        fsep_unshard_slots_kernel<<<fsep_big_grid((pieces + 255) / 256), 256, 0, st>>>(from, hosted, to, (uint32_t)N, E, pieces,
                                                                                      (uint32_t)chunk_p);
    }
    return launch_status(who);
}

extern "C" moe_status moe_fsep_reshard(int32_t N, int32_t E, int32_t C, int64_t psi, int32_t dtype, const void* grads,
                                       const int32_t* hosted, void* grad_shards, void* stream) {
    const char* who = "moe_fsep_reshard";
    MOE_RETURN_IF(fsep_check(who, N, E, C, psi, dtype));
    if (E > 65535) {
        set_error("%s: E=%d exceeds the grid's second dimension", who, E);
        return MOE_ERR_INVALID_ARG;
    }
    MOE_RETURN_IF(check_ptr(grads, "grads", who));
    MOE_RETURN_IF(check_ptr(hosted, "hosted", who));
    MOE_RETURN_IF(check_ptr(grad_shards, "grad_shards", who));
    const int64_t chunk_p = psi / N / (dtype == MOE_BF16 ? 8 : 4);
    const bool narrow = fsep_narrow(E, N * chunk_p);
    const int span = narrow ? 256 : 1024;
    auto kern = dtype == MOE_BF16 ? (narrow ? fsep_reshard_kernel<bf16_t, 1> : fsep_reshard_kernel<bf16_t, 4>)
                                  : (narrow ? fsep_reshard_kernel<float, 1> : fsep_reshard_kernel<float, 4>);
    kern<<<fsep_big_grid(E * ((N * chunk_p + span - 1) / span)), 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const fu32x4*>(grads), hosted, static_cast<fu32x4*>(grad_shards), N, E, C, chunk_p);
    return launch_status(who);
}
