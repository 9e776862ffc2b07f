// FSEP parameter layout (paper section 3.1, executor): shard, unshard, reshard for the buffers of N
// ranks held in one device's memory.  Pure data movement: 16-byte pieces, every source read once,
// non-temporal accesses (nothing is reused), index arithmetic per piece.
#include "moe_internal.h"
#include "moe_fsep.h"

namespace moe {

typedef uint32_t fu32x4 __attribute__((ext_vector_type(4)));
constexpr int kFsepMaxSlots = 4096;

// piece index -> (row, piece in row) without 64-bit division in the loop body where it can be avoided
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

// unshard and reshard: a unit of work is up to four passes of 1024 (or 256) consecutive pieces of one chunk, the part of expert e that
// rank n keeps; a workgroup takes one unit (the loop over units is for grids past the launch limit).
// It collects the slots that host e once (ascending order) and then needs no index arithmetic per piece: with a 64-bit
// division per piece and one read of a shard per slot these moved 3.8 and 5.2 TB/s
// (64 experts of 3 x 2048 x 1408 in bf16, 8 ranks of 16 slots: unshard 869 -> 610 us, reshard 629 -> 600 us, 5.4 and 5.5 TB/s).
struct FsepUnits {
    int64_t per_chunk, total;  // units per chunk, units
    int iters;                 // passes per unit; a pass is 256 threads x U pieces, U = 4, or 1 for exchanges of a few MB
};
// as many passes a unit, up to four and evenly, as leave eight units per resident workgroup
static FsepUnits fsep_units(int64_t chunks, int64_t chunk_p, int U) {
    FsepUnits u;
    const int64_t passes = (chunk_p + 256 * U - 1) / (256 * U);
    for (int most = 4;; most /= 2) {
        u.per_chunk = (passes + most - 1) / most;
        u.total = chunks * u.per_chunk;
        u.iters = (int)((passes + u.per_chunk - 1) / u.per_chunk);
        if (most == 1 || u.total >= 16384) return u;
    }
}
// one piece per thread where four would leave compute units without a workgroup (6 experts of 120 KB over 8 ranks:
// unshard 5.2 us with four, 4.4 with one; 34 experts of 370 KB: 14.8 and 16.2)
static bool fsep_narrow(int64_t chunks, int64_t chunk_p) { return chunks * ((chunk_p + 1023) / 1024) < 256; }

// slots hosting e (e == E: those that host no expert), by the first wavefront; every thread calls it
__device__ __forceinline__ int collect_slots(const int32_t* __restrict__ hosted, int n, int e, int E, int32_t* slots,
                                             int32_t* n_slots) {
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        int cnt = 0;
        for (int base = 0; base < n; base += 64) {
            const int q = base + lane;
            bool hit = false;
            if (q < n) {
                const int h = hosted[q];
                hit = e < E ? h == e : (h < 0 || h >= E);
            }
            const uint64_t m = __ballot(hit);
            if (hit) slots[cnt + __popcll(m & ((1ull << lane) - 1ull))] = q;
            cnt += __popcll(m);
        }
        if (lane == 0) *n_slots = cnt;
    }
    __syncthreads();
    return *n_slots;
}

// restored[slot][n] <- shards[n][e] for every slot that hosts e; slots without an expert become zeros
template <int U>
__global__ __launch_bounds__(256) void fsep_unshard_kernel(const fu32x4* __restrict__ shards,
                                                           const int32_t* __restrict__ hosted,
                                                           fu32x4* __restrict__ restored, int N, int E, int C,
                                                           int64_t chunk_p, FsepUnits un) {
    __shared__ int32_t slots[kFsepMaxSlots];
    __shared__ int32_t n_slots;
    for (int64_t unit = blockIdx.x; unit < un.total; unit += gridDim.x) {
        const int64_t chunk = unit / un.per_chunk;
        const int e = (int)(chunk / N), n = (int)(chunk - (int64_t)e * N);
        __syncthreads();  // (the slots of the previous unit are no longer read)
        int64_t v = (unit - chunk * un.per_chunk) * (256 * U * un.iters) + threadIdx.x;
        const fu32x4* src = shards + ((int64_t)n * E + e) * chunk_p;
        fu32x4 val[U];
        auto load = [&]() {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                val[u] = (fu32x4){0u, 0u, 0u, 0u};
                if (e < E && v + 256 * u < chunk_p) val[u] = __builtin_nontemporal_load(&src[v + 256 * u]);
            }
        };
        load();  // (in flight while the slots are looked up)
        const int cnt = collect_slots(hosted, N * C, e, E, slots, &n_slots);
        if (cnt == 0) continue;
        for (int it = 0; it < un.iters && v < chunk_p; ++it, v += 256 * U) {
            if (it > 0) load();
            for (int s = 0; s < cnt; ++s) {
                fu32x4* dst = restored + ((int64_t)slots[s] * N + n) * chunk_p;
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (v + 256 * u < chunk_p) __builtin_nontemporal_store(val[u], &dst[v + 256 * u]);
            }
        }
    }
}

// grad_shards[n][e] <- sum over the slots that host e of grads[slot][n], in fp32 and in ascending slot order
template <class T, int U>
__global__ __launch_bounds__(256) void fsep_reshard_kernel(const fu32x4* __restrict__ grads,
                                                           const int32_t* __restrict__ hosted,
                                                           fu32x4* __restrict__ grad_shards, int N, int E, int C,
                                                           int64_t chunk_p, FsepUnits un) {
    __shared__ int32_t slots[kFsepMaxSlots];
    __shared__ int32_t n_slots;
    for (int64_t unit = blockIdx.x; unit < un.total; unit += gridDim.x) {
        const int64_t chunk = unit / un.per_chunk;
        const int e = (int)(chunk / N), n = (int)(chunk - (int64_t)e * N);
        __syncthreads();  // (the slots of the previous unit are no longer read)
        const int cnt = collect_slots(hosted, N * C, e, E, slots, &n_slots);
        int64_t v = (unit - chunk * un.per_chunk) * (256 * U * un.iters) + threadIdx.x;
        fu32x4* dst = grad_shards + ((int64_t)n * E + e) * chunk_p;
        constexpr int VALS = 16 / sizeof(T);
        for (int it = 0; it < un.iters && v < chunk_p; ++it, v += 256 * U) {
            float acc[U][VALS];
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int z = 0; z < VALS; ++z) acc[u][z] = 0.f;
            for (int s = 0; s < cnt; ++s) {
                const fu32x4* src = grads + ((int64_t)slots[s] * N + n) * chunk_p;
                fu32x4 g[U];
#pragma unroll
                for (int u = 0; u < U; ++u) g[u] = __builtin_nontemporal_load(&src[min(v + 256 * u, chunk_p - 1)]);
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        if constexpr (sizeof(T) == 2) {
                            acc[u][2 * z] += __uint_as_float(g[u][z] << 16);
                            acc[u][2 * z + 1] += __uint_as_float(g[u][z] & 0xFFFF0000u);
                        } else {
                            acc[u][z] += __uint_as_float(g[u][z]);
                        }
                    }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (v + 256 * u >= chunk_p) break;
                fu32x4 out;
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    if constexpr (sizeof(T) == 2) out[z] = pack_bf16x2(acc[u][2 * z], acc[u][2 * z + 1]);
                    else out[z] = __float_as_uint(acc[u][z]);
                }
                __builtin_nontemporal_store(out, &dst[v + 256 * u]);
            }
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

static unsigned fsep_unit_grid(const FsepUnits& un) { return (unsigned)(un.total < (1 << 22) ? un.total : (1 << 22)); }

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
    const int64_t chunks = ((int64_t)E + 1) * N;
    const bool narrow = fsep_narrow(chunks, chunk_p);
    const FsepUnits un = fsep_units(chunks, chunk_p, narrow ? 1 : 4);
    auto kern = narrow ? fsep_unshard_kernel<1> : fsep_unshard_kernel<4>;
    kern<<<fsep_unit_grid(un), 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const fu32x4*>(shards), hosted, static_cast<fu32x4*>(restored), N, E, C, chunk_p, un);
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
    const int64_t chunks = (int64_t)E * N;
    const bool narrow = fsep_narrow(chunks, chunk_p);
    const FsepUnits un = fsep_units(chunks, chunk_p, narrow ? 1 : 4);
    auto kern = dtype == MOE_BF16 ? (narrow ? fsep_reshard_kernel<bf16_t, 1> : fsep_reshard_kernel<bf16_t, 4>)
                                  : (narrow ? fsep_reshard_kernel<float, 1> : fsep_reshard_kernel<float, 4>);
    kern<<<fsep_unit_grid(un), 256, 0, static_cast<hipStream_t>(stream)>>>(
        static_cast<const fu32x4*>(grads), hosted, static_cast<fu32x4*>(grad_shards), N, E, C, chunk_p, un);
    return launch_status(who);
}
