// What comes behind the last layer, for up to 16 rows of up to 1792: final LayerNorm, output projection over the (tied) embedding table and
// greedy choice, in one launch instead of three.
//
// Bound by the table's stream from memory (GPT-2's vocabulary at hidden 1024: 103 MB, 15 us); the LayerNorm and the choice as launches of their own
// leave memory idle for 3 to 5 us each.  One workgroup of eight waves per CU holds the normalised rows in LDS and walks the table in tiles of 16 columns
// per wave.  A tile's 32 KB (K = 1024; longer rows in pieces) are in the wave's registers before they are needed: whole lines per load
// instruction, turned into matrix-operand layout by way of LDS two vectors at a time, and as soon as two are there the next tile's two are requested
// into the same registers.  The rows are normalised while the first tiles are on their way.
// The choice: every lane keeps the best of the columns it writes, the workgroup's best goes out at agent scope, and the last workgroup to
// count itself has all of them to compare (no wait, no fence; it leaves the counter at zero for the next launch).
// us per pass of a prompt and 16 steps with GPT-2's vocabulary, three launches -> this: 24 x hidden 1024, 1 sequence 5336 -> 5198; 4 x 1024, 4 1461 ->
// 1383; 2 x 512, 3 791 -> 676; 1 x 256, 1 511 -> 411; 2 x 1024, 16 1270 -> 1225; 3 x 1536, 12 2345 -> 2229; 2 x 1792, 4 1568 -> 1467.  Where it stops: rows 4 KB
// apart stream slower here than through gemm_stream, whose workgroups start their walk over K in different places (2 x 2048, 2 sequences 1866 -> 1943).
#include <climits>
#include <type_traits>

#include "kernels.hpp"

namespace eet {

namespace {

constexpr int kHWaves = 8, kHThreads = 64 * kHWaves;
constexpr int kHRow = 72;                          // halfs of a staged row: 128 bytes + 16
constexpr int kHStage = 2 * 16 * kHRow;            // of a wave: two units of 16 columns
constexpr int kHNormVec = (kHeadMaxK + 511) / 512; // 16-byte vectors of a row per lane

struct Best {
    float v;
    int i;
};
__device__ __forceinline__ Best better(Best a, Best b) { return b.v > a.v || (b.v == a.v && b.i < a.i) ? b : a; }   // NaN never wins

// U: units of 64 of K that a wave holds at a time, K = 64 * U * pieces (no conditional around a load: the compiler would wait for all of them)
template <int U>
__global__ __launch_bounds__(kHThreads, 2) void head_rows(HeadArgs a) {
    extern __shared__ __attribute__((aligned(16))) half_t head_smem[];
    __shared__ Best sm_best[kHWaves][16];
    __shared__ int sm_last;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 15, G = lane >> 4, wrow = lane >> 3, chunk = lane & 7;
    const int K = a.K, units = K / 64, ldx = K + 8, tiles = a.N / 16;
    half_t* xs = head_smem;                                       // [a.x_rows][ldx]
    half_t* st = head_smem + (size_t)a.x_rows * ldx + wave * kHStage;

    // Steps of this wave: (tile, piece of K)
    const int pieces = units / U, stride = (int)gridDim.x * kHWaves;
    int tile = wave * (int)gridDim.x + (int)blockIdx.x, piece = 0;     // (the waves of a part-filled last turn on as many CUs as there are)
    half8v wf[U][2];
    const uint32_t lane_off = (uint32_t)(wrow * K + chunk * 8) * 2u, half_off = (uint32_t)(8 * K) * 2u;
    auto at = [&](int t, int p) { return reinterpret_cast<const char*>(a.w + (size_t)t * 16 * K + (size_t)p * (U * 64)); };
    auto request = [&](const char* base, int u) {
        wf[u][0] = *reinterpret_cast<const half8v*>(base + u * 128 + lane_off);
        wf[u][1] = *reinterpret_cast<const half8v*>(base + u * 128 + half_off + lane_off);
    };
    if (tile < tiles) {
        const char* base = at(tile, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) request(base, u);
    }

    // ---- the rows, normalised: one wave per row ----
    for (int m = wave; m < a.M; m += kHWaves) {
        const half_t* row = a.x + (size_t)(a.row_map ? a.row_map[m] : m) * K;
        half8v v[kHNormVec], g[kHNormVec], b[kHNormVec];
#pragma unroll
        for (int i = 0; i < kHNormVec; ++i) {
            const int c = (i * 64 + lane) * 8;
            if (c < K) {
                v[i] = *reinterpret_cast<const half8v*>(row + c);
                g[i] = *reinterpret_cast<const half8v*>(a.gamma + c);
                b[i] = *reinterpret_cast<const half8v*>(a.beta + c);
            }
        }
        float sum = 0.f, sq = 0.f;
#pragma unroll
        for (int i = 0; i < kHNormVec; ++i)
            if ((i * 64 + lane) * 8 < K) {
#pragma unroll
                for (int e = 0; e < 8; ++e) sum += (float)v[i][e];
            }
        const float mean = wave_sum(sum) / (float)K;
#pragma unroll
        for (int i = 0; i < kHNormVec; ++i)
            if ((i * 64 + lane) * 8 < K) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = (float)v[i][e] - mean;
                    sq += d * d;
                }
            }
        const float rstd = rsqrtf(wave_sum(sq) / (float)K + a.eps);
#pragma unroll
        for (int i = 0; i < kHNormVec; ++i) {
            const int c = (i * 64 + lane) * 8;
            if (c < K) {
                half8v o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (half_t)(((float)v[i][e] - mean) * rstd * (float)g[i][e] + (float)b[i][e]);
                *reinterpret_cast<half8v*>(&xs[(size_t)m * ldx + c]) = o;
            }
        }
    }
    __syncthreads();

    // ---- the table ----
    Best best{-__builtin_inff(), INT_MAX};
    const half_t* xrow = xs + (size_t)(fr & (a.x_rows - 1)) * ldx + G * 8;     // (rows past M come to columns that nobody writes)
    float4v acc[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
    // one step; AGAIN: the next one's vectors are requested as this one's leave their registers
    auto step = [&](auto again, const char* next) {
        const half_t* xp = xrow + piece * (U * 64);
#pragma unroll
        for (int u = 0; u < U; u += 2) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 2 && u + j < U; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) *reinterpret_cast<half8v*>(&st[(j * 16 + 8 * h + wrow) * kHRow + chunk * 8]) = wf[u + j][h];
            __builtin_amdgcn_wave_barrier();
            if constexpr (decltype(again)::value) {
#pragma unroll
                for (int j = 0; j < 2 && u + j < U; ++j) request(next, u + j);
            }
#pragma unroll
            for (int j = 0; j < 2 && u + j < U; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const half8v w = *reinterpret_cast<const half8v*>(&st[(j * 16 + fr) * kHRow + G * 8 + 32 * h]);
                    const half8v x = *reinterpret_cast<const half8v*>(xp + (u + j) * 64 + 32 * h);
                    acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, x, acc[h], 0, 0, 0);
                }
        }
        if (piece + 1 == pieces) {
            const int n0 = tile * 16 + 4 * G;
            half4v out;
#pragma unroll
            for (int e = 0; e < 4; ++e) out[e] = (half_t)(acc[0][e] + acc[1][e]);
            if (fr < a.M) *reinterpret_cast<half4v*>(a.logits + (size_t)fr * a.N + n0) = out;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n0 + e < a.vocab && (float)out[e] > best.v) best = Best{(float)out[e], n0 + e};     // columns rise: the first of equals stays
            acc[0] = acc[1] = float4v{0.f, 0.f, 0.f, 0.f};
        }
    };
    if (tile < tiles) {
        while (true) {
            const bool done = piece + 1 == pieces;
            const int next_tile = done ? tile + stride : tile, next_piece = done ? 0 : piece + 1;
            if (next_tile >= tiles) break;
            step(std::true_type{}, at(next_tile, next_piece));
            tile = next_tile;
            piece = next_piece;
        }
        step(std::false_type{}, nullptr);
    }
    if (a.next_ids == nullptr) return;

    // ---- the greedy choice ----
    {
        const auto v16 = pair_xor16(best.v);
        const auto i16 = pair_xor16(best.i);
        best = better(Best{v16.lower, i16.lower}, Best{v16.upper, i16.upper});
        const auto v32 = pair_xor32(best.v);
        const auto i32 = pair_xor32(best.i);
        best = better(Best{v32.lower, i32.lower}, Best{v32.upper, i32.upper});
    }
    if (lane < 16) sm_best[wave][lane] = best;
    __syncthreads();
    if (tid < a.M) {
        Best r = sm_best[0][tid];
#pragma unroll
        for (int w = 1; w < kHWaves; ++w) r = better(r, sm_best[w][tid]);
        __hip_atomic_store(a.best + (size_t)tid * gridDim.x + blockIdx.x, (unsigned long long)__builtin_bit_cast(uint32_t, r.v) << 32 | (uint32_t)r.i, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) sm_last = __hip_atomic_fetch_add(a.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1u;
    __syncthreads();
    if (!sm_last) return;
    for (int m = wave; m < a.M; m += kHWaves) {
        Best r{-__builtin_inff(), INT_MAX};
        for (int g = lane; g < (int)gridDim.x; g += 64) {
            const unsigned long long p = __hip_atomic_load(a.best + (size_t)m * gridDim.x + g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r = better(r, Best{__builtin_bit_cast(float, (uint32_t)(p >> 32)), (int)(uint32_t)p});
        }
        const auto v32 = pair_xor32(r.v);
        const auto i32 = pair_xor32(r.i);
        r = better(Best{v32.lower, i32.lower}, Best{v32.upper, i32.upper});
        const auto v16 = pair_xor16(r.v);
        const auto i16 = pair_xor16(r.i);
        r = better(Best{v16.lower, i16.lower}, Best{v16.upper, i16.upper});
        r = better(r, Best{dpp<0x128>(r.v), dpp<0x128>(r.i)});       // the steps of reduce16
        r = better(r, Best{dpp<0x124>(r.v), dpp<0x124>(r.i)});
        r = better(r, Best{dpp<0x4e>(r.v), dpp<0x4e>(r.i)});
        r = better(r, Best{dpp<0xb1>(r.v), dpp<0xb1>(r.i)});
        if (lane == 0) a.next_ids[m] = r.i == INT_MAX ? 0 : r.i;
    }
    if (tid == 0) __hip_atomic_store(a.arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace

// Units of K that a wave holds: all of up to 16, or half of an even number of up to 32
static int head_units(int width) { return width <= 1024 ? width / 64 : width / 128; }
bool head_takes(int rows, int width, int columns) {
    return rows >= 1 && rows <= kHeadMaxRows && width % 64 == 0 && width <= kHeadMaxK && (width <= 1024 || width % 128 == 0) && columns % 16 == 0;
}

hipError_t launch_head(HeadArgs a, hipStream_t s) {
    if (!head_takes(a.M, a.K, a.N)) return hipErrorInvalidValue;
    a.x_rows = a.M <= 1 ? 1 : a.M <= 2 ? 2 : a.M <= 4 ? 4 : a.M <= 8 ? 8 : 16;
    const int groups = (a.N / 16 + kHWaves - 1) / kHWaves;
    const size_t lds = ((size_t)a.x_rows * (a.K + 8) + (size_t)kHWaves * kHStage) * sizeof(half_t);
    const dim3 grid(groups < kHeadGroups ? groups : kHeadGroups), block(kHThreads);
    switch (head_units(a.K)) {
#define EET_HEAD(U) case U: hipLaunchKernelGGL(head_rows<U>, grid, block, lds, s, a); break;
        EET_HEAD(1) EET_HEAD(2) EET_HEAD(3) EET_HEAD(4) EET_HEAD(5) EET_HEAD(6) EET_HEAD(7) EET_HEAD(8)
        EET_HEAD(9) EET_HEAD(10) EET_HEAD(11) EET_HEAD(12) EET_HEAD(13) EET_HEAD(14) EET_HEAD(15) EET_HEAD(16)
#undef EET_HEAD
    }
    return hipGetLastError();
}

}  // namespace eet
