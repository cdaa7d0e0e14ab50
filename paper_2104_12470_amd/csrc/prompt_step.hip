// Short prompts: all layers of a prefill (or of an encoder pass) in one launch.
//
// A prompt of a few dozen to a few hundred rows through a narrow layer is a chain of phases that each take a microsecond or two of arithmetic,
// and as seven or eight dependent launches per layer each of them costs the floor of a launch (drain, start, first trip to memory: 4 to 5 us).
// Here the chain runs inside one launch, in the manner of decode_step.hip: a workgroup is one ITEM of one layer, takes its number from a counter
// when it starts to run, requests its weights into registers before its input exists, and waits only for items of lower numbers.
//
//   items       QKV: 64 columns of a row tile (16 rows), LayerNorm inside; attention: 128 query rows of a (sequence, head) pair; output
//               projection: as QKV, residual added; first feed-forward projection: LayerNorm inside, GELU; second: 64 columns and a range of at
//               most 1024 of K, whose fp32 sums the last item of a tile to arrive adds up in the order of the ranges.  Two workgroups share a CU
//               (115 registers, 78 KB of LDS), so one's weights arrive while the other waits or computes.
//   hand-over   Rows go through memory at agent scope (relaxed stores and loads, which is what makes them coherent between the XCDs' caches);
//               a producer waits until its stores are acknowledged, then raises a counter of its phase and row tile, and the consumers' first
//               wave polls that counter.  (Words that are their own flags, as in decode_step.hip, save the counter's trip, but here a
//               consumer would poll up to 128 KB.)  Counters only grow: layer l waits for (l + 1) times a layer's count, and the set-up launch
//               in front clears them.
//   reuse       Every buffer is used again in every layer.  What reads rows of tile r in layer l is an ancestor of the last output of layer l in those
//               rows, which every writer of layer l+1 waits for; except the keys and values of an encoder, whose layers share one
//               region: its QKV items also wait for the attention of every tile that shares a sequence with theirs.
//   progress    as in decode_step.hip: no assumption about how many workgroups are resident or what else runs.  The waits are bounded all the
//               same; an item whose wait comes to its bound hands NaN on, which reaches the output, and a prefill says so where its decode steps
//               would (kStepGaveUp, in every group's control words): the lengths come back with an error, and the steps that follow are NaN.
#include "kernels.hpp"

namespace eet {

namespace {

typedef unsigned long long word_t;
constexpr int kAgentScope = 16;                    // cache policy of a buffer access at agent scope: sc1
constexpr int kPWaves = 8, kPThreads = 64 * kPWaves;
constexpr int kPRows = 16;                        // rows of a tile
constexpr int kPRow = 72;                          // halfs of a staged row: 128 bytes + 16
constexpr int kPUnits = kPromptStepK / (64 * kPWaves);   // units of 64 K values a wave holds
constexpr int kPSpinLimit = 1 << 20;               // polls before an item gives up: a tenth of a second at the least
constexpr uint32_t kOutOfRange = 0x7ffffff0u;      // offset of a row that does not exist: a buffer load of it gives zeros
constexpr float kPLog2e = 1.4426950408889634f;

__device__ __forceinline__ uint32_t ld_count(const uint32_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void raise(uint32_t* p, uint32_t n) { __hip_atomic_fetch_add(p, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_agent(half_t* p, half4v v) {
    __hip_atomic_store(reinterpret_cast<word_t*>(p), __builtin_bit_cast(word_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_agent(float* p, float x, float y) {
    __hip_atomic_store(reinterpret_cast<word_t*>(p), __builtin_bit_cast(word_t, float2v{x, y}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a buffer of at most 2 GiB, read at agent scope; loads past its end give zeros
struct AgentBuffer {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ AgentBuffer(const void* p, uint32_t bytes) : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00027000)) {}
    template <class T>
    __device__ __forceinline__ T load16(uint32_t off) const {
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kAgentScope));
    }
};

template <int D>
struct PromptAttnSmem {
    half_t k[2][64 * (D + 8)];
    half_t v[2][64 * (D + 16)];
};
struct PromptSmem {
    static constexpr int kWaveBytes = kPRows * 68 * 4 > 2 * 16 * kPRow * 2 ? kPRows * 68 * 4 : 2 * 16 * kPRow * 2;
    uint32_t word;                                 // number of this item; arrivals at its tile
    int late;                                      // the wait came to its bound
    half_t scale[2][kPromptStepK];                 // of the LayerNorm, and its shift
    float stat[kPRows][kPWaves * 4 + 4];           // [row][wave] sum, mean and squared deviations of the wave's share of the row (+4: rows in other banks)
    union {
        // wave-private: two weight units of 16 rows, a unit of the input (rows of 72 halfs), then the wave's partial tile (rows of 68 floats)
        __attribute__((aligned(16))) char wave[kPWaves][kWaveBytes];
        PromptAttnSmem<64> attn64;
        PromptAttnSmem<128> attn128;
    };
};

struct Spot {                                      // where this item stands
    int layer, lane, wave, tid;
};

// Where a phase's counters lie (a line each): per row tile, and per tile and range of the second feed-forward projection
__device__ __forceinline__ uint32_t* counter(const PromptArgs& a, int row_tile, int which) {
    return a.ctl + (size_t)(1 + row_tile * a.counters + which) * kClearStride;
}
enum { kCntX = 0, kCntQkv = 1, kCntAtt = 2, kCntOut = 3, kCntFfn1 = 4 };   // kCntFfn1 + range, then one per column tile of the merge

// The first wave waits until each of its lanes' counters has come to its target (lanes without one: true); all threads go on together.
template <class Reached>
__device__ __forceinline__ void await(const PromptArgs& a, const Spot& w, int& late, const uint32_t* before, uint32_t at_least, Reached reached) {
    if (w.wave == 0) {
        if (before != nullptr)
            for (int spin = 0; spin < kPSpinLimit; ++spin) {
                if (ld_count(before) >= at_least) break;
                __builtin_amdgcn_s_sleep(16);
            }
        int spin = 0;
        bool ok;
        do {
            ok = __all(reached(w.lane));
            if (!ok) __builtin_amdgcn_s_sleep(1);
        } while (!ok & (++spin < kPSpinLimit));
        if (!ok) {
            if (w.lane == 0) late = 1;
            if (w.lane < a.step.groups) __hip_atomic_fetch_or(a.step.ctl + (size_t)w.lane * a.step.words, (word_t)kStepGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

enum PromptPhase { kPQkv = 0, kPOut = 1, kPFfn1 = 2, kPFfn2 = 3 };

// ---- one item of a projection: 64 columns of a row tile, K in units of 64 dealt round-robin to the waves ----
template <int PH, bool ONCE>
__device__ __forceinline__ void project(const PromptArgs& a, const Spot& w, PromptSmem& sm, int r, int tile, int range) {
    constexpr bool LN = PH == kPQkv || PH == kPFfn1, RES = PH == kPOut || PH == kPFfn2;
    constexpr int U = kPUnits, NT = 4, TR = kPRows, RT = 68, J = TR / 8;
    static_assert(TR * 16 <= kPThreads, "four columns of a row per thread, of the first half of the threads");
    const StepLayer& L = a.layer[w.layer];
    const int H = a.H, K = PH == kPFfn2 ? a.F : H, lane = w.lane, wave = w.wave;
    const bool first = w.layer == 0, last = w.layer == a.n_layers - 1;
    const int u0 = PH == kPFfn2 ? range * a.range_units : 0;                   // units of K of this item: [u0, u0 + units)
    const int units = PH == kPFfn2 ? (u0 + a.range_units < K / 64 ? a.range_units : K / 64 - u0) : K / 64;
    const int n0 = tile * 64, t0 = r * TR;
    const int wrow = lane >> 3, chunk = lane & 7, fr = lane & 15, G = lane >> 4;
    const half_t* weights = PH == kPQkv ? L.w_qkv : PH == kPOut ? L.w_o : PH == kPFfn1 ? L.w_fc1 : L.w_fc2;
    const half_t* bias = PH == kPQkv ? L.b_qkv : PH == kPOut ? L.b_o : PH == kPFfn1 ? L.b_fc1 : L.b_fc2;
    auto has = [&](int i) { return wave + kPWaves * i < units; };
    auto column = [&](int i) { return (u0 + wave + kPWaves * i) * 64 + chunk * 8; };

    // ---- what depends on nothing: weights, bias, scale and shift, places of the rows ----
    half8v wf[U][NT][2];
    const uint32_t lane_off = (uint32_t)(wrow * K + chunk * 8) * 2u;
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (has(i)) {
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const char* row0 = reinterpret_cast<const char*>(weights + (size_t)(n0 + t * 16 + h * 8) * K + (u0 + wave + kPWaves * i) * 64);
                    const half8v* p = reinterpret_cast<const half8v*>(row0 + lane_off);
                    wf[i][t][h] = ONCE ? load_once(p) : *p;
                }
        }
    if constexpr (LN) {
        static_assert(kPThreads / 2 * 8 >= kPromptStepK, "a vector per thread");
        const int c = (w.tid & (kPThreads / 2 - 1)) * 8, which = w.tid >= kPThreads / 2 ? 1 : 0;
        const half_t* src = which == 0 ? (PH == kPQkv ? L.ln1_g : L.ln2_g) : (PH == kPQkv ? L.ln1_b : L.ln2_b);
        if (c < K) *reinterpret_cast<half8v*>(&sm.scale[which][c]) = *reinterpret_cast<const half8v*>(src + c);
    }
    uint32_t off[J];                                                           // of this lane's part of the input rows
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int t = t0 + 8 * j + wrow;
        off[j] = kOutOfRange;
        if (t < a.T) off[j] = (uint32_t)(PH == kPQkv ? a.row_map[t] : t) * (uint32_t)(K * 2);
    }
    // what this thread writes: four columns, from ec on, of row et
    const int et = t0 + w.tid / 16, ec = n0 + (w.tid & 15) * 4;
    half4v eb, er;
    int place = -1;                                                            // row of the padded layout
    const int which = n0 / H, c0 = n0 - which * H;                             // Q, K or V; its first column
    size_t slot = 0;                                                           // where in the cache the row's keys or values go
    if (w.tid < TR * 16 && et < a.T) {
        eb = *reinterpret_cast<const half4v*>(bias + ec);
        place = PH == kPFfn1 ? et : a.row_map[et];
        if constexpr (PH == kPQkv) {
            const int b = place / a.S, col = c0 + (w.tid & 15) * 4;
            int pos = place - b * a.S;
            if (a.left_pad) pos -= a.S - a.lens[b];
            slot = ((size_t)(b * a.heads + col / a.d) * a.max_seq + pos) * a.d + col % a.d;
        }
    }
    // of the LayerNorm: the size of this wave's share of a row and of the one that this lane merges (worked out here: behind the wait they are in the chain)
    static_assert(kPWaves == 8, "a share per lane of a row");
    float inv_k, inv_share, weight;
    if constexpr (LN) {
        auto share = [&](int v) { return (float)(v < units ? 64 * ((units - v + kPWaves - 1) / kPWaves) : 0); };
        inv_k = 1.0f / (float)K;
        inv_share = wave < units ? __builtin_amdgcn_rcpf(share(wave)) : 0.f;     // a power of two, or rounded once: any value near the mean serves
        weight = share(chunk);
        asm volatile("" : "+v"(inv_k), "+v"(inv_share), "+v"(weight));
    }
    // weights into matrix-operand layout by way of LDS (whole lines per load instruction), two 16-row units at a time
    half_t* st = reinterpret_cast<half_t*>(sm.wave[wave]);
#pragma unroll
    for (int q = 0; q < U * NT; q += 2) {
        if (has(q / NT)) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) *reinterpret_cast<half8v*>(&st[(j * 16 + 8 * h + wrow) * kPRow + chunk * 8]) = wf[q / NT][(q + j) % NT][h];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int h = 0; h < 2; ++h) wf[q / NT][(q + j) % NT][h] = *reinterpret_cast<const half8v*>(&st[(j * 16 + fr) * kPRow + G * 8 + 32 * h]);
            __builtin_amdgcn_wave_barrier();
        }
    }

    // ---- the input ----
    const uint32_t lay = (uint32_t)w.layer, next = lay + 1u;
    if constexpr (PH == kPQkv) {
        if (!first) {
            int lo = r, hi = r;
            if (!a.causal) {                                                   // the layer before may still read this region in other tiles of the same sequences
                const int end = t0 + TR < a.T ? t0 + TR : a.T;
                lo = a.cu[a.row_map[t0] / a.S] / TR;
                hi = (a.cu[a.row_map[end - 1] / a.S + 1] - 1) / TR;
            }
            await(a, w, sm.late, counter(a, r, kCntFfn1), lay * (uint32_t)(a.range_units), [&](int i) {
                bool ok = true;
                if (i == 0) ok = ld_count(counter(a, r, kCntX)) >= lay * (uint32_t)(H / 64);
                const int o = lo + i;
                if (!a.causal && o <= hi) {
                    const int rows = a.T - o * TR < TR ? a.T - o * TR : TR;
                    ok &= ld_count(counter(a, o, kCntAtt)) >= lay * (uint32_t)(a.heads * rows);
                }
                return ok;
            });
        }
    } else if constexpr (PH == kPOut) {
        const int rows = a.T - t0 < TR ? a.T - t0 : TR;
        await(a, w, sm.late, counter(a, r, kCntQkv), next * (uint32_t)(3 * H / 64), [&](int i) { return i != 0 || ld_count(counter(a, r, kCntAtt)) >= next * (uint32_t)(a.heads * rows); });
    } else if constexpr (PH == kPFfn1) {
        const int rows = a.T - t0 < TR ? a.T - t0 : TR;
        await(a, w, sm.late, counter(a, r, kCntAtt), next * (uint32_t)(a.heads * rows), [&](int i) { return i != 0 || ld_count(counter(a, r, kCntOut)) >= next * (uint32_t)(H / 64); });
    } else {
        await(a, w, sm.late, counter(a, r, kCntOut), next * (uint32_t)(H / 64), [&](int i) { return i != 0 || ld_count(counter(a, r, kCntFfn1 + range)) >= next * (uint32_t)units; });
    }
    __syncthreads();
    const float poison = sm.late != 0 ? __builtin_nanf("") : 0.f;
    const half_t* rows_in = PH == kPQkv ? (first ? a.tokens : a.x) : PH == kPOut ? a.ctx : PH == kPFfn1 ? a.y : a.f;
    const AgentBuffer in(rows_in, (uint32_t)(PH == kPQkv ? a.padded_rows : a.T) * (uint32_t)(K * 2));
    half8v xv[U][J];
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (has(i)) {
#pragma unroll
            for (int j = 0; j < J; ++j) xv[i][j] = in.load16<half8v>(off[j] == kOutOfRange ? kOutOfRange : off[j] + (uint32_t)column(i) * 2u);
        }
    if constexpr (RES) {
        const half_t* res = PH == kPOut ? (first ? a.tokens : a.x) : a.y;
        if (place >= 0)
            er = __builtin_bit_cast(half4v, __hip_atomic_load(reinterpret_cast<const word_t*>(res + (size_t)(PH == kPOut ? place : et) * H + ec), __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT));
    }

    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if constexpr (LN) {
        // Sum and squared deviations of the wave's share of each row, then of the row (shares merged by their sizes).  As in the LayerNorm's own launches
        // the mean is one sum, divided once, and is taken from the values before anything else: a row far from zero loses no bits (x * rstd - mean *
        // rstd, an instruction less per value, has an error of 2e-5 deviations where the mean is a thousand of them).
#pragma unroll
        for (int j = 0; j < J; ++j) {
            float sum = 0.f, sq = 0.f;
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (has(i)) {
#pragma unroll
                    for (int e = 0; e < 8; e += 2) sum = __builtin_amdgcn_fdot2(half2v{xv[i][j][e], xv[i][j][e + 1]}, half2v{(half_t)1.f, (half_t)1.f}, sum, false);
                }
            sum = sum8(sum);
            const float mw = sum * inv_share;
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (has(i)) {
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        float d0, d1;
                        const half2v x2 = half2v{xv[i][j][e], xv[i][j][e + 1]};
                        minus_mean(x2, mw, d0, d1);
                        sq = __builtin_fmaf(d0, d0, sq);
                        sq = __builtin_fmaf(d1, d1, sq);
                    }
                }
            sq = sum8(sq);
            if (chunk == 0) *reinterpret_cast<float4v*>(&sm.stat[8 * j + wrow][wave * 4]) = float4v{sum, mw, sq, 0.f};
        }
        __syncthreads();
        // eight lanes per row, a wave's share each
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const float4v sv = *reinterpret_cast<const float4v*>(&sm.stat[8 * j + wrow][chunk * 4]);
            const float mean = mean_of(sum8(sv[0]), K, inv_k), d = sv[1] - mean, m2 = sum8(sv[2] + weight * d * d);
            const float rstd = rsqrtf(m2 * inv_k + a.eps);
#pragma unroll
            for (int i = 0; i < U; ++i)
                if (has(i)) {
                    const half8v gv = *reinterpret_cast<const half8v*>(&sm.scale[0][column(i)]), bv = *reinterpret_cast<const half8v*>(&sm.scale[1][column(i)]);
#pragma unroll
                    for (int e = 0; e < 8; e += 2) {
                        float d0, d1;
                        const half2v x2 = half2v{xv[i][j][e], xv[i][j][e + 1]};
                        minus_mean(x2, mean, d0, d1);
                        xv[i][j][e] = (half_t)__builtin_fmaf(d0 * rstd, (float)gv[e], (float)bv[e]);
                        xv[i][j][e + 1] = (half_t)__builtin_fmaf(d1 * rstd, (float)gv[e + 1], (float)bv[e + 1]);
                    }
                }
        }
    }

    // ---- contraction: acc[t][c] = output column n0 + 16t + 4G + c of row fr ----
    float4v acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < U; ++i)
        if (has(i)) {
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < J; ++j) *reinterpret_cast<half8v*>(&st[(8 * j + wrow) * kPRow + chunk * 8]) = xv[i][j];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const half8v xf = *reinterpret_cast<const half8v*>(&st[fr * kPRow + G * 8 + 32 * h]);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[i][t][h], xf, acc[t], 0, 0, 0);
            }
        }
    __builtin_amdgcn_wave_barrier();
    float* red = reinterpret_cast<float*>(sm.wave[wave]);
#pragma unroll
    for (int t = 0; t < NT; ++t) *reinterpret_cast<float4v*>(&red[fr * RT + 16 * t + 4 * G]) = acc[t];
    __syncthreads();
    float4v v = float4v{poison, poison, poison, poison};
    if (place >= 0) {
#pragma unroll
        for (int o = 0; o < kPWaves; ++o)
            if (o < units) v += *reinterpret_cast<const float4v*>(reinterpret_cast<const float*>(sm.wave[o]) + (w.tid / 16) * RT + (w.tid & 15) * 4);
    }
    if constexpr (PH == kPFfn2) {
        if (a.ranges > 1) {
            // the sums of this range, then, by whoever is the last to come, of all of them in their order
            float* part = a.part + ((size_t)(r * (H / 64) + tile) * a.ranges) * (TR * 64);
            if (place >= 0) {
                float* p = part + (size_t)range * (TR * 64) + w.tid * 4;
                st_agent(p, v[0], v[1]);
                st_agent(p + 2, v[2], v[3]);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (w.tid == 0) sm.word = __hip_atomic_fetch_add(counter(a, r, kCntFfn1 + a.ranges + tile), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            if (sm.word != next * (uint32_t)a.ranges - 1u) return;
            const AgentBuffer sums(part, (uint32_t)a.ranges * (TR * 64 * 4));
            if (place >= 0) {
                v = float4v{0.f, 0.f, 0.f, 0.f};
                for (int s = 0; s < a.ranges; ++s) v += sums.load16<float4v>((uint32_t)(s * TR * 64 + w.tid * 4) * 4u);
            }
        }
    }
    if (place >= 0) {
        half4v out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float f = v[e] + (float)eb[e];
            if (PH == kPFfn1) f = gelu_tanh(f);
            if (RES) f += (float)er[e];
            out[e] = (half_t)f;
        }
        if constexpr (PH == kPQkv) {
            if (which == 0) st_agent(a.q + (size_t)et * H + ec, out);
            else st_agent((which == 1 ? L.k_cache : L.v_cache) + slot, out);
        } else if constexpr (PH == kPOut) {
            st_agent(a.y + (size_t)et * H + ec, out);
        } else if constexpr (PH == kPFfn1) {
            st_agent(a.f + (size_t)et * a.F + ec, out);
        } else {
            if (last) *reinterpret_cast<half4v*>(a.out + (size_t)place * H + ec) = out;
            else st_agent(a.x + (size_t)place * H + ec, out);
        }
    }
    if (PH == kPFfn2 && last) return;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (w.tid == 0) raise(counter(a, r, PH == kPQkv ? kCntQkv : PH == kPOut ? kCntOut : PH == kPFfn1 ? kCntFfn1 + tile / a.range_units : kCntX), 1u);
}

// ---- 128 query rows of a (sequence, head) pair: the arithmetic of attn_prefill16 (attention.hip), 16 rows per wave ----
template <int D>
__device__ __forceinline__ void attend(const PromptArgs& a, const Spot& w, PromptSmem& base, int b, int g, int block) {
    constexpr int BKV = 64, KK = D / 32, DB = D / 16, LDK = D + 8, LDV = D + 16, CH = D / 8, VEC = BKV * CH / kPThreads, TR = kPRows, BQ = 16 * kPWaves;
    PromptAttnSmem<D>& sm = *reinterpret_cast<PromptAttnSmem<D>*>(base.wave[0]);
    const StepLayer& L = a.layer[w.layer];
    const int row0 = a.cu[b], len = a.cu[b + 1] - row0, i0 = block * BQ;
    if (i0 >= len) return;
    const int lane = w.lane, fr = lane & 15, G = lane >> 4, iw0 = i0 + w.wave * 16, i = iw0 + fr;
    const bool row_ok = i < len;
    const int rows = len - i0 < BQ ? len - i0 : BQ;                           // query rows of this item
    const int keys = a.causal ? i0 + rows : len;                              // keys it looks at
    const int lo = row0 / TR, hi = (row0 + (a.causal ? keys : len) - 1) / TR; // row tiles they and the queries lie in
    const uint32_t target = (uint32_t)(w.layer + 1) * (uint32_t)(3 * a.H / 64);
    await(a, w, base.late, w.layer == 0 ? nullptr : counter(a, hi, kCntX), (uint32_t)w.layer * (uint32_t)(a.H / 64), [&](int l) { return lo + l > hi || ld_count(counter(a, lo + l, kCntQkv)) >= target; });
    __syncthreads();
    const float c = base.late != 0 ? __builtin_nanf("") : rsqrtf((float)D) * kPLog2e;
    const AgentBuffer qb(a.q, (uint32_t)a.T * (uint32_t)(a.H * 2));
    const size_t head = ((size_t)b * a.heads + g) * a.max_seq * D;
    const AgentBuffer kb_(L.k_cache + head, (uint32_t)len * (D * 2)), vb_(L.v_cache + head, (uint32_t)len * (D * 2));
    const int ntiles = (keys + BKV - 1) / BKV;
    half8v rk[VEC], rv[VEC];
    auto gload = [&](int jt) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const int idx = w.tid + v * kPThreads;
            int jr = jt * BKV + idx / CH;
            jr = jr < len ? jr : len - 1;
            const uint32_t o = (uint32_t)(jr * D + idx % CH * 8) * 2u;
            rk[v] = kb_.load16<half8v>(o);
            rv[v] = vb_.load16<half8v>(o);
        }
    };
    auto sstore = [&](int buf) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            const int idx = w.tid + v * kPThreads, row = idx / CH, ch = idx % CH;
            *reinterpret_cast<half8v*>(&sm.k[buf][row * LDK + ch * 8]) = rk[v];
            *reinterpret_cast<half8v*>(&sm.v[buf][row * LDV + ch * 8]) = rv[v];
        }
    };
    gload(0);
    half8v qf[KK];
    {
        const uint32_t o = ((uint32_t)(row0 + (row_ok ? i : len - 1)) * (uint32_t)a.H + (uint32_t)(g * D + G * 8)) * 2u;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qf[kk] = qb.load16<half8v>(o + kk * 64);
    }
    float4v o[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) o[db] = float4v{0.f, 0.f, 0.f, 0.f};
    float m = -INFINITY, l = 0.f;
    sstore(0);
    __syncthreads();
    for (int jt = 0; jt < ntiles; ++jt) {
        const int buf = jt & 1, j0 = jt * BKV;
        if (jt + 1 < ntiles) gload(jt + 1);
        if (iw0 < len && !(a.causal && j0 > iw0 + 15)) {
            float4v st[4];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) st[kb] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int kb = 0; kb < 4; ++kb) {
                    const half8v kf = *reinterpret_cast<const half8v*>(&sm.k[buf][(kb * 16 + fr) * LDK + kk * 32 + G * 8]);
                    st[kb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf, qf[kk], st[kb], 0, 0, 0);
                }
            float tmax = -INFINITY;
            const int jmax = a.causal ? (i < len ? i : len - 1) : len - 1;      // last key this lane's query sees
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (j0 + kb * 16 + G * 4 + e > jmax) st[kb][e] = -INFINITY;
                    tmax = fmaxf(tmax, st[kb][e]);
                }
            tmax = max_xor32(max_xor16(tmax));
            constexpr float kSlack = 8.0f;                                    // the reference moves only where a maximum grew by more (attn_prefill), or is NaN: a wait given up
            const float tm = tmax * c;
            if (__any(!(tm <= m + kSlack))) {
                const float m_new = fmaxf(m, tm), alpha = __builtin_amdgcn_exp2f(m - m_new);
                l *= alpha;
                m = m_new;
#pragma unroll
                for (int db = 0; db < DB; ++db)
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[db][e] *= alpha;
            }
            half8v pf[2];
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(st[kb][e], c, -m));
                    l += p;
                    pf[kb >> 1][(kb & 1) * 4 + e] = (half_t)p;
                }
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    const char* vp = reinterpret_cast<const char*>(&sm.v[buf][(p * 32 + G * 4 + (fr >> 2)) * LDV + db * 16 + (fr & 3) * 4]);
                    const half4v x = lds_read_tr16(vp), y = lds_read_tr16(vp + 16 * LDV * 2);
                    o[db] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7), pf[p], o[db], 0, 0, 0);
                }
        }
        if (jt + 1 < ntiles) {
            sstore(buf ^ 1);
            __syncthreads();
        }
    }
    l = sum_xor32(sum_xor16(l));
    if (row_ok) {
        const float inv = 1.0f / l;
        half_t* op = a.ctx + (size_t)(row0 + i) * a.H + g * D + G * 4;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            half4v t;
#pragma unroll
            for (int e = 0; e < 4; ++e) t[e] = (half_t)(o[db][e] * inv);
            st_agent(op + db * 16, t);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    // rows of each tile that the item covers
    const int first = row0 + i0, past = first + rows, t = first / TR + w.tid;
    if (t * TR < past) {
        const int from = t * TR > first ? t * TR : first, to = (t + 1) * TR < past ? (t + 1) * TR : past;
        raise(counter(a, t, kCntAtt), (uint32_t)(to - from));
    }
}

template <bool ONCE>
__global__ __launch_bounds__(kPThreads, 2) void prompt_layers(PromptArgs a) {
    __shared__ __attribute__((aligned(16))) PromptSmem sm;
    Spot w;
    w.tid = threadIdx.x;
    w.lane = w.tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(w.tid >> 6);
    if (w.tid == 0) {
        sm.word = __hip_atomic_fetch_add(a.ctl, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sm.late = 0;
    }
    __syncthreads();
    const uint32_t item = __builtin_amdgcn_readfirstlane(sm.word);
    if (item >= (uint32_t)a.items) return;
    w.layer = (int)(item / (uint32_t)a.per_layer);
    int i = (int)(item - (uint32_t)w.layer * (uint32_t)a.per_layer);
    const int R = a.row_tiles;
    if (i < a.n_qkv) { project<kPQkv, ONCE>(a, w, sm, i % R, i / R, 0); return; }
    i -= a.n_qkv;
    if (i < a.n_att) {
        const int g = i % a.heads, bb = i / a.heads, b = bb % a.batch, block = bb / a.batch;
        if (a.d == 64) attend<64>(a, w, sm, b, g, block);
        else attend<128>(a, w, sm, b, g, block);
        return;
    }
    i -= a.n_att;
    if (i < a.n_out) { project<kPOut, ONCE>(a, w, sm, i % R, i / R, 0); return; }
    i -= a.n_out;
    if (i < a.n_ffn1) { project<kPFfn1, ONCE>(a, w, sm, i % R, i / R, 0); return; }
    i -= a.n_ffn1;
    const int rest = i / R;
    project<kPFfn2, ONCE>(a, w, sm, i % R, rest / a.ranges, rest % a.ranges);
}

// One wave per padded row: its place in the packed order, or zeros in `out`; then the exchange area of the decode steps to come and the
// counters of the launch that follows.
__global__ __launch_bounds__(256) void prompt_setup(SeqLens lens, int batch, int S, int width, int32_t* __restrict__ cache_lens, int32_t* __restrict__ cu,
                                                    int32_t* __restrict__ row_map, half_t* out, int left, uint32_t* ctl, int ctl_words, StepArea step) {
    const int lane = threadIdx.x & 63, row_blocks = (batch * S + 3) / 4;
    if ((int)blockIdx.x >= row_blocks) {
        const uint32_t part = blockIdx.x - row_blocks, parts = gridDim.x - row_blocks, n = parts * 256, at = part * 256 + threadIdx.x;
        for (uint32_t i = at; i < (uint32_t)ctl_words; i += n) ctl[i] = 0u;
        for (uint32_t i = at; i < step.words * (uint32_t)step.groups; i += n) step.ctl[i] = i % step.words < (uint32_t)kStepCtlWords ? 0ull : ~0ull;
        return;
    }
    const int r = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= batch * S) return;
    const int b = r / S, i = r - b * S, len = lens.len[b], first = left ? S - len : 0;
    const int before = tokens_before(lens, b, lane);
    if (i == 0 && lane == 0) {
        cache_lens[b] = len;
        cu[b] = before;
        if (b == batch - 1) cu[batch] = before + len;
    }
    if (i >= first && i < first + len) {
        if (lane == 0) row_map[before + i - first] = r;
    } else {
        const half8v z = {(half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f, (half_t)0.f};
        for (int c = lane; c < (width >> 3); c += 64) reinterpret_cast<half8v*>(out + (int64_t)r * width)[c] = z;
    }
}

}  // namespace

// What a layer costs here is its items, up to about 1300 of them, against seven or eight launches that grow little with the rows.  us per pass, launch by
// launch / one launch, rows (items), stacks of 4: hidden 256 x 1024, 40 rows 115 / 70, 240 (564) 125 / 81, 480 (1128) 125 / 96; 384 x 1536, 240 (936) 136 / 106, 480
// (1872) 142 / 148; 512 x 2048, 40 121 / 93, 240 (1248) 149 / 120, 400 (2080) 157 / 168; 768 x 3072, 40 129 / 112, 120 (1092) 161 / 133, 200 (1740) 171 / 168; 1024 x 4096, 40
// 144 / 131, 80 (992) 171 / 148, 120 (1584) 174 / 165, 200 (2528) 184 / 242; 24 of it, 37 rows 917 / 744.  One layer: 256, 40 rows 36 / 21, 480 35 / 30; 512, 240
// 38.3 / 37.7; 768, 120 42.6 / 41.3, 240 (2052) 44 / 55; 1024, 40 39.8 / 40.3, 80 46.3 / 44.0 (33 to 64 rows: the launches are up to 3 % ahead in passes behind
// one another, 10 % behind where each pass is waited for; taken all the same, so that a stack has the bits of its layers one by one).  Up to 16 rows are taken by the small-layer kernel
// elsewhere, which is ahead from 1024 x 4096 on (10 rows, 4 layers 104 / 113; 1024 x 2688 118 / 109); feed-forward parts of more than 4096 columns
// (1024 x 8192, 80 rows 184 / 195) are not worth their ranges.  (Row tiles of 32 and 64: 24 x 1024, 37 rows 892 and 1098; 512, 250 rows 32.5, 34.9 and 42.6 per layer.)
constexpr int kPromptStepItems = 1280;
static int items_of_rows(int64_t rows, int hidden, int ffn) {
    const PromptShape p = prompt_step_shape((int)rows, hidden, ffn);
    return p.row_tiles * (hidden / 16 + ffn / 64 + hidden / 64 * p.ranges);
}
static bool takes_layer(int64_t rows, int hidden, int heads, int ffn) {
    const int d = hidden / heads;
    if (rows < 1 || rows > kPromptStepRows || (d != 64 && d != 128) || hidden % 64 != 0 || hidden > kPromptStepK || ffn % 64 != 0 || ffn > kPromptStepRanges * kPromptStepK) return false;
    return (rows > 16 || (int64_t)hidden * ffn <= (int64_t)3 << 20) && items_of_rows(rows, hidden, ffn) <= kPromptStepItems;
}
bool prompt_step_fits(int64_t rows, int64_t padded_rows, int batch, int max_len, int hidden, int heads, int ffn) {
    return takes_layer(rows, hidden, heads, ffn) && padded_rows * hidden * (int64_t)sizeof(half_t) < (int64_t)1 << 31 &&
           items_of_rows(rows, hidden, ffn) + heads * batch * ((max_len + 16 * kPWaves - 1) / (16 * kPWaves)) <= kPromptStepItems;
}
PromptShape prompt_step_shape(int rows, int hidden, int ffn) {
    PromptShape p{};
    p.row_tiles = (rows + kPRows - 1) / kPRows;
    p.ranges = (ffn + kPromptStepK - 1) / kPromptStepK;
    p.range_units = (ffn / 64 + p.ranges - 1) / p.ranges;
    p.ranges = (ffn / 64 + p.range_units - 1) / p.range_units;
    p.counters = 4 + p.ranges + hidden / 64;
    p.ctl_words = (uint32_t)(1 + p.row_tiles * p.counters) * kClearStride;
    // everything that the launch hands on, one after the other
    uint32_t at = 0;
    auto place = [&](uint32_t bytes) { const uint32_t here = at; at += (bytes + 255u) / 256u * 256u; return here; };
    p.at_ctl = place(p.ctl_words * (uint32_t)sizeof(uint32_t));
    p.at_f = place((uint32_t)rows * ffn * (uint32_t)sizeof(half_t));
    p.at_q = place((uint32_t)rows * hidden * (uint32_t)sizeof(half_t));
    p.at_ctx = place((uint32_t)rows * hidden * (uint32_t)sizeof(half_t));
    p.at_y = place((uint32_t)rows * hidden * (uint32_t)sizeof(half_t));
    p.at_part = place(p.ranges > 1 ? (uint32_t)(p.row_tiles * kPRows) * hidden * p.ranges * (uint32_t)sizeof(float) : 0u);
    p.bytes = at;
    return p;
}
// For any prompt of up to max_rows rows: more rows take more, so the most rows of the most tiles (17 rows: two tiles, past the rule for few rows)
size_t prompt_step_bytes_up_to(int64_t max_rows, int hidden, int heads, int ffn) {
    if (!takes_layer(max_rows < 17 ? max_rows : 17, hidden, heads, ffn)) return 0;
    int64_t rows = kPRows * (kPromptStepItems / items_of_rows(1, hidden, ffn));
    rows = rows < kPromptStepRows ? rows : kPromptStepRows;
    return prompt_step_shape((int)(rows < max_rows ? rows : max_rows), hidden, ffn).bytes;
}

hipError_t launch_prompt_setup(const SeqLens& lens, const PromptArgs& a, int32_t* cache_lens, int32_t* cu, int32_t* row_map, StepArea step, hipStream_t s) {
    const int ctl_words = (int)a.ctl_words;
    const int extra = (int)((step.words * (uint32_t)step.groups + ctl_words + 1023) / 1024);
    hipLaunchKernelGGL(prompt_setup, dim3((a.padded_rows + 3) / 4 + extra), dim3(256), 0, s, lens, a.batch, a.S, a.H, cache_lens, cu, row_map, a.out, a.left_pad,
                       a.ctl, ctl_words, step);
    return hipGetLastError();
}

hipError_t launch_prompt_layers(PromptArgs& a, bool read_once, hipStream_t s) {
    a.d = a.H / a.heads;
    a.n_qkv = a.row_tiles * (3 * a.H / 64);
    a.n_att = a.heads * a.batch * ((a.max_len + 16 * kPWaves - 1) / (16 * kPWaves));
    a.n_out = a.row_tiles * (a.H / 64);
    a.n_ffn1 = a.row_tiles * (a.F / 64);
    a.per_layer = a.n_qkv + a.n_att + a.n_out + a.n_ffn1 + a.n_out * a.ranges;
    a.items = a.per_layer * a.n_layers;
    const dim3 grid(a.items), block(kPThreads);
    if (read_once) hipLaunchKernelGGL(prompt_layers<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(prompt_layers<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace eet
