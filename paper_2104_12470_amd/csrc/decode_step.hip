// Decode steps of small layers: all layers of a step in one launch.
//
// A decode step of a small layer (up to 16 sequences, or several groups of as many, a few MB per projection) is a chain of five dependent
// phases, and as five launches each of them costs the floor of a dependent launch (drain, start, first trip to memory: about 4 us for 1 to 8 MB of
// weights), whatever its bytes.  Here the chain runs inside one launch.  A workgroup is one ITEM of one layer: 64 columns of a projection (16
// of the second feed-forward one), or one key range of a (sequence, head) pair.  It requests its weights (or K/V rows), up to 256 KB, into
// registers first, since they depend on nothing, and only then waits for its input, which the items of the phase before hand
// over through memory.  While a phase runs, the CUs that it leaves idle hold the weights of the next ones: HBM never waits for the chain, and a
// phase costs its hand-over (1.0 to 1.5 us from the producers' sums to a consumer's whole input, of which 0.45 to 0.7 is one store seen by
// one load across the chip) and its arithmetic.
// us per layer-step, five launches -> now: hidden 1024 in a stack of 24, 1 sequence 21.2 -> 9.7, 8 sequences of 384 to 768 tokens
// 26.4 -> 13.3; 60 drawn sizes (hidden 256 to 2048, 1 to 24 layers, 1 to 8 sequences of 1 to 3200 tokens) 1.18 to 3.1 times as
// fast, geometric mean 1.86; 30 of 9 to 16 sequences 1.09 to 2.9, 1.58.
//
//   hand-over   The exchange buffers hold 8-byte words (four halfs, or two floats) that are all ones until their producer stores them,
//               and a producer never stores all ones in either half (a NaN of that pattern becomes another NaN).  A consumer loads
//               the words it needs until none is empty: the data is its own flag, one trip to memory per phase.  Stores and loads are at
//               agent scope (relaxed), which is what makes them coherent between the XCDs' caches; nothing else is ordered by them and nothing
//               else needs to be.  Flags or a counter beside the data cost a second trip (256 workgroups, all to all: 2.9 and 4.8 us
//               against 2.5), release and acquire fences write back and invalidate whole caches (22).
//   lines       A line is written by one workgroup, in one go: every store to a line that others are polling takes the line away from all
//               of them first.  Four producers per line: 21.8 us per layer-step where 16-column items with a line each take 20.4, and
//               64-column items, with a quarter of the lines to poll, 12.4 (one sequence, on the variant of 8 rows).
//   reuse       Layer number g (counted on over all steps since the last prefill) uses exchange set g % 2.  An item of the QKV
//               projection of layer g has seen all of x(g) when it starts to normalise: every item of layer g-1 has handed on its result, so
//               nobody reads the other set any more, and the QKV items empty it, each its part, and count themselves in `resets` when their
//               part is empty in memory.  An item of layer g touches its set only once resets >= g * (QKV items); the second feed-forward projection,
//               which writes x(g+1) into the other set, once resets >= (g+1) * (QKV items).
//   progress    An item waits only for items with lower numbers, and a workgroup takes its number from a counter when it starts
//               to run, so whatever an item waits for runs already or has finished: no assumption about how many workgroups are resident, in
//               which order they start, or what else runs on the device.  The waits are bounded all the same (kSpinLimit).  Words that did
//               not come read as NaN, an item that found its exchange set still in use hands NaN on, and both say so in ctl: the sets
//               may hold words of another layer from then on, so the output of every later launch is NaN until the area is set up again
//               (prefill, restore).
//
//   groups      Steps of more sequences are groups of up to 16 (8 of the wider layers), each a chain of its own: a ticket counter, a count of resets
//               and exchange sets for every group, workgroups dealt to the groups in turn.  What another step leaves out it does not touch, so
//               steps of other numbers of sequences may come in between.
//
// K/V rows of earlier tokens are ordinary memory (written by earlier launches); the new token's K and V row reaches the attention
// through the exchange set, and the cache for the steps that follow.
//
// One workgroup per CU (the registers see to that): two, with 128 registers each, start so far ahead that their polling
// slows the phases they wait for (12.4 -> 14.2 us per layer-step with one sequence on the variant of 8 rows, 9.7 on its own).
#include "kernels.hpp"

namespace eet {

namespace {

typedef unsigned long long word_t;                 // four halfs or two floats
typedef unsigned uint4v __attribute__((ext_vector_type(4)));
constexpr word_t kEmpty = ~0ull;
constexpr unsigned kEmptyHalf = ~0u;
constexpr int kAgentScope = 16;                    // cache policy of a buffer load at agent scope: sc1
constexpr int kSWaves = 8, kSThreads = 64 * kSWaves;
constexpr int kSRow = 72;                          // halfs of a staged row: 128 bytes + 16
constexpr int kSUnitsH = 4, kSUnitsF = 16;         // units of 64 K values a wave holds: K = hidden up to 2048, K = ffn up to 8192
// Polls before an item gives up (the launch still ends): a tenth of a second at the least, where a wait takes microseconds and
// whatever it waits for is running.  (The loops below end in one place, `ok` or the bound: with a way out for each the compiler copies
// the loop, a quarter more code for the kernel.)
constexpr int kSpinLimit = 1 << 20;

__device__ __forceinline__ word_t ld_word(const word_t* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void st_word(word_t* p, word_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// Neither 4-byte half of a published word is all ones, so a consumer may also load 16 bytes at once and look at each.
__device__ __forceinline__ void publish(word_t* p, half4v v) {
    const word_t w = __builtin_bit_cast(word_t, v);
    const unsigned lo = (unsigned)w, hi = (unsigned)(w >> 32);
    st_word(p, (word_t)(hi == kEmptyHalf ? 0xFE00FE00u : hi) << 32 | (lo == kEmptyHalf ? 0xFE00FE00u : lo));
}
__device__ __forceinline__ void publish(word_t* p, float x, float y) {
    const unsigned lo = __builtin_bit_cast(unsigned, x), hi = __builtin_bit_cast(unsigned, y);
    st_word(p, (word_t)(hi == kEmptyHalf ? 0xFFC00000u : hi) << 32 | (lo == kEmptyHalf ? 0xFFC00000u : lo));
}

// words of a key range's partial result: D/2 of values, one of (maximum, sum), whole lines
__host__ __device__ constexpr int step_range_words(int d) { return d / 2 + 16; }

struct StepSmem {
    // wave-private: 2 weight units of 16 rows, or units of the input with 32 rows in all; the attention's merge lies over it
    half_t stage[kSWaves][2 * 16 * kSRow];
    float red[kSWaves][16 * 68];                   // [wave][row][up to 64 columns + 4]
    float stat[16][kSWaves * 4 + 4];               // [row][wave] sum, mean and squared deviations of the wave's share of the row (+4: rows in other banks)
    word_t ticket;
    int in_use;                                    // the wait for the exchange set came to its bound
};

template <int LANES>
__device__ __forceinline__ float sum_shares(float v) {   // over aligned groups of 4 or 8 lanes
    static_assert(LANES == 4 || LANES == 8, "lanes");
    v += dpp<0xb1>(v);
    v += dpp<0x4e>(v);
    return LANES == 8 ? v + dpp<0x141>(v) : v;
}

// where this item stands
struct Where {
    int layer;                                     // inside the launch
    uint32_t g;                                    // layer number since the last prefill
    int lane, wave, tid;
    int row0, M;                                   // this group's rows
    word_t* ctl;                                   // ... and control words
    word_t* set;                                   // exchange set of layer g
    word_t* other;                                 // ... and of layers g-1 and g+1
    bool void_area;                                // a wait was given up since the area was set up
};

// A wait came to its bound: said in ctl.  (At the wait itself, and read with the item's number in later launches, where neither costs the chain
// anything: a flag looked at before each result is handed on was 10.56 -> 10.72 us per layer-step of 24 x hidden 1024, ctl looked at before
// the last output is written up to 0.9 us per launch, 28.2 -> 29.0 for one layer of hidden 1280.)
__device__ __forceinline__ void give_up(const Where& w) { __hip_atomic_fetch_or(w.ctl, (word_t)kStepGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Thread 0 waits until the exchange set is this layer's, then for one word of the phase before the one whose output the item
// needs: the tight polling that follows lasts one phase instead of a whole layer.  `input`: a word of the input itself, for the QKV
// projection, whose faster items empty the set of that earlier word as soon as they have all of theirs; looked at now and then only, since
// every look at a line that is still to be written makes the write slower.  (Giving up on that word loses nothing: the input
// itself is waited for next.)
__device__ __forceinline__ void wait_resets(const StepArgs& a, const Where& w, StepSmem& sm, uint32_t layers) {
    const uint32_t* resets = reinterpret_cast<const uint32_t*>(w.ctl + 16);
    const uint32_t target = layers * (uint32_t)a.n_qkv;
    int spin = 0;
    while (true) {
        if ((int32_t)(__hip_atomic_load(resets, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - target) >= 0) return;
        if (++spin == kSpinLimit) break;
        __builtin_amdgcn_s_sleep(16);
    }
    sm.in_use = 1;
    give_up(w);
}
// -> whether that set came in time
__device__ __forceinline__ bool gate(const StepArgs& a, const Where& w, StepSmem& sm, const word_t* before, const word_t* input, bool emptied_by_this_layer) {
    if (w.tid == 0) {
        wait_resets(a, w, sm, w.g);
        if (before != nullptr)
            for (int spin = 0; spin < kSpinLimit; ++spin) {
                if (ld_word(before) != kEmpty) break;
                if (input != nullptr && spin % 16 == 15 && ld_word(input) != kEmpty) break;
                __builtin_amdgcn_s_sleep(4);
            }
        if (emptied_by_this_layer) wait_resets(a, w, sm, w.g + 1u);
    }
    __syncthreads();
    return sm.in_use == 0;
}

__device__ __forceinline__ word_t wait_word(const Where& w, const word_t* p) {
    word_t v;
    int spin = 0;
    do v = ld_word(p);
    while ((v == kEmpty) & (++spin < kSpinLimit));
    if (v == kEmpty) give_up(w);
    return v;
}

__device__ __forceinline__ half_t no_value() { return __builtin_bit_cast(half_t, (unsigned short)0x7e00); }

// ---- one item of a projection: 16*NT columns, all rows (at most 16), K in units of 64 dealt round-robin to the waves ------------
enum StepPhase { kStepQkv = 0, kStepOut = 1, kStepFfn1 = 2, kStepFfn2 = 3 };

// Exchange buffers hold a producer's output as a block: [row][its columns], whole lines of 16 words.  Word of (row, column):
__device__ __forceinline__ uint32_t word_at(const StepBuffer& b, int row, int col) {
    return b.at + (uint32_t)(col >> b.log_cols) * b.block + (((uint32_t)row << b.log_cols) + (uint32_t)(col & ((1 << b.log_cols) - 1))) / 4u;
}

// How the 16 words of a unit's rows lie over a wave: VW words per lane, LPR lanes per row, UPI units per load instruction.  Rows
// that do not exist cost lanes, i.e. instructions of the LayerNorm and of the polling, hence the variants of 1, 2, 4, 8 and 16 rows
// (one sequence on the variant of 8: 12.4 us per layer-step instead of 10.6).
template <int ROWS>
struct RowLanes {
    static constexpr int VW = ROWS == 16 ? 4 : ROWS == 8 ? 2 : 1, LPR = 16 / VW, UPI = 64 / (LPR * ROWS);
};
// sum over the lanes of a row
template <int ROWS>
__device__ __forceinline__ float row_sum(float v) {
    v += dpp<0xb1>(v);                                    // lane ^ 1
    v += dpp<0x4e>(v);                                    // lane ^ 2: 4 lanes
    if (ROWS <= 8) v += dpp<0x141>(v);                    // 8 lanes
    if (ROWS <= 4) v += dpp<0x140>(v);                    // 16 lanes
    if (ROWS == 1) v = sum_xor16(v);
    if (ROWS <= 2) v = sum_xor32(v);
    return v;
}

// Partial sums of neighbouring columns, in pairs: the order in which row_sum goes on over the lanes
template <int N>
__device__ __forceinline__ float pair_sum(const float (&p)[N]) {
    static_assert(N == 1 || N == 2 || N == 4, "partial sums");
    if constexpr (N == 4) return (p[0] + p[1]) + (p[2] + p[3]);
    else if constexpr (N == 2) return p[0] + p[1];
    else return p[0];
}

// E columns of the input of the first layer, from column c on
template <int E>
__device__ __forceinline__ void input_row(const StepArgs& a, int row, int c, half_t (&out)[E]) {
    typedef half_t halfE __attribute__((ext_vector_type(E), aligned(E == 4 ? 8 : 16)));
    halfE v;
    if (a.tok.ids == nullptr) {
        v = *reinterpret_cast<const halfE*>(a.x + (size_t)row * a.H + c);
    } else {
        const int id = a.tok.ids[row], pos = a.lens[row];
        if (id < 0 || id >= a.tok.vocab || pos < 0 || pos >= a.tok.max_pos) {
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = no_value();
        } else {
            const halfE t = *reinterpret_cast<const halfE*>(a.tok.wte + (size_t)id * a.H + c), p = *reinterpret_cast<const halfE*>(a.tok.wpe + (size_t)pos * a.H + c);
#pragma unroll
            for (int e = 0; e < E; ++e) v[e] = (half_t)((float)t[e] + (float)p[e]);     // exact in fp32, rounded once
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) out[e] = v[e];
}

template <int ROWS, int U, int NT, int PH, bool ONCE>
__device__ __forceinline__ void project(const StepArgs& a, const Where& w, StepSmem& sm, int tile) {
    constexpr bool LN = PH == kStepQkv || PH == kStepFfn1, RES = PH == kStepOut || PH == kStepFfn2;
    constexpr int TN = 16 * NT, RT = TN + 4;                   // columns, floats of a row of a partial tile
    constexpr int VW = RowLanes<ROWS>::VW, LPR = RowLanes<ROWS>::LPR, UPI = RowLanes<ROWS>::UPI, E = 4 * VW;
    constexpr int STEPS = (U + UPI - 1) / UPI;
    typedef half_t halfE __attribute__((ext_vector_type(E), aligned(E == 4 ? 8 : 16)));
    constexpr int XU = ROWS == 16 ? 2 : 4;                     // units of the input staged at a time
    const StepLayer& L = a.layer[w.layer];
    const int M = w.M, H = a.H, K = PH == kStepFfn2 ? a.F : H;
    const int units = K / 64, n0 = tile * TN;
    const int lane = w.lane, wave = w.wave;
    const int wrow = lane >> 3, wchunk = lane & 7;             // this lane's 16 bytes of 8 weight rows
    const int row = lane / LPR % ROWS, sub = lane / (LPR * ROWS), e0 = lane % LPR * E;   // its part of the input: row, unit of a step, first column in it
    const int fr = lane & 15, G = lane >> 4;                   // ... and as a matrix operand
    const half_t* weights = PH == kStepQkv ? L.w_qkv : PH == kStepOut ? L.w_o : PH == kStepFfn1 ? L.w_fc1 : L.w_fc2;
    const half_t* bias = PH == kStepQkv ? L.b_qkv : PH == kStepOut ? L.b_o : PH == kStepFfn1 ? L.b_fc1 : L.b_fc2;
    const bool first = w.layer == 0, last = w.layer == a.n_layers - 1;
    auto has = [&](int s) { return s * UPI + sub < U && wave + kSWaves * (s * UPI + sub) < units; };   // step s brings this lane a unit
    auto column = [&](int s) { return (wave + kSWaves * (s * UPI + sub)) * 64 + e0; };

    // ---- what depends on nothing: weights, scale and shift, bias, cache slot ----
    half8v wf[U][NT][2];
    {
        const char* wb = reinterpret_cast<const char*>(weights) + (size_t)n0 * K * 2;
        const uint32_t off = ((uint32_t)wrow * K + wchunk * 8) * 2u;
#pragma unroll
        for (int i = 0; i < U; ++i)
            if (wave + kSWaves * i < units) {
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const half8v* p = reinterpret_cast<const half8v*>(wb + (off + (uint32_t)((t * 16 + h * 8) * K + (wave + kSWaves * i) * 64) * 2u));
                        wf[i][t][h] = ONCE ? load_once(p) : *p;
                    }
            }
    }
    halfE gv[LN ? STEPS : 1], bv[LN ? STEPS : 1];
    if constexpr (LN) {
        const half_t* gamma = PH == kStepQkv ? L.ln1_g : L.ln2_g;
        const half_t* beta = PH == kStepQkv ? L.ln1_b : L.ln2_b;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (has(s)) {
                gv[s] = *reinterpret_cast<const halfE*>(gamma + column(s));
                bv[s] = *reinterpret_cast<const halfE*>(beta + column(s));
            }
    }
    const int em = w.tid / (TN / 4), ec = (w.tid % (TN / 4)) * 4, en = n0 + ec;   // the M * TN/4 threads that write: row, first of four columns
    const bool writer = w.tid < M * (TN / 4);
    half4v eb, er;
    half_t* slot = nullptr;                                    // where in the cache the row's keys or values go
    if (writer) {
        eb = *reinterpret_cast<const half4v*>(bias + en);
        if (PH == kStepQkv) {
            const int which = n0 / H, c = en - which * H, epos = a.lens[w.row0 + em];      // (a tile lies in one of Q, K and V)
            if (which != 0 && epos >= 0 && epos < a.max_seq)      // past the capacity (replays the host never saw): dropped
                slot = (which == 1 ? L.k_cache : L.v_cache) + ((size_t)((w.row0 + em) * a.heads + c / a.d) * a.max_seq + epos) * a.d + c % a.d;
        }
        if (PH == kStepOut && first) {
            half_t r[4];
            input_row(a, w.row0 + em, en, r);
            er = half4v{r[0], r[1], r[2], r[3]};
            if (a.tok.ids != nullptr) *reinterpret_cast<half4v*>(a.tok.rows + (size_t)(w.row0 + em) * H + en) = er;
        }
    }
    // of the LayerNorm: the size of this wave's share of a row and of those that this lane merges (worked out here: behind the wait they are in the chain)
    constexpr int SL = LPR < kSWaves ? LPR : kSWaves, SN = kSWaves / SL;       // the waves' shares, neighbours dealt to the lanes of a row
    float inv_k, inv_share, weight[SN];
    if constexpr (LN) {
        auto share = [&](int v) { return (float)(v < units ? 64 * ((units - v + kSWaves - 1) / kSWaves) : 0); };
        inv_k = 1.0f / (float)K;
        inv_share = wave < units ? __builtin_amdgcn_rcpf(share(wave)) : 0.f;     // a power of two, or rounded once: any value near the mean serves
#pragma unroll
        for (int v = 0; v < SN; ++v) {
            weight[v] = share(lane % SL * SN + v);
            asm volatile("" : "+v"(weight[v]));
        }
        asm volatile("" : "+v"(inv_k), "+v"(inv_share));
    }
    // weights into matrix-operand layout by way of LDS (whole lines per load instruction), while there is nothing else to do: two
    // 16-row units at a time
    half_t* st = sm.stage[wave];
#pragma unroll
    for (int q = 0; q < U * NT; q += 2) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (q + j < U * NT && wave + kSWaves * ((q + j) / NT) < units)
#pragma unroll
                for (int h = 0; h < 2; ++h) *reinterpret_cast<half8v*>(&st[(j * 16 + 8 * h + wrow) * kSRow + wchunk * 8]) = wf[(q + j) / NT][(q + j) % NT][h];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (q + j < U * NT && wave + kSWaves * ((q + j) / NT) < units)
#pragma unroll
                for (int h = 0; h < 2; ++h) wf[(q + j) / NT][(q + j) % NT][h] = *reinterpret_cast<const half8v*>(&st[(j * 16 + fr) * kSRow + G * 8 + 32 * h]);
    }

    // ---- the input ----
    const StepBuffer& in = PH == kStepQkv ? a.bx : PH == kStepOut ? a.bctx : PH == kStepFfn1 ? a.by : a.bf;
    const word_t* before = PH == kStepQkv ? (first ? nullptr : w.other + a.bf.at)
                         : PH == kStepOut ? w.set + a.bqkv.at
                         : PH == kStepFfn1 ? w.set + a.bctx.at : w.set + a.by.at;
    const bool in_time = gate(a, w, sm, before, PH == kStepQkv ? w.set + in.at : nullptr, PH == kStepFfn2);
    if (RES && writer && !(PH == kStepOut && first))
        er = __builtin_bit_cast(half4v, wait_word(w, w.set + word_at(PH == kStepOut ? a.bx : a.by, em, en)));
    // not in time: every value of the item becomes NaN, by way of the LayerNorm or of the residual
    const float eps = in_time ? a.eps : __builtin_nanf("");
    if (RES && !in_time) er = half4v{no_value(), no_value(), no_value(), no_value()};
    halfE xv[STEPS];
    const bool mine = row < M;
    if (PH == kStepQkv && first) {
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (has(s) && mine) {
                half_t r[E];
                input_row(a, w.row0 + row, column(s), r);
#pragma unroll
                for (int e = 0; e < E; ++e) xv[s][e] = r[e];
            }
    } else if (PH == kStepOut && a.splits > 1) {
        // the attention's key ranges: merge them (common maximum, rescaled sums, one division)
        const int stride = step_range_words(a.d);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            float lsum = 0.f, mx = -INFINITY, av[E];
#pragma unroll
            for (int e = 0; e < E; ++e) av[e] = 0.f;
            if (has(s) && mine) {
                const int k = column(s);
                const word_t* p = w.set + in.at + (size_t)(row * a.heads + k / a.d) * a.splits * stride;
                const int at = (k % a.d) / 2;
                for (int s0 = 0; s0 < a.splits; s0 += 2, p += 2 * stride) {      // a power of two of them
                    word_t v[2][E / 2 + 1];
                    int spin = 0;
                    bool ok;
                    do {
                        ok = true;
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
#pragma unroll
                            for (int e = 0; e < E / 2; ++e) v[r][e] = ld_word(p + r * stride + at + e);
                            v[r][E / 2] = ld_word(p + r * stride + a.d / 2);
                        }
#pragma unroll
                        for (int r = 0; r < 2; ++r)
#pragma unroll
                            for (int e = 0; e <= E / 2; ++e) ok &= v[r][e] != kEmpty;
                    } while (!ok & (++spin < kSpinLimit));
                    if (!ok) give_up(w);
#pragma unroll
                    for (int r = 0; r < 2; ++r) {
                        const float2v ml = __builtin_bit_cast(float2v, v[r][E / 2]);
                        const float m_new = fmaxf(mx, ml[0]);
                        const float keep = exp2f(mx - m_new), add = exp2f(ml[0] - m_new);
                        lsum = lsum * keep + ml[1] * add;
#pragma unroll
                        for (int e = 0; e < E / 2; ++e) {
                            const float2v q = __builtin_bit_cast(float2v, v[r][e]);
                            av[2 * e] = av[2 * e] * keep + q[0] * add;
                            av[2 * e + 1] = av[2 * e + 1] * keep + q[1] * add;
                        }
                        mx = m_new;
                    }
                }
            }
            const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;
#pragma unroll
            for (int e = 0; e < E; ++e) xv[s][e] = (half_t)(av[e] * inv);
        }
    } else {
        // (a unit is a whole number of blocks)
        const word_t* p = w.set + word_at(in, row, column(0));
        const uint32_t per_step = (uint32_t)(UPI * kSWaves) * (64u >> in.log_cols) * in.block;
        word_t v[STEPS][VW];
        const auto set = __builtin_amdgcn_make_buffer_rsrc(w.set, 0, (int)(a.set_words * sizeof(word_t)), 0x00027000);
        const uint32_t off = (uint32_t)(p - w.set);
        int spin = 0;
        bool ok;
        do {
            asm volatile("" ::: "memory");
            unsigned most = 0;                                 // a half that is kEmptyHalf is the largest there is
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                if (has(s) && mine) {
                    if constexpr (VW >= 2) {
#pragma unroll
                        for (int q = 0; q < VW; q += 2) {
                            const uint4v r = __builtin_amdgcn_raw_buffer_load_b128(set, (int)((off + s * per_step + q) * sizeof(word_t)), 0, kAgentScope);
                            v[s][q] = (word_t)r[1] << 32 | r[0];
                            v[s][(q + 1) % VW] = (word_t)r[3] << 32 | r[2];
                        }
                    } else {
                        v[s][0] = ld_word(p + s * per_step);
                    }
                }
            // (a loop of its own: every load is requested before the first is waited for)
#pragma unroll
            for (int s = 0; s < STEPS; ++s)
                if (has(s) && mine) {
#pragma unroll
                    for (int q = 0; q < VW; ++q) most = max(most, max((unsigned)v[s][q], (unsigned)(v[s][q] >> 32)));
                }
            ok = __all(most != kEmptyHalf);
        } while (!ok & (++spin < kSpinLimit));
        if (!ok) give_up(w);
        struct Words { word_t w[VW]; };
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
            Words x;
#pragma unroll
            for (int q = 0; q < VW; ++q) x.w[q] = v[s][q];
            xv[s] = __builtin_bit_cast(halfE, x);
        }
    }
    asm volatile("" ::: "memory");
    if constexpr (PH == kStepFfn2) {
        // everyone who reads the cache lengths in this step is an ancestor of this item's input
        if (last && a.bump && tile == 0) {
            __syncthreads();                                   // all waves have their share of the input: together, all of it
            if (w.tid < M) a.lens[w.row0 + w.tid] += 1;
        }
    }

    if constexpr (LN) {
        // Sum and squared deviations of the wave's share of each row, then of the row (shares merged by their sizes).  The mean is one sum, divided once, as in
        // the LayerNorm's own launches, and the share's own mean is taken from the values before anything else, which leaves a small shift: a row far
        // from zero loses no bits.  (x * rstd - mean * rstd has an error of 2e-5 deviations where the mean is a thousand of them.)
        // Added up per four columns, then in pairs: a row has the same bits on the variants of 4, 8 and 16 rows, whose lanes hold 4, 8 and 16 columns.
        float psum[E / 4], psq[E / 4], dev[STEPS][E];
#pragma unroll
        for (int p = 0; p < E / 4; ++p) psum[p] = psq[p] = 0.f;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (has(s)) {
#pragma unroll
                for (int e = 0; e < E; e += 2) psum[e / 4] = __builtin_amdgcn_fdot2(half2v{xv[s][e], xv[s][e + 1]}, half2v{(half_t)1.f, (half_t)1.f}, psum[e / 4], false);
            }
        const float sum = row_sum<ROWS>(pair_sum(psum));
        const float mw = sum * inv_share;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
            if (has(s)) {
#pragma unroll
                for (int e = 0; e < E; e += 2) {
                    minus_mean(half2v{xv[s][e], xv[s][e + 1]}, mw, dev[s][e], dev[s][e + 1]);
                    psq[e / 4] = __builtin_fmaf(dev[s][e], dev[s][e], psq[e / 4]);
                    psq[e / 4] = __builtin_fmaf(dev[s][e + 1], dev[s][e + 1], psq[e / 4]);
                }
            }
        const float sq = row_sum<ROWS>(pair_sum(psq));
        if (lane % LPR == 0 && sub == 0) *reinterpret_cast<float4v*>(&sm.stat[row][wave * 4]) = float4v{sum, mw, sq, 0.f};
        __syncthreads();
        if constexpr (PH == kStepQkv) {
            // all waves together have seen all of x(g): layer g-1 is finished, its exchange set is nobody's (the acknowledgement
            // is awaited below, before anything of this item is handed on)
            const uint32_t per = ((a.set_words + a.n_qkv - 1) / a.n_qkv + 15) / 16 * 16, lo = tile * per;
            const uint32_t hi = lo + per < a.set_words ? lo + per : a.set_words;
            for (uint32_t c = lo + w.tid; c < hi; c += kSThreads) st_word(w.other + c, kEmpty);
        }
        float4v sv[SN];
        float total = 0.f, m2 = 0.f;
#pragma unroll
        for (int v = 0; v < SN; ++v) sv[v] = *reinterpret_cast<const float4v*>(&sm.stat[row][(lane % SL * SN + v) * 4]);
#pragma unroll
        for (int v = 0; v < SN; ++v) total += sv[v][0];
        const float mean = mean_of(sum_shares<SL>(total), K, inv_k);
#pragma unroll
        for (int v = 0; v < SN; ++v) {
            const float d = sv[v][1] - mean;
            m2 += __builtin_fmaf(weight[v] * d, d, sv[v][2]);
        }
        m2 = sum_shares<SL>(m2);
        const float rstd = rsqrtf(m2 * inv_k + eps), shift = (mw - mean) * rstd;
#pragma unroll
        for (int s = 0; s < STEPS; ++s)
#pragma unroll
            for (int e = 0; e < E; ++e) {
                // fused multiply-adds that take their fp16 operands directly
                const float t = __builtin_fmaf(dev[s][e], rstd, shift);
                xv[s][e] = (half_t)__builtin_fmaf(t, (float)gv[s][e], (float)bv[s][e]);
            }
    }

    // ---- contraction: acc[t][r] = output column n0 + 16t + 4G + r of row fr ----
    float4v acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < U; i += XU) {                          // through the staging area
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int s = i / UPI; s < (i + XU) / UPI && s < STEPS; ++s)
            if (has(s)) *reinterpret_cast<halfE*>(&st[((s * UPI + sub - i) * ROWS + row) * kSRow + e0]) = xv[s];
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < XU && i + j < U; ++j)
            if (wave + kSWaves * (i + j) < units) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const half8v xf = *reinterpret_cast<const half8v*>(&st[(j * ROWS + (fr & (ROWS - 1))) * kSRow + G * 8 + 32 * h]);
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[i + j][t][h], xf, acc[t], 0, 0, 0);
                }
            }
    }
    static_assert(ROWS * RT <= (int)(sizeof(sm.red[0]) / sizeof(float)), "a wave's partial tile");
    if (fr < ROWS) {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<float4v*>(&sm.red[wave][fr * RT + 16 * t + 4 * G]) = acc[t];
    }
    __syncthreads();
    if (writer) {
        float4v v = *reinterpret_cast<const float4v*>(&sm.red[0][em * RT + ec]);
#pragma unroll
        for (int o = 1; o < kSWaves; ++o) v += *reinterpret_cast<const float4v*>(&sm.red[o][em * RT + ec]);
        half4v out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float f = v[e] + (float)eb[e];
            if (PH == kStepFfn1) f = gelu_tanh(f);
            if (RES) f += (float)er[e];
            out[e] = (half_t)f;
        }
        if constexpr (PH == kStepQkv) {
            publish(w.set + word_at(a.bqkv, em, en), out);
            if (slot != nullptr) *reinterpret_cast<half4v*>(slot) = out;
        } else if constexpr (PH == kStepOut) {
            publish(w.set + word_at(a.by, em, en), out);
        } else if constexpr (PH == kStepFfn1) {
            publish(w.set + word_at(a.bf, em, en), out);
        } else {
            if (last) {
                if (w.void_area) out = half4v{no_value(), no_value(), no_value(), no_value()};
                *reinterpret_cast<half4v*>(a.out + (size_t)(w.row0 + em) * H + en) = out;
            } else publish(w.other + word_at(a.bx, em, en), out);
        }
    }
    if constexpr (PH == kStepQkv) {
        // what this item emptied of the other set is empty in memory before it is counted
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (w.tid == 0) __hip_atomic_fetch_add(reinterpret_cast<uint32_t*>(w.ctl + 16), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---- one key range of a (sequence, head) pair ----------------------------------------------------------------------------------
// As attn_decode (attention.hip): a key row over D/8 adjacent lanes, running (max, sum, values) per lane group, merged at the end.
// Up to 1024 keys (heads of 64; 512 of 128) are in registers before the query arrives; half as many cost 0.9 us per layer-step with
// eight sequences of 384 to 768 tokens.
template <int D, bool ONCE>
__device__ __forceinline__ void attend(const StepArgs& a, const Where& w, StepSmem& sm, int item) {
    constexpr int LPK = D / 8, KPI = 64 / LPK, U = 4, BK = U * KPI, PF = 4;      // PF blocks of BK keys in flight per wave
    constexpr float kNone = -1e30f, kLog2e = 1.4426950408889634f;
    const StepLayer& L = a.layer[w.layer];
    const int sp = item % a.splits, bh = item / a.splits, b = bh / a.heads, h = bh - b * a.heads;
    if (b >= w.M) return;                                     // (the last group may have fewer rows)
    const int lane = w.lane, wave = w.wave, kslot = lane / LPK, chunk = lane % LPK;
    int n = a.lens[w.row0 + b];                                        // cached keys; the new token's is number n
    n = n < 0 ? 0 : n;
    const bool room = n < a.max_seq;
    const int visible = room ? n + 1 : a.max_seq;
    int per = (visible + a.splits - 1) / a.splits;
    per = (per + 15) & ~15;
    const int c0 = sp * per, c1 = c0 + per < visible ? c0 + per : visible;
    const bool has_new = room && c0 <= n && n < c1;
    const int ce = has_new ? n : c1;                          // cached keys of the range: [c0, ce)
    const char* kbase = reinterpret_cast<const char*>(L.k_cache + (size_t)(w.row0 * a.heads + bh) * a.max_seq * D);
    const char* vbase = reinterpret_cast<const char*>(L.v_cache + (size_t)(w.row0 * a.heads + bh) * a.max_seq * D);
    half8v kr[PF][U], vr[PF][U];
    auto request = [&](half8v (&kf)[U], half8v (&vf)[U], int j0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int r = j0 + u * KPI + kslot;
            r = r < ce ? r : ce - 1;
            const uint32_t off = (uint32_t)r * (uint32_t)(D * 2) + (uint32_t)chunk * 16u;
            const half8v* kp = reinterpret_cast<const half8v*>(kbase + off);
            const half8v* vp = reinterpret_cast<const half8v*>(vbase + off);
            kf[u] = ONCE ? load_once(kp) : *kp;
            vf[u] = ONCE ? load_once(vp) : *vp;
        }
    };
    const int j0 = c0 + wave * BK;                            // blocks wave, wave + 8, ... of the range
#pragma unroll
    for (int i = 0; i < PF; ++i)
        if (j0 + i * kSWaves * BK < ce) request(kr[i], vr[i], j0 + i * kSWaves * BK);
    const bool in_time = gate(a, w, sm, w.layer == 0 ? nullptr : w.set + a.bx.at, nullptr, false);
    const word_t* qkv = w.set + word_at(a.bqkv, b, h * D + chunk * 8);
    const uint32_t to_k = (uint32_t)(a.H >> a.bqkv.log_cols) * a.bqkv.block;
    half8v qv, kn, vn;
    const bool take_new = has_new && wave == 0;
    {
        word_t v[6];
        const word_t* p = qkv;
        int spin = 0;
        bool ok;
        do {
            v[0] = ld_word(p);
            v[1] = ld_word(p + 1);
            if (take_new) {
                v[2] = ld_word(p + to_k);
                v[3] = ld_word(p + to_k + 1);
                v[4] = ld_word(p + 2 * to_k);
                v[5] = ld_word(p + 2 * to_k + 1);
            }
            ok = v[0] != kEmpty && v[1] != kEmpty;
            if (take_new) ok &= v[2] != kEmpty && v[3] != kEmpty && v[4] != kEmpty && v[5] != kEmpty;
            ok = __all(ok);
        } while (!ok & (++spin < kSpinLimit));
        if (!ok) give_up(w);
        auto join = [](word_t x, word_t y) {
            return __builtin_shufflevector(__builtin_bit_cast(half4v, x), __builtin_bit_cast(half4v, y), 0, 1, 2, 3, 4, 5, 6, 7);
        };
        qv = join(v[0], v[1]);
        if (take_new) {
            kn = join(v[2], v[3]);
            vn = join(v[4], v[5]);
        }
    }
    const float c = in_time ? rsqrtf((float)D) * kLog2e : __builtin_nanf("");      // not in time: NaN
    auto score = [&](const half8v& k) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_fdot2(half2v{k[2 * e], k[2 * e + 1]}, half2v{qv[2 * e], qv[2 * e + 1]}, d, false);
        d = sum8(d);
        if (LPK == 16) d += dpp<0x140>(d);
        return d * c;
    };
    float acc[8], m = kNone, l = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.f;
    auto consume = [&](const half8v (&kf)[U], const half8v (&vf)[U], int j) {
        float sc[U], mx = kNone;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float s = score(kf[u]);
            sc[u] = j + u * KPI + kslot < ce ? s : -INFINITY;
            mx = fmaxf(mx, sc[u]);
        }
        const float m_new = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f(m - m_new);
        l *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= alpha;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float p = __builtin_amdgcn_exp2f(sc[u] - m_new);
            l += p;
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(p, (float)vf[u][e], acc[e]);
        }
        m = m_new;
    };
    for (int jb = j0; jb < ce; jb += PF * kSWaves * BK) {
#pragma unroll
        for (int i = 0; i < PF; ++i) {
            const int jc = jb + i * kSWaves * BK, jn = jc + PF * kSWaves * BK;
            if (jc >= ce) break;
            consume(kr[i], vr[i], jc);
            if (jn < ce) request(kr[i], vr[i], jn);
        }
    }
    if (take_new) {                                           // the new token's key: lane group 0 of wave 0
        const float s = kslot == 0 ? score(kn) : -INFINITY;
        const float m_new = fmaxf(m, s), alpha = __builtin_amdgcn_exp2f(m - m_new), p = __builtin_amdgcn_exp2f(s - m_new);
        l = l * alpha + p;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(p, (float)vn[e], acc[e] * alpha);
        m = m_new;
    }
    // lane groups, then waves
    float mw = m;
    if (LPK == 8) mw = fmaxf(mw, dpp<0x128>(mw));
    mw = max_xor32(max_xor16(mw));
    const float r = __builtin_amdgcn_exp2f(m - mw);
    l *= r;
    if (LPK == 8) l += dpp<0x128>(l);
    l = sum_xor32(sum_xor16(l));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        acc[e] *= r;
        if (LPK == 8) acc[e] += dpp<0x128>(acc[e]);
        acc[e] = sum_xor32(sum_xor16(acc[e]));
    }
    float* sm_acc = reinterpret_cast<float*>(&sm.stage[0][0]);       // [waves][D]
    static_assert(sizeof(float) * kSWaves * 128 <= sizeof(sm.stage), "merge over the staging areas");
    if (lane < LPK) {
#pragma unroll
        for (int e = 0; e < 8; ++e) sm_acc[wave * D + lane * 8 + e] = acc[e];
    }
    if (lane == 0) *reinterpret_cast<float2v*>(&sm.stat[wave][0]) = float2v{mw, l};
    __syncthreads();
    if (w.tid >= D / 2) return;
    float2v ml[kSWaves];
    float mx = kNone;
#pragma unroll
    for (int v = 0; v < kSWaves; ++v) {
        ml[v] = *reinterpret_cast<const float2v*>(&sm.stat[v][0]);
        mx = fmaxf(mx, ml[v][0]);
    }
    float sum = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
    for (int v = 0; v < kSWaves; ++v) {
        const float f = __builtin_amdgcn_exp2f(ml[v][0] - mx);
        const float2v x = *reinterpret_cast<const float2v*>(&sm_acc[v * D + w.tid * 2]);
        sum += ml[v][1] * f;
        a0 += x[0] * f;
        a1 += x[1] * f;
    }
    if (a.splits > 1) {
        word_t* p = w.set + a.bctx.at + (size_t)item * step_range_words(D);
        publish(p + w.tid, a0, a1);
        if (w.tid == 0) publish(p + D / 2, mx, sum);
        return;
    }
    const float inv = sum > 0.f ? 1.0f / sum : 0.f;
    const float b0 = a0 * inv, b1 = a1 * inv;
    const float c0_ = dpp<0xb1>(b0), c1_ = dpp<0xb1>(b1);
    if ((w.tid & 1) == 0)
        publish(w.set + word_at(a.bctx, b, h * D + w.tid * 2), half4v{(half_t)b0, (half_t)b1, (half_t)c0_, (half_t)c1_});
}

// ROWS: rows, rounded up.  UH, NTH: units of K = hidden per wave and blocks of 16 columns per item in the three projections from
// there; UF: units of K = ffn per wave.  The weights of an item take 64 registers per lane (hidden up to 1024) or 128.
template <int ROWS, int UH, int NTH, int UF, bool ONCE>
__global__ __launch_bounds__(kSThreads, 2) void decode_layers(StepArgs a) {
    __shared__ __attribute__((aligned(16))) StepSmem sm;
    Where w;
    w.tid = threadIdx.x;
    w.lane = w.tid & 63;
    w.wave = __builtin_amdgcn_readfirstlane(w.tid >> 6);
    // The number of this item, in the order in which workgroups start (low half), and the layer number of the launch's first layer
    // (high half).  The launch's last workgroup to ask turns both on for the next launch.
    const int group = (int)blockIdx.x % a.groups;
    w.row0 = group * a.rows;
    w.M = a.M - w.row0 < a.rows ? a.M - w.row0 : a.rows;
    w.ctl = a.ctl + (size_t)group * (kStepCtlWords + 2 * (size_t)a.set_words);
    word_t* const ex = w.ctl + kStepCtlWords;
    if (w.tid == 0) {
        const word_t t = __hip_atomic_fetch_add(w.ctl, (word_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (((uint32_t)t & ~kStepGaveUp) == (uint32_t)a.items - 1u)
            __hip_atomic_fetch_add(w.ctl, ((word_t)a.n_layers << 32) - (word_t)a.items, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sm.ticket = t;
        sm.in_use = 0;
    }
    __syncthreads();
    const uint32_t low = __builtin_amdgcn_readfirstlane((uint32_t)sm.ticket), item = low & ~kStepGaveUp, g0 = __builtin_amdgcn_readfirstlane((uint32_t)(sm.ticket >> 32));
    if (item >= (uint32_t)a.items) return;
    w.layer = (int)(item / (uint32_t)a.per_layer);
    int r = (int)(item - (uint32_t)w.layer * (uint32_t)a.per_layer);
    w.g = g0 + (uint32_t)w.layer;
    w.set = ex + (size_t)(w.g & 1u) * a.set_words;
    w.other = ex + (size_t)(~w.g & 1u) * a.set_words;
    w.void_area = (low & kStepGaveUp) != 0;
    if (r < a.n_qkv) { project<ROWS, UH, NTH, kStepQkv, ONCE>(a, w, sm, r); return; }
    r -= a.n_qkv;
    if (r < a.n_att) {
        if (a.d == 64) attend<64, ONCE>(a, w, sm, r);
        else attend<128, ONCE>(a, w, sm, r);
        return;
    }
    r -= a.n_att;
    if (r < a.n_out) { project<ROWS, UH, NTH, kStepOut, ONCE>(a, w, sm, r); return; }
    r -= a.n_out;
    if (r < a.n_ffn1) { project<ROWS, UH, NTH, kStepFfn1, ONCE>(a, w, sm, r); return; }
    project<ROWS, UF, 1, kStepFfn2, ONCE>(a, w, sm, r - a.n_ffn1);
}

// Key ranges per pair: up to 128 items of at least 128 keys at full capacity, so that the attention's items leave CUs to the
// projections that follow (256 of them: 8 sequences of 384 to 768 tokens, 16 heads: 15.6 -> 19.9 us per layer-step).
int step_splits(int rows, int heads, int capacity) {
    const int pairs = rows * heads;
    int s = 1;
    while (2 * s * pairs <= 128 && capacity / (2 * s) >= 128 && s < 16) s *= 2;
    return s;
}

}  // namespace

// More than 8 rows double the registers of the input: only where the weights leave them.
static bool step_is_narrow(int hidden, int ffn) { return hidden <= 64 * kSWaves * 2 && ffn <= 64 * kSWaves * 8; }
static int step_group_rows(int hidden, int ffn) { return step_is_narrow(hidden, ffn) ? 16 : 8; }
// The groups of a step of `rows` rows (as even as they come) and the rows of the largest
static void step_groups(int rows, int hidden, int ffn, int& groups, int& group_rows) {
    const int most = step_group_rows(hidden, ffn);
    group_rows = (rows + (rows + most - 1) / most - 1) / ((rows + most - 1) / most);
    groups = (rows + group_rows - 1) / group_rows;
}
// More than one group: what the launch costs is its items, about 7 us per 256 of them beyond the first 512, against launches that grow
// little with the rows.  us per layer-step (stacks of 2, 200 to 400 keys unless said), launch by launch / one launch, items: 24 sequences of hidden 256 27.5 / 14.3 (156);
// 128 of it 33.8 / 23.2 (624); 96 of 512 (heads of 64) 39.5 / 34.1 (1344); 32 of 768 36.3 / 25.8 (672), 64 42.0 / 37.6 (1344), 20 to 40 keys 34.9 / 34.5, 128 60 /
// 70 (2688); 1024 x 4096, 24 37.8 / 26.9 (768), 48 45.4 / 40.3 (1344), 64 51.1 / 49.1, 20 to 40 keys 41.6 / 45.2 (1792).  Where it stops besides: more than 256
// pairs over 512 slots and more keep the attention kernel of their own, whose bits are the operator's (24 x 16 heads, 800 to 1600 keys 55.0 / 41.7, so
// not for speed); up to 256 pairs gain there too (24 x 4 heads 33.8 / 18.1).  The wider layers' groups of 8 rows read the weights once more each: level from
// 16 sequences of 1792 on (43.3 / 45.6), and below that their steps of 9 to 16 stay with the small-layer kernel and its LayerNorms.
// A layer on its own has no next layer to begin with while the last items end, and its launches find their weights in the caches: it stops earlier, and the
// sooner the more attention items stand before the rest of a wide layer.  us per step of one layer, launch by launch / one launch, 20 to 40, 100 to 200, 250 to 450
// keys: 1024 with 16 heads, 30 sequences 26.7 / 29.9, 30.5 / 31.0, 33.2 / 32.8; 40 30.3 / 32.4, 33.8 / 33.8, 39.0 / 37.3; 44 30.4 / 38.1, 34.6 / 39.8, 40.4 / 43.9; with
// 8 heads, 48 30.9 / 29.1, 35.3 / 31.3, 42.5 / 36.5; 768 with 12, 48 29.6 / 27.2, 30.4 / 28.9, 33.3 / 31.7; 56 29.4 / 30.4, 30.4 / 32.2, 35.0 / 35.1; 64 30.3 / 32.8, 31.5 /
// 34.8, 37.6 / 38.3; 512 with 8, 80 29.8 / 26.0, 29.8 / 27.4, 32.0 / 30.7; 96 29.9 / 29.5, 30.1 / 31.6, 34.5 / 35.5.  Stacks do not lose
// at any of these, of 6 layers, short keys: 48 of 1024 1645 / 1604 in 8 steps, 40 1604 / 1568, 64 of 768 1477 / 1479, 96 of 512 1344 / 1317; of 2, 200 to 450 keys, 40 of 1024
// 709 / 600.  (So here, and only here, a layer's bits are not those of the same layer in a stack.)
constexpr int kStepGroupItems = 1350, kStepGroupItemsAlone = 1280, kStepPairsAlone = 460 << 10;    // the last: pairs times hidden
bool decode_step_fits(int rows, int hidden, int heads, int ffn, int max_seq, int layers) {
    const int d = hidden / heads;
    if (rows < 1 || rows > kStepGroups * step_group_rows(hidden, ffn) || (d != 64 && d != 128) || hidden % 64 != 0 || ffn % 64 != 0 ||
        hidden > 64 * kSWaves * kSUnitsH || ffn > 64 * kSWaves * kSUnitsF) return false;
    int groups, group_rows;
    step_groups(rows, hidden, ffn, groups, group_rows);
    if (groups == 1) return true;
    const int items = groups * (hidden / 16 + ffn / 64 + hidden / 16 + group_rows * heads);
    return step_is_narrow(hidden, ffn) && items <= kStepGroupItems && (rows * heads <= 256 || max_seq < 512) &&
           (layers > 1 || (items <= kStepGroupItemsAlone && rows * heads * hidden <= kStepPairsAlone));
}

// Long sequences: a CU streams the K/V rows of one item at a time, and next to that the launches that are saved count for little.  Where
// the pairs leave CUs idle (65 to 112 of them are not split) or their number fills a round that the QKV items have already begun (224
// and more), the attention kernel of its own is ahead from 6000 to 10000 tokens per sequence on.  us per layer-step, launch by launch / one
// launch, 16000 tokens: 96 pairs of heads of 128: hidden 1024 161 / 181, 1536 151 / 184, 2048 163 / 194; 80 of 640 158 / 174; 112 of 2048 178 /
// 202; 256 of heads of 64: 1024 193 / 206, 2048 192 / 223.  8000: 99 / 103, 105 / 101, 118 / 110, 97 / 94, 127 / 115, 108 / 111, 130 / 124.  Others
// stay, 16000: 128 pairs of hidden 1024, heads of 128 208 / 199, of 64 199 / 105; 144 of 64 121 / 113, 192 148 / 131; 96 of 768, heads of 64,
// 8000 95.7 / 55.6.
bool decode_step_fits_keys(int rows, int heads, int d, size_t visible) {
    const int pairs = rows * heads;
    // (several groups of sequences, launch by launch / one launch: 17 of hidden 512, 8500 keys each 79 / 68; of 256, 12000 66 / 91; 20 of 384 89 / 99)
    if (rows > 16) return visible <= (size_t)8192 * rows;
    return visible <= (size_t)8192 * rows || !(pairs >= 224 || (d == 128 && pairs > 64 && pairs <= 112));
}

// Where the buffers of a step of a.M rows lie in an exchange set; the words that they take
static uint32_t step_layout(StepArgs& a) {
    const int d = a.H / a.heads, log_h = 6;                   // 64 columns per item
    a.d = d;
    step_groups(a.M, a.H, a.F, a.groups, a.rows);
    a.splits = step_splits(a.M, a.heads, a.max_seq);
    uint32_t at = 0;
    auto buffer = [&](int cols, int log_cols) {
        const uint32_t block = (uint32_t)((a.rows << log_cols) / 4 + 15) / 16 * 16;
        const StepBuffer b{at, block, log_cols};
        at += (uint32_t)(cols >> log_cols) * block;
        return b;
    };
    a.bx = buffer(a.H, 4);
    a.bqkv = buffer(3 * a.H, log_h);
    a.bctx = buffer(a.H, 6);
    if (a.splits > 1) at = a.bctx.at + (uint32_t)(a.rows * a.heads * a.splits * step_range_words(d));
    a.by = buffer(a.H, log_h);
    a.bf = buffer(a.F, log_h);
    return at;
}

int decode_step_groups(int max_rows, int hidden, int heads, int ffn, int max_seq) {
    const int limit = kStepGroups * step_group_rows(hidden, ffn);
    for (int rows = max_rows < limit ? max_rows : limit; rows >= 1; --rows) {   // more rows, more groups
        if (!decode_step_fits(rows, hidden, heads, ffn, max_seq, 2)) continue;                 // (a stack's: a layer on its own has no more)
        int groups, group_rows;
        step_groups(rows, hidden, ffn, groups, group_rows);
        return groups;
    }
    return 0;
}

uint32_t decode_step_set_words(int max_rows, int hidden, int heads, int ffn, int max_seq) {
    uint32_t most = 0;
    for (int rows = 1; rows <= max_rows && rows <= step_group_rows(hidden, ffn) && decode_step_fits(rows, hidden, heads, ffn, max_seq, 2); ++rows) {
        StepArgs a{};
        a.M = rows; a.H = hidden; a.heads = heads; a.F = ffn; a.max_seq = max_seq;
        const uint32_t words = step_layout(a);
        most = words > most ? words : most;
    }
    return most;
}

hipError_t launch_decode_layers(StepArgs& a, bool read_once, hipStream_t s) {
    if (step_layout(a) > a.set_words) return hipErrorInvalidValue;
    const int log_h = a.bqkv.log_cols;
    a.n_qkv = 3 * a.H >> log_h;
    a.n_att = a.rows * a.heads * a.splits;
    a.n_out = a.H >> log_h;
    a.n_ffn1 = a.F >> log_h;
    a.per_layer = a.n_qkv + a.n_att + a.n_out + a.n_ffn1 + a.H / 16;
    a.items = a.per_layer * a.n_layers;
    const dim3 grid(a.items * a.groups), block(kSThreads);
#define EET_STEP(ROWS, UH, UF) do { if (read_once) hipLaunchKernelGGL((decode_layers<ROWS, UH, 4, UF, true>), grid, block, 0, s, a); \
                                    else hipLaunchKernelGGL((decode_layers<ROWS, UH, 4, UF, false>), grid, block, 0, s, a); } while (0)
    if (step_is_narrow(a.H, a.F)) {
        if (a.rows <= 1) EET_STEP(1, 2, 8);
        else if (a.rows <= 2) EET_STEP(2, 2, 8);
        else if (a.rows <= 4) EET_STEP(4, 2, 8);
        else if (a.rows <= 8) EET_STEP(8, 2, 8);
        else EET_STEP(16, 2, 8);
    } else {
        if (a.rows <= 1) EET_STEP(1, 4, 16);
        else if (a.rows <= 2) EET_STEP(2, 4, 16);
        else if (a.rows <= 4) EET_STEP(4, 4, 16);
        else EET_STEP(8, 4, 16);
    }
#undef EET_STEP
    return hipGetLastError();
}

}  // namespace eet
