// Dense projections y = x W^T + b with fused epilogues (QKV scatter into the K/V cache,
// add-bias+GELU, add-bias+residual with optional row scatter back to the padded layout).
//
// The paper leaves these to library GEMM calls followed by separate bias/activation kernels
// (Section 3.2 notes that fusion stops at the GEMM calls).  Here the epilogue
// runs on the accumulators, so the intermediate never visits HBM.
//
// Kernels:
//   gemm_mfma_dma64  prefill (M = valid tokens of the batch, packed) and decode steps of many sequences: 256x256 tiles
//                    for the large problems, 128x128, 128x64 and 64x64 when there are few; direct global->LDS loads,
//                    v_mfma_f32_16x16x32_f16; bound by the matrix cores.
//   gemm_flat        decode (M <= 16 rows), small layers: one memory round trip, few instructions.
//   gemm_stream      decode, large layers: every weight is read from HBM exactly once per step, so
//                    the kernel is a weight stream; v_mfma_f32_16x16x32_f16 does the 16-row contraction.
//   gemm_skinny      decode, shapes the two above do not take.
// All compute the transposed tile (weights as the MFMA "A" operand) so that each lane ends up
// with 4 consecutive output columns of one row (the tile kernel: 8, see tile_column).
#include <cstdlib>
#include <mutex>
#include <set>
#include <type_traits>
#include <utility>

#include "kernels.hpp"
#include "pipeline.hpp"

namespace eet {

// --------------------------------------------------------------------------------------------
// epilogue on 4 consecutive output columns n..n+3 of row m
// --------------------------------------------------------------------------------------------
// Operands of the epilogue that come from memory; a latency-bound kernel fetches them before its
// main loop so that no dependent round trip is left after the last MFMA.
struct EpiOperands {
    half4v bias, res;
    int pos;            // QKV only: padded row of the token (prefill) or cache slot n_b (decode)
};

template <int EPI>
__device__ __forceinline__ void epilogue_fetch(const GemmArgs& a, int m, int n, EpiOperands& o) {
    o.bias = *reinterpret_cast<const half4v*>(a.bias + n);
    if (EPI == EPI_BIAS_RES) {
        const int64_t rr = a.res_row_map ? (int64_t)a.res_row_map[m] : (int64_t)m;
        o.res = *reinterpret_cast<const half4v*>(a.res + rr * a.N + n);
    }
    if (EPI == EPI_QKV) o.pos = a.tok_row_map ? a.tok_row_map[m] : a.lens[m];
}

template <int EPI>
__device__ __forceinline__ half4v epilogue_apply(const GemmArgs& a, int m, int n, float v0, float v1, float v2, float v3,
                                                 const EpiOperands& e) {   // returns the four values as stored
    v0 += (float)e.bias[0]; v1 += (float)e.bias[1]; v2 += (float)e.bias[2]; v3 += (float)e.bias[3];
    if (EPI == EPI_BIAS_GELU) {
        v0 = gelu_tanh(v0); v1 = gelu_tanh(v1); v2 = gelu_tanh(v2); v3 = gelu_tanh(v3);
    }
    if (EPI == EPI_BIAS_RES) {
        v0 += (float)e.res[0]; v1 += (float)e.res[1]; v2 += (float)e.res[2]; v3 += (float)e.res[3];
    }
    half4v o;
    o[0] = (half_t)v0; o[1] = (half_t)v1; o[2] = (half_t)v2; o[3] = (half_t)v3;
    if (EPI == EPI_QKV) {
        const int which = n / a.hidden;          // 0 = Q, 1 = K, 2 = V
        const int c = n - which * a.hidden;
        if (which == 0) {
            *reinterpret_cast<half4v*>(a.y + (int64_t)m * a.hidden + c) = o;
        } else {
            int b_, pos;
            if (a.tok_row_map) {                 // prefill: token -> (sequence, position)
                b_ = e.pos / a.S;
                pos = e.pos - b_ * a.S;
                if (a.left_pad) pos -= a.S - a.lens[b_];
            } else {                             // decode: the new token goes to slot n_b
                b_ = m;
                pos = e.pos;
            }
            if (pos < 0 || pos >= a.max_seq) return o;   // device-side lengths advanced past the capacity (replays the host never saw): drop, never write outside the slots
            const int g = c / a.d, dd = c - g * a.d;
            half_t* cache = which == 1 ? a.k_cache : a.v_cache;
            *reinterpret_cast<half4v*>(cache + (((int64_t)b_ * a.heads + g) * a.max_seq + pos) * a.d + dd) = o;
        }
        return o;
    }
    const int64_t orow = a.out_row_map ? (int64_t)a.out_row_map[m] : (int64_t)m;
    *reinterpret_cast<half4v*>(a.y + orow * a.N + n) = o;
    return o;
}

template <int EPI>
__device__ __forceinline__ void epilogue4(const GemmArgs& a, int m, int n, float v0, float v1, float v2, float v3) {
    EpiOperands e;
    epilogue_fetch<EPI>(a, m, n, e);
    epilogue_apply<EPI>(a, m, n, v0, v1, v2, v3, e);
}

// --------------------------------------------------------------------------------------------
// epilogue of the MFMA tile kernels
// --------------------------------------------------------------------------------------------
// A lane of an accumulator block holds four values of one row.  Which columns they are is free, since the weight rows may be dealt to the
// blocks in any order: block j, operand row i is column tile_column(j, i) of the wave tile, so that a lane has 8 consecutive columns in each pair of
// blocks and the four lanes of a row 32, and the output goes straight out of the accumulators in pieces of 64 bytes.  (Blocks
// of 16 consecutive columns left a lane 8 bytes here and 8 there: 0.7 TB/s.)  Turned around through LDS to whole lines first, as it was, a 256 x 256 tile took 5.6 us
// behind its K loop with a bias, 10.1 with GELU and 12.2 with a residual, most of it one wave's chain of LDS writes, reads and stores; now 5.2, 7.2 and 9.
// What is left: 1 us of look-ups, 3.4 for 33 MB of output from all CUs at once, 5 for as much of residual.  us, before -> now: 6758 x 8192 x 2048 with GELU 209
// -> 198, 12288 x 4096 x 2048 177 -> 167, 3054 x 4096 x 1024 29.9 -> 28.3; with a residual 6758 x 2048 x 8192 188 -> 184, 12288 x 4096 x 2048 185 -> 179, 20000 x
// 768 x 768 34.4 -> 31.2.
__host__ __device__ constexpr int tile_column(int j, int i) { return (j / 2) * 32 + (i / 4) * 8 + (j % 2) * 4 + i % 4; }

// Two loads of 8 rows by 64 columns (lanes 0-7 of 16 a row's 16 bytes of the first 32 columns, lanes 8-15 of the last 32) into 16 rows by 32 columns
// each: the lower lanes keep the first load and take its other half from the upper lanes, which keep the second.
__device__ __forceinline__ void lines_to_rows(half8v& first, half8v& second, bool upper) {
    typedef int int4v __attribute__((ext_vector_type(4)));
    int4v d0 = __builtin_bit_cast(int4v, first), d1 = __builtin_bit_cast(int4v, second);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int y0 = __builtin_amdgcn_update_dpp(0, d0[q], 0x128, 0xf, 0xf, false);      // lane ^ 8
        const int y1 = __builtin_amdgcn_update_dpp(0, d1[q], 0x128, 0xf, 0xf, false);
        d0[q] = upper ? y1 : d0[q];
        d1[q] = upper ? d1[q] : y0;
    }
    first = __builtin_bit_cast(half8v, d0);
    second = __builtin_bit_cast(half8v, d1);
}

// Rows m of the problem: r0 = output row (EPI_QKV: the sequence whose cache the row's K and V go to), r1 = residual row (EPI_QKV: the cache slot; negative
// or >= max_seq: dropped).  Every look-up is requested before anything waits for one.  Rows past M come as M-1; they are never stored.
template <int EPI, int R>
__device__ __forceinline__ void epilogue_rows(const GemmArgs& a, const int (&m)[R], int (&r0)[R], int (&r1)[R]) {
    if constexpr (EPI == EPI_QKV) {
        if (a.tok_row_map) {                             // prefill: token -> (sequence, position)
            int tok[R];
#pragma unroll
            for (int i = 0; i < R; ++i) tok[i] = a.tok_row_map[m[i]];
#pragma unroll
            for (int i = 0; i < R; ++i) {
                r0[i] = tok[i] / a.S;
                r1[i] = tok[i] - r0[i] * a.S;
            }
            if (a.left_pad) {                            // pads lead: token 0 of the sequence is at row S - L_b
                int len[R];
#pragma unroll
                for (int i = 0; i < R; ++i) len[i] = a.lens[r0[i]];
#pragma unroll
                for (int i = 0; i < R; ++i) r1[i] -= a.S - len[i];
            }
        } else {                                         // decode: the new token goes to slot n_b
#pragma unroll
            for (int i = 0; i < R; ++i) {
                r0[i] = m[i];
                r1[i] = a.lens[m[i]];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            r0[i] = a.out_row_map ? a.out_row_map[m[i]] : m[i];
            r1[i] = (EPI == EPI_BIAS_RES && a.res_row_map) ? a.res_row_map[m[i]] : m[i];
        }
    }
}

// A bias alone or with a residual out of the tiles of which two workgroups share a CU (192 x 128 and 128 x 128 with two stages, under either schedule) goes
// out through LDS all the same: the stages are free, a CU has the other workgroup to go on with, and whole lines out in one go get in its way less.  us, straight
// out / through LDS (rows x N x K): with a residual 1066 x 7232 x 128 10.4 / 9.2, 367 x 13952 x 128 9.25 / 8.4, 1753 x 11904 x 320 1.07 / 0.99 of what it
// took when all tiles went through LDS; a bias alone 5535 x 2176 x 128 1.06 / 1.01, 523 x 14336 x 448 1.06 / 1.01; from K = 512 on level; 59 of 128 x 128 tiles with a
// residual and spread loads, K = 512 to 3072, 0.989 / 0.968 of that.  GELU and the scatter to Q and the caches go straight out: GELU 1667 x 2816 x 128
// 7.8 / 8.7, 2319 x 3328 x 384 0.95 / 1.0; Q, K and V by 192 x 128 tiles K = 320 14.8 / 18.0, 128 x 128 tiles K = 256 11.4 / 13.4 and 24.0 / 27.6, spread
// loads K = 1088 22.4 / 23.9.  128 x 64 tiles, three to a CU, all go straight out: level with a residual or a bias, 0.96 / 1.01 with GELU.
//
// `stage`: AM*16*128 bytes of LDS no other wave touches, a row of 64 columns in 128 bytes, its sixteen 8-byte units XOR-permuted by (row/2)%16 so
// that both access patterns spread over all banks.  Whole-line pattern: row it*8 + lane/8, 16-byte chunk lane%8.
template <int AM, int EPI>
__device__ __forceinline__ void epilogue_via_lds(const GemmArgs& a, const float4v (&acc)[AM][4], char* stage, int mw, int nw, int lane) {
    static_assert(EPI == EPI_BIAS || EPI == EPI_BIAS_RES, "outputs that are better through LDS");
    constexpr int R = AM * 2;
    const int M = a.M, N = a.N, r8 = lane >> 3, c8 = lane & 7;
    if (nw >= N) return;
    int m[R], r0[R], r1[R];
#pragma unroll
    for (int it = 0; it < R; ++it) {
        m[it] = mw + it * 8 + r8;
        m[it] = m[it] < M ? m[it] : M - 1;
    }
    epilogue_rows<EPI>(a, m, r0, r1);
    if constexpr (EPI == EPI_BIAS_RES) {
        half8v rv[R];
#pragma unroll
        for (int it = 0; it < R; ++it) rv[it] = *reinterpret_cast<const half8v*>(a.res + (int64_t)r1[it] * N + nw + c8 * 8);
#pragma unroll
        for (int it = 0; it < R; ++it) {
            const int row = it * 8 + r8, sw = (row >> 1) & 15;
            half8v v = rv[it];
            if (sw & 1) v = __builtin_shufflevector(v, v, 4, 5, 6, 7, 0, 1, 2, 3);
            *reinterpret_cast<half8v*>(stage + row * 128 + ((c8 ^ (sw >> 1)) * 16)) = v;
        }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int unit = tile_column(j, (lane >> 4) * 4) / 4;
        const half4v bias = *reinterpret_cast<const half4v*>(a.bias + nw + unit * 4);
#pragma unroll
        for (int i = 0; i < AM; ++i) {
            const int row = i * 16 + (lane & 15);
            half4v* slot = reinterpret_cast<half4v*>(stage + row * 128 + ((unit ^ ((row >> 1) & 15)) * 8));
            half4v v, r{};
            if (EPI == EPI_BIAS_RES) r = *slot;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float f = acc[i][j][e] + (float)bias[e];
                if (EPI == EPI_BIAS_RES) f += (float)r[e];
                v[e] = (half_t)f;
            }
            *slot = v;
        }
    }
#pragma unroll
    for (int it = 0; it < R; ++it) {
        const int row = it * 8 + r8, sw = (row >> 1) & 15;
        if (mw + row >= M) continue;
        half8v v = *reinterpret_cast<const half8v*>(stage + row * 128 + ((c8 ^ (sw >> 1)) * 16));
        if (sw & 1) v = __builtin_shufflevector(v, v, 4, 5, 6, 7, 0, 1, 2, 3);
        const int n = nw + c8 * 8;
        *reinterpret_cast<half8v*>(a.y + (int64_t)r0[it] * (a.ldy ? a.ldy : N) + n) = v;
    }
}

// mw, nw: first row and column of the wave tile; its columns are inside N in groups of 64, or outside (N % 64 == 0).  Row maps and residual are all
// requested before anything waits for them: one trip to memory per tile.  (8192 x 16384 x 2048 with a residual: 634 -> 552 us; 25082 x 12288 x
// 12288: 6.56 -> 6.37 ms).
template <int AM, int AN, int EPI, bool NTS>
__device__ __forceinline__ void epilogue_tile(const GemmArgs& a, const float4v (&acc)[AM][AN], int mw, int nw, int lane) {
    constexpr int P = AN / 2;                             // pairs of blocks: 32 columns each, 8 of them this lane's
    const int M = a.M, N = a.N, fr = lane & 15, G = lane >> 4;
    if (nw >= N) return;
    auto inside = [&](int p) { return P <= 2 || nw + (p / 2) * 64 < N; };
    int m[AM], r0[AM], r1[AM];
#pragma unroll
    for (int i = 0; i < AM; ++i) {
        m[i] = mw + i * 16 + fr;
        m[i] = m[i] < M ? m[i] : M - 1;
    }
    epilogue_rows<EPI>(a, m, r0, r1);
    half8v bias[P];
#pragma unroll
    for (int p = 0; p < P; ++p)
        if (inside(p)) bias[p] = *reinterpret_cast<const half8v*>(a.bias + nw + p * 32 + G * 8);
    // The residual comes in whole lines, 8 rows by 64 columns per load: pair p of block i has rows 8*(p%2) ..+8, and its lanes of the upper half of
    // 16 the columns 32 to 63 (64-byte pieces of 16 rows, as the output goes, slow the other workgroup of a CU down: 3054 x 3072 x 1024 27.8 us, so 27.0)
    const bool upper = fr >= 8;
    half8v res[EPI == EPI_BIAS_RES ? AM : 1][P];
    if constexpr (EPI == EPI_BIAS_RES) {
        int rrow[AM][2];
#pragma unroll
        for (int i = 0; i < AM; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                int r = mw + i * 16 + 8 * h + (fr & 7);
                r = r < M ? r : M - 1;
                rrow[i][h] = a.res_row_map ? a.res_row_map[r] : r;
            }
#pragma unroll
        for (int i = 0; i < AM; ++i)
#pragma unroll
            for (int p = 0; p < P; ++p)
                if (inside(p)) res[i][p] = *reinterpret_cast<const half8v*>(a.res + (int64_t)rrow[i][p % 2] * N + nw + (p / 2) * 64 + (upper ? 32 : 0) + G * 8);
    }
    half_t* col[P];                                       // where column nw + p*32 + G*8 of row 0 goes
    bool to_cache[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int n = nw + p * 32 + G * 8;
        to_cache[p] = false;
        if constexpr (EPI == EPI_QKV) {
            const int which = n / a.hidden, c = n - which * a.hidden, g = c / a.d;      // 0 = Q, 1 = K, 2 = V
            to_cache[p] = which != 0;
            col[p] = which == 0 ? a.y + c : (which == 1 ? a.k_cache : a.v_cache) + (int64_t)g * a.max_seq * a.d + (c - g * a.d);
        } else {
            col[p] = a.y + n;
        }
    }
    const int64_t ldy = EPI == EPI_QKV ? a.hidden : a.ldy ? a.ldy : N;
#pragma unroll
    for (int i = 0; i < AM; ++i) {
        const bool row_inside = mw + i * 16 + fr < M;
        const bool slot = EPI == EPI_QKV && r1[i] >= 0 && r1[i] < a.max_seq;            // see epilogue_apply: never outside the sequence's slots
        const int64_t at = EPI == EPI_QKV ? (int64_t)m[i] * ldy : (int64_t)r0[i] * ldy;
        const int64_t at_cache = EPI == EPI_QKV ? ((int64_t)r0[i] * a.heads * a.max_seq + r1[i]) * a.d : 0;
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if constexpr (EPI == EPI_BIAS_RES) {
                if (p % 2 == 0) lines_to_rows(res[i][p], res[i][p + 1], upper);
            }
            half8v v;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float f = acc[i][2 * p + e / 4][e % 4] + (float)bias[p][e];
                if (EPI == EPI_BIAS_GELU) f = gelu_tanh(f);
                if (EPI == EPI_BIAS_RES) f += (float)res[EPI == EPI_BIAS_RES ? i : 0][p][e];
                v[e] = (half_t)f;
            }
            if (!(row_inside && inside(p) && (!to_cache[p] || slot))) continue;
            half8v* dst = reinterpret_cast<half8v*>(col[p] + (to_cache[p] ? at_cache : at));
            if constexpr (NTS) __builtin_nontemporal_store(v, dst);   // an output too large to stay cached for its reader
            else *dst = v;
        }
    }
}

// --------------------------------------------------------------------------------------------
// MFMA tile kernel
// --------------------------------------------------------------------------------------------
// Tile order: pipe::tile_of_block (pipeline.hpp; the host-side audit checks that it visits every tile exactly once).
// --------------------------------------------------------------------------------------------
// MFMA tile kernel with direct global->LDS loads
// --------------------------------------------------------------------------------------------
// BM x BN tile (256x256 for the large problems, 128x128 and 128x64 for fewer tiles), WGM x WGN waves with wave tiles
// of 64 columns, K steps of 64 through NS LDS stages filled by
// global_load_lds_dwordx4 (no staging registers, no ds_write): with two stages the loads of K step kt+1 are issued
// at the start of step kt, with three (the small tiles, where few workgroups share a CU and nothing else hides the
// trip to memory) those of step kt+2.  An LDS row is the 128 bytes of one operand row, and a wave-level load
// covers 8 rows x 128 bytes, i.e. whole cache lines.  Instead of padding, the eight 16-byte chunks
// of a row are XOR-permuted by half the row's number in its block (activations: (row/2)%8; weights: see tile_column) -- applied on the
// global address of each lane when loading and on the LDS address when reading fragments -- which spreads the rows of a block over all banks.
// MFMA fragments are double-buffered in registers: the reads of the next quarter-step are issued
// before the MFMAs of the current one.
//
// Fragment reads and every wait in the main loop are inline assembly / raw builtins.  The compiler
// cannot tell that an LDS read does not alias an in-flight global->LDS load and would otherwise
// drain all of them (vmcnt(0)) before each read and before each barrier, which undoes the pipeline.

// 16 bytes per lane from global memory straight into LDS: lane l lands at lds + 16*l (the LDS
// base must be wave-uniform).  Kept out of the templates: the builtin only exists for the device.
// NT: with the non-temporal hint (cache policy bit 1), for weights that the launch reads once (common.hpp: load_once).
template <bool NT = false>
__device__ __forceinline__ void load_lds_16B(const half_t* gptr, half_t* lds) {
    __builtin_amdgcn_global_load_lds(gptr, lds, 16, 0, NT ? 2 : 0);
}

template <int N>
__device__ __forceinline__ void wait_lgkm() {
    static_assert(N == 0 || N == 3 || N == 4 || N == 6 || N == 8, "add the count");
    if (N == 0) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (N == 3) asm volatile("s_waitcnt lgkmcnt(3)" ::: "memory");
    if (N == 4) asm volatile("s_waitcnt lgkmcnt(4)" ::: "memory");
    if (N == 6) asm volatile("s_waitcnt lgkmcnt(6)" ::: "memory");
    if (N == 8) asm volatile("s_waitcnt lgkmcnt(8)" ::: "memory");
}
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N == 0 || N == 6 || N == 8 || N == 16, "add the count");
    if (N == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (N == 6) asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
    if (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    if (N == 16) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
}

// The instructions of the tile kernel's K loop.  The loop itself -- which stage is loaded, read, waited for and released
// when -- is pipe::gemm_k_loop or pipe::gemm_k_loop_spread (pipeline.hpp), shared with the host-side audit of the hand-over; this executor supplies the
// instructions, all forced inline.  (Namespace scope because a local class cannot have member templates.)
//
// Matrix instruction: v_mfma_f32_16x16x32_f16.  Under this part's power management the 16x16x32 form sustains about a
// sixth more than 32x32x16 (measured with bare loops of either: 2.08 against 1.79 PFLOP/s over tens of milliseconds): per
// flop it reads and writes half the accumulator registers.  Weights are the A operand (16 output columns x 32 k), the
// activations the B operand (32 k x 16 rows): a lane holds 4 consecutive output columns of one row.
// A wave tile of WM x WN is AM = WM/16 by AN = WN/16 accumulator blocks (WN = 64, or 128 for the four-wave 256 x 256 tile,
// whose 64 blocks per wave live in the accumulation registers).  With two waves per SIMD (pipe::gemm_k_loop) a K tile of
// 64 is walked in four sub-steps s = 2h + mh: k half h (32 columns) times row half mh (AM/2 blocks).  The weight
// fragments of a k half (AN reads of 16 bytes per lane) serve both row halves and are read with the first; every sub-step
// reads AM/2 activation fragments; both kinds are double-buffered in registers, so the reads of sub-step s+1 fly during
// the AM/2 * AN multiplies of sub-step s, and the other wave of the SIMD covers what still shows.  With one wave per SIMD
// (pipe::gemm_k_loop_spread) nothing covers a stall, and a burst of LDS reads stalls the issuing wave, multiplies
// included, until the LDS queue drains (16 reads in a row in front of 64 multiplies: 1840 cycles against 1055 for the
// multiplies alone; one read after every third multiply: 1080); there the fragments of a whole k half are
// double-buffered and every request sits between two multiplies.
template <int BM, int BN, int NW, int NS, int KS, int AM, int AN, bool NTW = false, bool ROT = false>
struct GemmTileExec {
    static constexpr int BK = 64, AH = AM / 2;
    static constexpr int LRA = BM / NW, LRW = BN / NW, LIA = LRA / 8, LIW = LRW / 8;
    static_assert(AM >= 2 && AH <= 4 && (AN == 4 || AN == 8), "wave tile shape");
    const half_t* pa[LIA];                 // this lane's source of each load instruction, K tile 0
    const half_t* pw[LIW];
    half_t* as_base;                       // stage 0 of this wave's K group: As[kg * NS], Ws[kg * NS]
    half_t* ws_base;
    unsigned a_lds, w_lds;                 // LDS byte address of this lane's row of the wave tile's first block, stage 0
    unsigned foff[2];                      // byte offset of this lane's 16 bytes of k half h inside the (permuted) row
    int kg, wave;
    half8v fa[2][AH], fw[2][AN];           // fa[s & 1]: activations of sub-step s; fw[h & 1]: weights of k half h
    half8v ga[2][AM], gw[2][AN];           // the one-wave-per-SIMD schedule: all fragments of k half h
    float4v acc[AM][AN];

    int k_first, k_count;                  // ROT: the walk over the K tiles starts at k_first and wraps at k_count

    __device__ __forceinline__ void load(int tile, int stage) {
        if constexpr (ROT) {
            tile += k_first;
            if (tile >= k_count) tile -= k_count;
        }
#pragma unroll
        for (int v = 0; v < LIA; ++v)
            load_lds_16B(pa[v] + (int64_t)(tile * KS + kg) * BK, as_base + stage * (BM * BK) + (wave * LRA + v * 8) * BK);
#pragma unroll
        for (int v = 0; v < LIW; ++v)
            load_lds_16B<NTW>(pw[v] + (int64_t)(tile * KS + kg) * BK, ws_base + stage * (BN * BK) + (wave * LRW + v * 8) * BK);
    }
    template <int L>
    __device__ __forceinline__ void wait_vmem() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L * (LIA + LIW)) : "memory");
    }
    __device__ __forceinline__ void barrier() { __builtin_amdgcn_s_barrier(); }
    // LDS reads of sub-step SUB: 16 bytes per lane per fragment, blocks 2 KB apart
    static constexpr int reads_of(int sub) { return AH + ((sub & 1) == 0 ? AN : 0); }
#define EET_DREAD(DST, ADDR, OFF) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(DST) : "v"(ADDR), "n"(OFF) : "memory")
    template <int BUF, int SUB>
    __device__ __forceinline__ void frag(int stage) {
        static_assert(BUF == (SUB & 1), "activation buffer of a sub-step");
        constexpr int H = SUB >> 1, MH = SUB & 1;
        const unsigned va_ = a_lds + stage * (BM * BK * 2) + foff[H];
        EET_DREAD(fa[BUF][0], va_, (MH * AH + 0) * 2048);
        if (AH > 1) EET_DREAD(fa[BUF][1 % AH], va_, (MH * AH + 1) * 2048);
        if (AH > 2) EET_DREAD(fa[BUF][2 % AH], va_, (MH * AH + 2) * 2048);
        if (AH > 3) EET_DREAD(fa[BUF][3 % AH], va_, (MH * AH + 3) * 2048);
        if (MH == 0) {
            const unsigned vw_ = w_lds + stage * (BN * BK * 2) + foff[H];
            static_assert(AN == 4, "wave tiles of 64 columns");
            EET_DREAD(fw[H][0], vw_, tile_column(0, 0) * 128);
            EET_DREAD(fw[H][1], vw_, tile_column(1, 0) * 128);
            EET_DREAD(fw[H][2], vw_, tile_column(2, 0) * 128);
            EET_DREAD(fw[H][3], vw_, tile_column(3, 0) * 128);
        }
    }
#undef EET_DREAD
    // The reads of sub-step SUB have landed; those of sub-step NEWER (issued after them; -1: none) may stay in flight.
    template <int BUF, int SUB, int NEWER>
    __device__ __forceinline__ void wait_frag() {
        static_assert(BUF == (SUB & 1), "activation buffer of a sub-step");
        asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(NEWER < 0 ? 0 : reads_of(NEWER & 3)) : "memory");
#pragma unroll
        for (int i = 0; i < AH; ++i) asm volatile("" : "+v"(fa[BUF][i]));      // the fragments are defined from here on
        if ((SUB & 1) == 0) {
#pragma unroll
            for (int j = 0; j < AN; ++j) asm volatile("" : "+v"(fw[SUB >> 1][j]));
        }
    }
    // ---- the one-wave-per-SIMD schedule (pipe::gemm_k_loop_spread): whole k halves, double-buffered -------------
    // LDS read number R of k half H into buffer H: the AN weight fragments, then the AM activation fragments
    template <int H, int R>
    __device__ __forceinline__ void half_read(unsigned va_, unsigned vw_) {
        if constexpr (R < AN) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(gw[H][R % AN]) : "v"(vw_), "n"(tile_column(R, 0) * 128) : "memory");
        else asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(ga[H][(R - AN) % AM]) : "v"(va_), "n"((R - AN) * 2048) : "memory");
    }
    template <int H, int... R>
    __device__ __forceinline__ void half_read_all(unsigned va_, unsigned vw_, std::integer_sequence<int, R...>) {
        (half_read<H, R>(va_, vw_), ...);
    }
    __device__ __forceinline__ void wait_fetched() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int j = 0; j < AN; ++j) asm volatile("" : "+v"(gw[h][j]));
#pragma unroll
            for (int i = 0; i < AM; ++i) asm volatile("" : "+v"(ga[h][i]));
        }
    }
    // multiply number IDX of k half H, followed by its share of the side work: the reads of the other k half and the tile
    // loads of one operand (LOADS: 1 the activations, 2 the weights), each spread over the first three quarters of the phase (the last quarter
    // lets the reads land; loads issued later arrive later); scheduling barriers pin each request between the two multiplies it was written between
    template <int H, int LOADS, int IDX>
    __device__ __forceinline__ void half_mma_one(unsigned va_, unsigned vw_, int64_t koff, int lstage) {
        constexpr int MF = AM * AN, NR = AM + AN, NL = LOADS == 1 ? LIA : LIW;
        constexpr int RS = (MF * 3 / 4) / NR, LS = (MF * 3 / 4) / NL;       // multiplies per read, per load (256 x 256 tile, 64 multiplies: 3 and 6)
        static_assert(RS >= 1 && LS >= 1, "side work fits between the multiplies");
        constexpr int i = IDX / AN, j = IDX % AN;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(gw[H][j], ga[H][i], acc[i][j], 0, 0, 0);
        if constexpr (IDX % RS == 0 && IDX / RS < NR) {
            __builtin_amdgcn_sched_barrier(0);
            half_read<1 - H, IDX / RS>(va_, vw_);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (IDX % LS == LS / 2 && IDX / LS < NL) {
            constexpr int v = IDX / LS;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (LOADS == 1) load_lds_16B(pa[v % LIA] + koff, as_base + lstage * (BM * BK) + (wave * LRA + v * 8) * BK);
            else load_lds_16B(pw[v % LIW] + koff, ws_base + lstage * (BN * BK) + (wave * LRW + v * 8) * BK);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    template <int H, int LOADS, int... I>
    __device__ __forceinline__ void half_mma_seq(unsigned va_, unsigned vw_, int64_t koff, int lstage, std::integer_sequence<int, I...>) {
        __builtin_amdgcn_sched_barrier(0);
        (half_mma_one<H, LOADS, I>(va_, vw_, koff, lstage), ...);
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ int64_t column(int tile) { return (int64_t)(tile * KS + kg) * BK; }    // first column of this group's K tile `tile`
    __device__ __forceinline__ void load_a(int tile, int stage) {
#pragma unroll
        for (int v = 0; v < LIA; ++v) load_lds_16B(pa[v] + column(tile), as_base + stage * (BM * BK) + (wave * LRA + v * 8) * BK);
    }
    __device__ __forceinline__ void load_w(int tile, int stage) {
#pragma unroll
        for (int v = 0; v < LIW; ++v) load_lds_16B(pw[v] + column(tile), ws_base + stage * (BN * BK) + (wave * LRW + v * 8) * BK);
    }
    template <int LA, int LW>
    __device__ __forceinline__ void wait_loads() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LA * LIA + LW * LIW) : "memory");
    }
    template <int H>
    __device__ __forceinline__ void fetch_half(int astage, int wstage) {
        half_read_all<H>(a_lds + astage * (BM * BK * 2) + foff[H], w_lds + wstage * (BN * BK * 2) + foff[H], std::make_integer_sequence<int, AM + AN>{});
    }
    template <int H>
    __device__ __forceinline__ void mma_fetch_load_a(int astage, int wstage, int tile, int lstage) {
        half_mma_seq<H, 1>(a_lds + astage * (BM * BK * 2) + foff[1 - H], w_lds + wstage * (BN * BK * 2) + foff[1 - H], column(tile), lstage,
                           std::make_integer_sequence<int, AM * AN>{});
    }
    template <int H>
    __device__ __forceinline__ void mma_fetch_load_w(int astage, int wstage, int tile, int lstage) {
        half_mma_seq<H, 2>(a_lds + astage * (BM * BK * 2) + foff[1 - H], w_lds + wstage * (BN * BK * 2) + foff[1 - H], column(tile), lstage,
                           std::make_integer_sequence<int, AM * AN>{});
    }
    template <int BUF, int SUB>
    __device__ __forceinline__ void mma() {
        static_assert(BUF == (SUB & 1), "activation buffer of a sub-step");
        constexpr int H = SUB >> 1, MH = SUB & 1;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < AH; ++i)
#pragma unroll
            for (int j = 0; j < AN; ++j)
                acc[MH * AH + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fw[H][j], fa[BUF][i], acc[MH * AH + i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
};

// SCHED: 0 = the schedule of pipe::gemm_k_loop<NS>; the schedule for one wave per SIMD (wave tiles of an odd number of 16-row blocks too; and for the
// two K groups of a small tile, two waves per SIMD, whose few multiplies per step want every request spread just as much) with NS stages of both operands, 2 = pipe::gemm_k_loop_spread<NS, NS>, or with one more of the activations, 1 = <NS + 1, NS>.
// us, all loads of a step behind its barrier -> spread over both halves (rows x N x K): 256 x 256 tiles, two stages -> three and two: 3262 x 4096 x 4096
// 95.9 -> 88.1, 6758 x 2048 x 8192 208 -> 186, 3262 x 4096 x 16384 351 -> 324, 12288 x 4096 x 12288 932 -> 873, 4096 x 8192 x 32768 2192 -> 1532 (rows
// 64 KB apart; 128 bytes further 1884 -> 1532), at K = 2048 0 to 2 %; pairs of 128 x 128: 1200 x 6144 x 2048 33.5 -> 31.9; 192 x 128: 700 x 6144 x
// 2048 24.4 -> 22.4; two K groups, from gemm_k_loop<3>: 300 x 1024 x 4096 17.4 -> 14.3, 100 x 8192 x 2048 11.3 -> 9.9, 300 x 1536 x 1536 9.0 -> 8.2, 160 x 2304 x
// 768 6.5 -> 6.2 (the weight stream of 17 to 128 rows gains nothing: 120 x 12288 x 12288 79.2 -> 81.7, and one row tile over weights past the L2 loses:
// tile_rules.hpp, reads_weights_past_l2); 96 x 128: 1200 x 2048 x 2048 15.4 -> 14.5, 3054 x 1024 x 4096 29.5 -> 28.4; 128 x 256: 400 x 12288 x 4096 55.4 -> 54.5.  More stages
// than these gain nothing (96 x 128 in five, 192 x 128 in four, 128 x 256 in four and three: level or 1 to 3 % slower).
// NTS: the output is stored with the non-temporal hint (outputs of 256 MB and more, which no cache keeps for their reader:
// 24576 x 49152 x 12288 21.70 -> 21.53 ms, 24576 x 12288 x 12288 5.69 -> 5.59, 8192 x 16384 x 12288 2.436 -> 2.393).
// NTW: the weights are loaded with the non-temporal hint (one row tile: every weight is read once by the launch).
// ROT: the workgroups of an XCD start their walk over K in eight different places and wrap, as in gemm_stream, so that not
// all of them ask for the same K offset of weight rows a power of two apart, and for the same activation lines, at the same
// time (48 x 16384 x 4096: 28.0 -> 24.9 us, 48 x 4096 x 16384 in four K ranges: 37.2 -> 29.1).
// EPI_PARTIAL: the K range is cut into a.k_ranges parts, one workgroup per tile and part, and the fp32 accumulators go
// to a.part[range][row][column] for finish_rows to add up.
template <int BM, int BN, int WGM, int WGN, int EPI, int NS, int KS, int SCHED, bool NTS = false, bool NTW = false, bool ROT = false>
// (192 x 128 tiles are made for two workgroups per CU: the residual and cache-row look-ups of their epilogue would take the
// kernel past 256 registers and halve that: 2000 x 4096 x 4096 with a residual 135 us)
__global__ __launch_bounds__(WGM* WGN* KS * 64, BM == 192 && BN == 128 && NS == 2 ? 2 : 1) void gemm_mfma_dma64(GemmArgs a, int tiles_m, int tiles_n) {
    static_assert(SCHED == 0 || (!NTW && !ROT && (SCHED == 1 || (SCHED == 2 && NS > 2))), "schedule");
    // KS > 1: KS groups of WGM x WGN waves share the tile and take every KS-th K step each, through LDS stages of their
    // own; the other groups' accumulators are added to the first's through LDS at the end.  For the few
    // tiles of a narrow output with a long K, where nothing else puts more loads in flight per CU.
    constexpr int NW = WGM * WGN, BK = 64;
    static_assert(NS == 2 || NS == 3 || (NS == 4 && SCHED == 2), "LDS stages");
    static_assert(KS == 1 || KS == 2 || KS == 4, "K groups");
    constexpr int WM = BM / WGM, WN = BN / WGN, AM = WM / 16, AN = WN / 16;   // wave tile in 16 x 16 accumulator blocks
    constexpr int LRA = BM / NW, LRW = BN / NW;   // rows of each operand tile a wave loads per K step
    constexpr int LIA = LRA / 8, LIW = LRW / 8;   // wave-level load instructions per operand per K step
    static_assert(LRA % 8 == 0 && LRW % 8 == 0 && LIA >= 1 && LIW >= 1 && WM % (SCHED != 0 ? 16 : 32) == 0 && (WN == 64 || WN == 128), "tile shape");
    constexpr int NSA = SCHED == 1 ? NS + 1 : NS;            // stages of the activations
    __shared__ __attribute__((aligned(1024))) half_t As[KS * NSA][BM * BK];
    __shared__ __attribute__((aligned(1024))) half_t Ws[KS * NS][BN * BK];

    int tile_m, tile_n;
    int range = 0;                                           // K range of this workgroup
    if constexpr (EPI == EPI_PARTIAL) {
        // consecutive workgroups, which go to different XCDs, take different ranges: with 2, 4 or 8 of them an XCD's L2
        // holds the activations of one range only
        range = (int)blockIdx.x % a.k_ranges;
        const int t = (int)blockIdx.x / a.k_ranges;
        tile_m = t % tiles_m;
        tile_n = t / tiles_m;
    } else {
        pipe::tile_of_block((int)blockIdx.x, tiles_m, tiles_n, tile_m, tile_n);
    }
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform by construction: keeps LDS bases in scalar registers
    const int kg = KS == 1 ? 0 : wv / NW;                    // K group of this wave
    const int wave = KS == 1 ? wv : wv % NW;                 // wave inside its group
    const int wm0 = (wave / WGN) * WM, wn0 = (wave % WGN) * WN;
    const int M = a.M, N = a.N, K = a.K;
    // steps of this group (the host sends whole multiples); the ranges of a cut K differ by at most one step
    const int k_step0 = EPI == EPI_PARTIAL ? K / (BK * KS) * range / a.k_ranges : 0;
    const int nk = (EPI == EPI_PARTIAL ? K / (BK * KS) * (range + 1) / a.k_ranges : K / (BK * KS)) - k_step0;
    const int k0 = k_step0 * (BK * KS);

    GemmTileExec<BM, BN, NW, NS, KS, AM, AN, NTW, ROT> ex;
    static_assert(decltype(ex)::LIA == LIA && decltype(ex)::LIW == LIW, "load instructions per K step");
    ex.kg = kg;
    ex.wave = wave;
    if constexpr (ROT) {
        ex.k_first = (((int)blockIdx.x >> 3) & 7) * nk >> 3;
        ex.k_count = nk;
    }
    ex.as_base = &As[kg * NSA][0];
    ex.ws_base = &Ws[kg * NS][0];
#pragma unroll
    for (int v = 0; v < LIA; ++v) {
        const int row = wave * LRA + v * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((row >> 1) & 7);
        int gr = m0 + row;
        gr = gr < M ? gr : M - 1;
        ex.pa[v] = a.x + (int64_t)gr * (a.lda ? a.lda : K) + k0 + c * 8;
    }
#pragma unroll
    for (int v = 0; v < LIW; ++v) {
        const int row = wave * LRW + v * 8 + (lane >> 3);
        const int c = (lane & 7) ^ (((row >> 1) & 1) | ((row >> 3) & 3) << 1);    // of the rows tile_column(j, 0..15), two share a permutation each
        int gr = n0 + row;
        gr = gr < N ? gr : N - 1;
        ex.pw[v] = a.w + (int64_t)gr * K + k0 + c * 8;
    }
    // fragment rows: lane l reads operand row l%16 of a block (of the weights: row tile_column(j, l%16) of the wave tile), the 16 bytes (l/16) of k half
    // h; rows are 128 bytes with their 16-byte chunks XOR-permuted by (operand row)/2, so the permutation is the lane's own
    const int frow = lane & 15, fG = lane >> 4, fsw = frow >> 1;
    ex.a_lds = (unsigned)(uintptr_t)&As[kg * NSA][(wm0 + frow) * BK];
    ex.w_lds = (unsigned)(uintptr_t)&Ws[kg * NS][(wn0 + tile_column(0, frow)) * BK];
#pragma unroll
    for (int h = 0; h < 2; ++h) ex.foff[h] = (unsigned)(((h * 4 + fG) ^ fsw) * 16);

    float4v (&acc)[AM][AN] = ex.acc;
#pragma unroll
    for (int i = 0; i < AM; ++i)
#pragma unroll
        for (int j = 0; j < AN; ++j) acc[i][j] = float4v{0.f, 0.f, 0.f, 0.f};
    if constexpr (SCHED != 0) pipe::gemm_k_loop_spread<NSA, NS>(ex, nk);
    else pipe::gemm_k_loop<NS>(ex, nk);

    if constexpr (KS > 1) {
        __syncthreads();                                  // every wave is done with the operand stages
        // the other groups' partial tiles go over the weight stages, lane-major (no bank conflicts), to the first
        constexpr int PT = AM * AN * 4 * 64;                  // floats of one wave's partial tile
        static_assert((KS - 1) * NW * PT * 4 <= (int)sizeof(Ws), "partial tiles over the weight stages");
        float* red = reinterpret_cast<float*>(&Ws[0][0]) + wave * PT + lane;
        if (kg > 0) {
            float* mine = red + (kg - 1) * (NW * PT);
#pragma unroll
            for (int i = 0; i < AM; ++i)
#pragma unroll
                for (int j = 0; j < AN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mine[((i * AN + j) * 4 + r) * 64] = acc[i][j][r];
        }
        __syncthreads();
        if (kg > 0) return;
#pragma unroll
        for (int g = 0; g < KS - 1; ++g)
#pragma unroll
            for (int i = 0; i < AM; ++i)
#pragma unroll
                for (int j = 0; j < AN; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[i][j][r] += red[g * (NW * PT) + ((i * AN + j) * 4 + r) * 64];
    }
    if constexpr (EPI == EPI_PARTIAL) {
#pragma unroll
        for (int i = 0; i < AM; ++i) {
            const int m = m0 + wm0 + i * 16 + (lane & 15);
            if (m >= M) continue;
#pragma unroll
            for (int j = 0; j < AN; ++j) {
                const int n = n0 + wn0 + tile_column(j, (lane >> 4) * 4);
                if (n < N) *reinterpret_cast<float4v*>(a.part + ((int64_t)range * M + m) * N + n) = acc[i][j];
            }
        }
        return;
    }
    if constexpr (NS == 2 && BN == 128 && (EPI == EPI_BIAS || EPI == EPI_BIAS_RES)) {
        __syncthreads();                                  // every wave is done with the operand stages
        static_assert(NW * WM * 128 <= (int)sizeof(As) && !NTS, "turn-around areas");
        epilogue_via_lds<AM, EPI>(a, acc, reinterpret_cast<char*>(&As[0][0]) + wave * WM * 128, m0 + wm0, n0 + wn0, lane);
    } else {
        epilogue_tile<AM, AN, EPI, NTS>(a, acc, m0 + wm0, n0 + wn0, lane);
    }
}

// --------------------------------------------------------------------------------------------
// weight-streaming kernel for M <= 16 rows per grid.y slice
// --------------------------------------------------------------------------------------------
// Workgroup = NW waves; it owns 16*NF output columns.  K steps of 32 are dealt round-robin to
// the waves (adjacent waves read adjacent 64-byte pieces of the same weight rows).
// LN = true fuses the LayerNorm that precedes the projection (decode: LN1 -> QKV, LN2 -> FFN-1):
// every workgroup first computes mean and 1/std of its <= 16 activation rows (two passes over
// rows that stay in L1/L2), then normalises the activation fragments on their way into the MFMA,
// so the normalised activations never exist in memory and one launch per projection is saved.
// BUMP: the workgroup with blockIdx 0 also advances the per-sequence cache lengths (n_b += 1).
template <int NF, int EPI, bool LN, int NW>
__global__ __launch_bounds__(NW * 64) void gemm_skinny(GemmArgs a) {
    constexpr int UN = 4;                       // K steps in flight per wave
    __shared__ float red[NW][NF * 16][17];
    __shared__ float ln_mean[16], ln_rstd[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, G = lane >> 4;
    const int n0 = blockIdx.x * (NF * 16), mc = blockIdx.y * 16;
    const int M = a.M, N = a.N, K = a.K;
    const int nsteps = K / 32;

    if (a.bump_lens != nullptr && blockIdx.x == 0 && blockIdx.y == 0 && tid < a.bump_count) a.bump_lens[tid] += 1;

    int xr = mc + fr;
    xr = xr < M ? xr : M - 1;
    const half_t* xp = a.x + (int64_t)xr * K + G * 8;
    const half_t* wp[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        int wr = n0 + f * 16 + fr;
        wr = wr < N ? wr : N - 1;
        wp[f] = a.w + (int64_t)wr * K + G * 8;
    }
    float4v acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = float4v{0.f, 0.f, 0.f, 0.f};

    // The weight (and gamma/beta) fragments of a chunk of UN K steps are requested one chunk ahead
    // of their use; the first chunk is requested before the LayerNorm statistics, whose latency
    // (two passes over cached activation rows) then hides behind the first trip to HBM.
    half8v xf[UN], wf[UN][NF], gf[UN], bf[UN];
    auto request = [&](int s0) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int step = s0 + NW * u;
            const int k = (step < nsteps ? step : wave) * 32;      // past the end: any valid step, zeroed below
            xf[u] = *reinterpret_cast<const half8v*>(xp + k);
            if (LN) {
                gf[u] = *reinterpret_cast<const half8v*>(a.ln_gamma + k + G * 8);
                bf[u] = *reinterpret_cast<const half8v*>(a.ln_beta + k + G * 8);
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) wf[u][f] = *reinterpret_cast<const half8v*>(wp[f] + k);
        }
    };
    if (wave < nsteps) request(wave);
    float mean = 0.f, rstd = 1.f;
    if (LN) {
        // 16 threads per row: thread (row = tid/16, sub = tid%16) walks the row in 16-byte vectors
        const int row = (tid >> 4) & 15, sub = tid & 15;       // (workgroups wider than 256 threads repeat the work)
        int rr = mc + row;
        rr = rr < M ? rr : M - 1;
        const half_t* rp = a.x + (int64_t)rr * K;
        // loads go out in batches of 8 independent 16-byte vectors (a scalar loop would pay one
        // memory round trip per vector)
        float sum = 0.f;
        for (int c0 = sub * 8; c0 < K; c0 += 8 * 128) {
            half8v v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int cidx = c0 + i * 128;
                v[i] = *reinterpret_cast<const half8v*>(rp + (cidx < K ? cidx : sub * 8));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (c0 + i * 128 < K) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) sum += (float)v[i][e];
                }
        }
        sum = reduce16(sum, [](float x, float y) { return x + y; });
        const float mu = sum / (float)K;
        float sq = 0.f;
        for (int c0 = sub * 8; c0 < K; c0 += 8 * 128) {
            half8v v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int cidx = c0 + i * 128;
                v[i] = *reinterpret_cast<const half8v*>(rp + (cidx < K ? cidx : sub * 8));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (c0 + i * 128 < K) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float dlt = (float)v[i][e] - mu;
                        sq += dlt * dlt;
                    }
                }
        }
        sq = reduce16(sq, [](float x, float y) { return x + y; });
        if (sub == 0) {
            ln_mean[row] = mu;
            ln_rstd[row] = rsqrtf(sq / (float)K + a.ln_eps);
        }
        __syncthreads();
        mean = ln_mean[fr];
        rstd = ln_rstd[fr];
    }
    for (int s0 = wave; s0 < nsteps; s0 += NW * UN) {
        half8v cx[UN], cw[UN][NF];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            cx[u] = xf[u];
            if (LN) {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    cx[u][e] = (half_t)(((float)xf[u][e] - mean) * rstd * (float)gf[u][e] + (float)bf[u][e]);
            }
            if (s0 + NW * u >= nsteps) {
#pragma unroll
                for (int e = 0; e < 8; ++e) cx[u][e] = (half_t)0.f;
            }
#pragma unroll
            for (int f = 0; f < NF; ++f) cw[u][f] = wf[u][f];
        }
        if (s0 + NW * UN < nsteps) request(s0 + NW * UN);            // next chunk in flight during the MFMAs
#pragma unroll
        for (int u = 0; u < UN; ++u)
#pragma unroll
            for (int f = 0; f < NF; ++f)
                acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(cw[u][f], cx[u], acc[f], 0, 0, 0);
    }
    // acc[f][r]: output column n0 + f*16 + 4G + r, row mc + lane%16
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][f * 16 + 4 * G + r][fr] = acc[f][r];
    __syncthreads();
    for (int t = tid; t < 64 * NF; t += NW * 64) {
        const int ng = t % (4 * NF), ml = t / (4 * NF);
        const int m = mc + ml, n = n0 + ng * 4;
        if (m >= M || n >= N) continue;
        float v[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            float part = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) part += red[w][ng * 4 + c][ml];
            v[c] = part;
        }
        epilogue4<EPI>(a, m, n, v[0], v[1], v[2], v[3]);
    }
}

// --------------------------------------------------------------------------------------------
// latency-bound variant of the weight-streaming kernel (small layers)
// --------------------------------------------------------------------------------------------
// When one projection moves only a few MB, its time is a chain of memory round trips plus the
// instructions each wave has to issue (a wave64 vector instruction takes 4 cycles: a thousand of
// them are two microseconds), not bytes.  This variant is built for both:
//   * K = 64 * NW * UPW is a compile-time constant (NW waves, UPW units of 64 K values per wave),
//     so address arithmetic folds into immediate offsets and nothing is conditional;
//   * a workgroup owns TN = 16 output columns (8 when 16 would leave most CUs without work: the
//     staging rows 8..15 then hold nothing and their results are dropped); every wave requests its whole share of the weights at
//     once, after the activation rows and before the epilogue's bias / residual / cache slot:
//     one round trip to memory in all;
//   * every load instruction reads whole 128-byte lines (8 lanes x 16 bytes per row; measured on
//     this part: an instruction that takes 64 bytes from each of 16 lines, which is what the MFMA
//     operand layout asks for, moves data several times slower out of L2).  The MFMA layout is
//     produced in LDS instead: a wave writes each 16 x 128-byte unit it loaded into a private
//     staging area and reads back 16 bytes per lane at (row lane%16, chunk lane/16 + 4u) for the
//     two MFMAs u of the unit.  LDS operations of one wave execute in order, so the private
//     areas need no barrier (and the wave's partial sums reuse the first one);
//   * the activation rows (8, or 16 when M > 8; rows past M repeat row M-1 and their results
//     are never written) are read as contiguous 16-byte vectors spread over all threads and
//     shared through LDS: one barrier, after which every operand fragment is a 16-byte LDS read.
//     With LN a row belongs to 8*NW lanes of one wave: its statistics are reduced by lane
//     exchanges over values held in registers, and the row reaches LDS normalised.
//
// Dynamic LDS: [8 or 16][K + 8] activations, then per wave SA staging areas of 16 x 144 bytes.
constexpr int kFlatStageRow = 72;                           // halves per staged row: 128 bytes + 16 padding
__host__ __device__ constexpr int flat_stage_areas(int nw, int upw) { return (nw >= 16 && upw > 2) ? 2 : upw; }
__host__ __device__ constexpr int flat_lds_bytes(int nw, int upw, int xrows) {
    return xrows * (64 * nw * upw + 8) * 2 + nw * flat_stage_areas(nw, upw) * 16 * kFlatStageRow * 2;
}

// sum over aligned groups of W lanes (W = 32 or 64), result in every lane of the group
template <int W>
__device__ __forceinline__ float group_sum(float v) {
    v += dpp<0xb1>(v);                                      // quad_perm [1,0,3,2]: lane ^ 1
    v += dpp<0x4e>(v);                                      // quad_perm [2,3,0,1]: lane ^ 2
    v += dpp<0x141>(v);                                     // row_half_mirror: the other quad of 8
    v += dpp<0x140>(v);                                     // row_mirror: the other half of 16
    v = sum_xor16(v);
    if (W == 64) v = sum_xor32(v);
    return v;
}

// A launch of the weight-streaming kernels with gridDim.y > 1 (template flag SL) cuts the rows into slices of 16: the
// workgroups of row blockIdx.y see rows [16 y, 16 y + 16) as a problem of their own (a decode step of 17 to 64
// sequences: the slices run side by side and all but the first find the weights in L2).  Used without row maps, fused
// LayerNorm, prefetch workgroups or length bump.  A flag of its own because even this much scalar arithmetic shows in
// the launch-bound decode of small layers (0.2 % of the 24-layer pass).
template <int EPI>
__device__ __forceinline__ void take_row_slice(GemmArgs& a) {
    const int m0 = (int)blockIdx.y * 16;
    const int rows = a.M - m0;
    a.M = rows < 16 ? rows : 16;
    a.x += (size_t)m0 * a.K;
    if (EPI == EPI_QKV) {                       // decode: row m is sequence m, its token goes to slot lens[m] of its own cache
        a.y += (size_t)m0 * a.hidden;
        a.lens += m0;
        const size_t seq = (size_t)a.heads * a.max_seq * a.d;
        a.k_cache += (size_t)m0 * seq;
        a.v_cache += (size_t)m0 * seq;
    } else {
        a.y += (size_t)m0 * a.N;
        if (EPI == EPI_BIAS_RES) a.res += (size_t)m0 * a.N;
    }
}

template <int NW, int UPW, int TN, int EPI, bool LN, bool SL, bool XM = false>
__global__ __launch_bounds__(NW * 64) void gemm_flat(GemmArgs a) {
    static_assert(!XM || (EPI == EPI_BIAS_RES && !LN && !SL), "merging attention ranges: the output projection of a decode step");
    if (SL) take_row_slice<EPI>(a);
    constexpr int NT = NW * 64;
    constexpr int K = 64 * NW * UPW, KV = K / 8, LDX = K + 8;   // LDX: 16-byte reads of 16 rows spread over all banks
    constexpr int SA = flat_stage_areas(NW, UPW);
    constexpr int TPR = NT / 8;                             // LN: lanes per activation row (32 or 64)
    static_assert(!LN || TPR <= 64, "a row's statistics are reduced inside one wave");
    extern __shared__ __attribute__((aligned(16))) unsigned char flat_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, G = lane >> 4;
    constexpr int WA = TN / 8;                              // load instructions per unit (8 weight rows each)
    const int n0 = blockIdx.x * TN;
    const int M = a.M;
    const int xrows = M <= 8 ? 8 : 16;
    half_t* xs = reinterpret_cast<half_t*>(flat_smem);
    half_t* wst = xs + xrows * LDX + wave * (SA * 16 * kFlatStageRow);
    float* red = reinterpret_cast<float*>(xs + xrows * LDX);            // after the MFMAs: wave w's tile over its staging areas
    constexpr int RW = SA * 16 * kFlatStageRow / 2;                     // floats between the waves' tiles
    static_assert(RW >= 16 * 20, "partial-sum tile must fit the wave's own staging space");

    if (a.pf.blocks > 0 && (int)blockIdx.x >= a.N / TN) {   // extra workgroups: operands of the launches that follow
        run_prefetch(a.pf, (int)blockIdx.x - a.N / TN, a.pf.blocks, tid, NT);
        return;
    }
    if (a.bump_lens != nullptr && blockIdx.x == 0 && tid < a.bump_count) a.bump_lens[tid] += 1;

    // ---- requests, oldest first: activations, weights, epilogue operands --------------------
    // half h of the activations = rows 8h .. 8h+7; thread -> (row, 16-byte vectors) per half:
    //   LN:  row tid/TPR, vectors tid%TPR + TPR*i      (a row stays inside one wave)
    //   else: vector tid + NT*i of the 8*KV vectors of the half
    half8v xv[2][UPW], gv[LN ? UPW : 1], bv[LN ? UPW : 1];
    uint32_t xdst[UPW];                                       // LDS offset (halves) of vector i inside a half
    auto request_x = [&](int h) {
#pragma unroll
        for (int i = 0; i < UPW; ++i) {
            const int row = LN ? tid / TPR : (tid + NT * i) / KV;
            const int col = LN ? tid % TPR + TPR * i : (tid + NT * i) % KV;
            int src = 8 * h + row;
            src = src < M ? src : M - 1;
            xv[h][i] = *reinterpret_cast<const half8v*>(reinterpret_cast<const char*>(a.x) + (uint32_t)(src * K + col * 8) * 2u);
            xdst[i] = row * LDX + col * 8;
            if (LN && h == 0) {
                gv[i] = *reinterpret_cast<const half8v*>(reinterpret_cast<const char*>(a.ln_gamma) + (uint32_t)col * 16u);
                bv[i] = *reinterpret_cast<const half8v*>(reinterpret_cast<const char*>(a.ln_beta) + (uint32_t)col * 16u);
            }
        }
    };
    if (!XM) {
        request_x(0);
        if (M > 8) request_x(1);
    }
    // weights: per unit, lane l takes 16 bytes (chunk l%8) of rows l/8 and 8 + l/8
    const int wrow = lane >> 3, wchunk = lane & 7;
    half8v wreg[UPW][WA];
    {
        const char* wbase = reinterpret_cast<const char*>(a.w) + (size_t)n0 * K * 2;
        const uint32_t woff = (uint32_t)(wrow * K + wave * (UPW * 64) + wchunk * 8) * 2u;
#pragma unroll
        for (int q = 0; q < UPW; ++q)
#pragma unroll
            for (int h = 0; h < WA; ++h)
                wreg[q][h] = *reinterpret_cast<const half8v*>(wbase + woff + (uint32_t)(h * 8 * K + q * 64) * 2u);
    }
    // epilogue operands of the 4*TN threads that write the 16 x TN outputs (no row maps in decode)
    const int eml = tid / (TN / 4), enl = (tid % (TN / 4)) * 4, en = n0 + enl;
    const bool writer = tid < 4 * TN && eml < M;
    EpiOperands eo;
    if (writer) {
        eo.bias = *reinterpret_cast<const half4v*>(a.bias + en);
        if (EPI == EPI_BIAS_RES) eo.res = *reinterpret_cast<const half4v*>(a.res + (uint32_t)(eml * a.N + en));
        if (EPI == EPI_QKV) eo.pos = a.lens[eml];
    }

    // ---- XM: the activations are the attention output of this step, one partial per key range; merge them ----
    // (what attn_decode_combine does in a launch of its own: common maximum, rescaled sums, one division)
    if constexpr (XM) {
        constexpr int MAXS = NW >= 16 ? 2 : 8;                  // ranges in flight at a time (1024 threads: 128 VGPRs each)
        const int splits = a.x_splits;
        auto merge_x = [&](int h) {
#pragma unroll
            for (int i = 0; i < UPW; ++i) {
                const int row = (tid + NT * i) / KV, col = (tid + NT * i) % KV;
                const int src = 8 * h + row;
                xdst[i] = row * LDX + col * 8;
                half8v o;
#pragma unroll
                for (int e = 0; e < 8; ++e) o[e] = (half_t)0.f;
                if (src < M) {                                  // rows past M feed outputs nobody writes
                    const int g = (col * 8) / a.d, dd = (col * 8) % a.d;
                    const int64_t bh = (int64_t)src * a.heads + g;
                    const float* ml = a.x_part_ml + bh * splits * 2;
                    const float* pa = a.x_part_acc + bh * splits * a.d + dd;
                    float lsum = 0.f, av[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) av[e] = 0.f;
                    auto fetch = [&](int s0, float2v (&mlv)[MAXS], float4v (&lo)[MAXS], float4v (&hi)[MAXS]) {
#pragma unroll
                        for (int u = 0; u < MAXS; ++u) {
                            const int s = s0 + u < splits ? s0 + u : splits - 1;
                            mlv[u] = *reinterpret_cast<const float2v*>(ml + s * 2);
                            lo[u] = *reinterpret_cast<const float4v*>(pa + (int64_t)s * a.d);
                            hi[u] = *reinterpret_cast<const float4v*>(pa + (int64_t)s * a.d + 4);
                        }
                    };
                    auto add = [&](int s0, float mx, const float2v (&mlv)[MAXS], const float4v (&lo)[MAXS], const float4v (&hi)[MAXS]) {
#pragma unroll
                        for (int u = 0; u < MAXS; ++u) {
                            const float sc = s0 + u < splits ? exp2f(mlv[u][0] - mx) : 0.f;
                            lsum += mlv[u][1] * sc;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                av[e] += lo[u][e] * sc;
                                av[4 + e] += hi[u][e] * sc;
                            }
                        }
                    };
                    float2v mlv[MAXS];
                    float4v lo[MAXS], hi[MAXS];
                    if (splits <= MAXS) {                       // the usual case: everything in one trip to memory
                        fetch(0, mlv, lo, hi);
                        float mx = mlv[0][0];                   // empty ranges report a finite maximum and a zero sum (clamped slots repeat the last range)
#pragma unroll
                        for (int u = 1; u < MAXS; ++u) mx = fmaxf(mx, mlv[u][0]);
                        add(0, mx, mlv, lo, hi);
                    } else {
                        float mx = -INFINITY;
                        for (int s = 0; s < splits; ++s) mx = fmaxf(mx, ml[s * 2]);
                        for (int s0 = 0; s0 < splits; s0 += MAXS) {
                            fetch(s0, mlv, lo, hi);
                            add(s0, mx, mlv, lo, hi);
                        }
                    }
                    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;     // a pair that saw no key at all: zeros, not 0/0
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = (half_t)(av[e] * inv);
                }
                xv[h][i] = o;
            }
        };
        merge_x(0);
        if (M > 8) merge_x(1);
    }

    // ---- activations -> LDS (normalised when LN) ----------------------------------------------
    auto publish_x = [&](int h) {
        if (LN) {
            // shifted sums: d = x - p with p the row's first element keeps the variance formula
            // free of cancellation whatever the row's mean is
            const half_t p = (half_t)__shfl((float)xv[h][0][0], lane & ~(TPR - 1), kWave);
            const half2v p2 = {p, p}, one2 = {(half_t)1.f, (half_t)1.f};
            float sd = 0.f, sq = 0.f;
#pragma unroll
            for (int i = 0; i < UPW; ++i)
#pragma unroll
                for (int e = 0; e < 8; e += 2) {
                    const half2v d2 = half2v{xv[h][i][e], xv[h][i][e + 1]} - p2;
                    sd = __builtin_amdgcn_fdot2(d2, one2, sd, false);
                    sq = __builtin_amdgcn_fdot2(d2, d2, sq, false);
                }
            sd = group_sum<TPR>(sd);
            sq = group_sum<TPR>(sq);
            const float md = sd * (1.0f / K);
            const float mu = (float)p + md;
            const float rstd = rsqrtf(fmaxf(sq * (1.0f / K) - md * md, 0.f) + a.ln_eps);
#pragma unroll
            for (int i = 0; i < UPW; ++i) {
                half8v o;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    // three fused multiply-adds that take their fp16 operand directly
                    const float sc = __builtin_fmaf((float)gv[i][e], rstd, 0.f);
                    const float sh = __builtin_fmaf(-mu, sc, (float)bv[i][e]);
                    o[e] = (half_t)__builtin_fmaf((float)xv[h][i][e], sc, sh);
                }
                *reinterpret_cast<half8v*>(&xs[8 * h * LDX + xdst[i]]) = o;
            }
        } else {
#pragma unroll
            for (int i = 0; i < UPW; ++i) *reinterpret_cast<half8v*>(&xs[8 * h * LDX + xdst[i]]) = xv[h][i];
        }
    };
    publish_x(0);
    if (M > 8) publish_x(1);

    // ---- weights -> MFMA layout, contraction ---------------------------------------------------
    const uint32_t st_w = (uint32_t)(wrow * kFlatStageRow + wchunk * 8);                  // staging write (halves)
    const uint32_t st_r = (uint32_t)(fr * kFlatStageRow + G * 8);                         // staging read
    const uint32_t xs_r = (uint32_t)((fr & (xrows - 1)) * LDX + wave * (UPW * 64) + G * 8);
    float4v acc = float4v{0.f, 0.f, 0.f, 0.f};
    auto stage = [&](int q0, int n) {
#pragma unroll
        for (int j = 0; j < n; ++j)
#pragma unroll
            for (int h = 0; h < WA; ++h)
                *reinterpret_cast<half8v*>(&wst[st_w + (j * 16 + 8 * h) * kFlatStageRow]) = wreg[q0 + j][h];
    };
    auto contract = [&](int q0, int n) {
        half8v wf[SA][2], xf[SA][2];
#pragma unroll
        for (int j = 0; j < n; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                wf[j][u] = *reinterpret_cast<const half8v*>(&wst[st_r + j * 16 * kFlatStageRow + 32 * u]);
                xf[j][u] = *reinterpret_cast<const half8v*>(&xs[xs_r + (q0 + j) * 64 + 32 * u]);
            }
#pragma unroll
        for (int j = 0; j < n; ++j)
#pragma unroll
            for (int u = 0; u < 2; ++u) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf[j][u], xf[j][u], acc, 0, 0, 0);
    };
    stage(0, SA);
    __syncthreads();
    contract(0, SA);
    if (SA < UPW) {
        __builtin_amdgcn_wave_barrier();
        stage(SA, UPW - SA);
        __builtin_amdgcn_wave_barrier();
        contract(SA, UPW - SA);
    }
    __builtin_amdgcn_wave_barrier();
    // acc[r]: output column n0 + 4G + r, row fr
    *reinterpret_cast<float4v*>(&red[wave * RW + fr * 20 + 4 * G]) = acc;
    __syncthreads();
    if (writer) {
        const float* rp = &red[eml * 20 + enl];
        float4v v = *reinterpret_cast<const float4v*>(rp);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            const float4v pw = *reinterpret_cast<const float4v*>(rp + w * RW);
            v[0] += pw[0]; v[1] += pw[1]; v[2] += pw[2]; v[3] += pw[3];
        }
        epilogue_apply<EPI>(a, eml, en, v[0], v[1], v[2], v[3], eo);
    }
}

// --------------------------------------------------------------------------------------------
// weight streaming for large layers (M <= 16 rows, tens of MB to GBs of weights per projection)
// --------------------------------------------------------------------------------------------
// Same data path as gemm_flat (whole-line loads, MFMA layout made in wave-private LDS staging
// areas, no barrier inside the K loop), but K is a loop and the activations do not fit in LDS:
//   * a workgroup of 4 waves owns 16*NF output columns; groups of UQ = 4 units (256 K values,
//     512 contiguous bytes of every weight row; 2 units with NF = 3, for the registers) are dealt
//     round-robin to the waves;
//   * a wave loads, per group, NF*UQ*2 instructions of weights and UQ*XH of activations (the
//     16 x 64 activation unit has the shape of a weight unit and takes the same road through the
//     staging areas; XH = 1 when M <= 8), for group i+1 before group i is consumed (two register
//     buffers); the scalar base pointers advance by one stride per group, so a load costs no
//     vector arithmetic at all; a group is staged two units at a time, which keeps the staging
//     space small enough for two workgroups per CU;
//   * the four partial tiles are summed through LDS once, at the end.
//
// LNS hands the statistics of the LayerNorm between two such projections from one launch to the next (GemmArgs::
// row_stats_*), so that a decode step of a large layer has no LayerNorm launch between its output projection and its first
// feed-forward projection:
//   LNS = 1 (bias + residual): the threads that write the 16 x 16*NF outputs also leave, per row, the mean and the sum of
//           squared deviations of the workgroup's columns of the rounded output;
//   LNS = 2: the workgroup first merges the producer's groups (equal sizes, so group means average; squared deviations add
//           up with the spread of the group means, taken relative to the first group's mean) into mean and 1/std per row,
//           while its first weights are in flight, and normalises every activation vector (three fused multiply-adds per
//           element) before it is staged for the matrix instructions.
// NT: the weights are loaded with the non-temporal hint (GemmArgs::read_once).  A template parameter, not a branch: the compiler
// merges the two arms of a branch whose loads differ in nothing but the hint, and drops it.
constexpr int kStreamStagedUnits = 2;
constexpr int kStreamStatsLds = 1024;                       // bytes behind the staging areas: the merged row statistics (LNS = 2)

template <int NF, int EPI, int XH, bool SL, int LNS = 0, bool NT = false>
__global__ __launch_bounds__(256) void gemm_stream(GemmArgs a) {
    static_assert(!NT || !SL, "row slices read the weights once from memory and then from the caches: plain loads");
    static_assert(LNS == 0 || !SL, "row statistics: at most 16 rows, one slice");
    static_assert(LNS != 1 || EPI == EPI_BIAS_RES, "the producer of row statistics is a bias + residual projection");
    if (SL) take_row_slice<EPI>(a);
    constexpr int UQ = NF >= 3 ? 2 : 4;                     // units per group (three or four column blocks: half as many, for the registers)
    constexpr int SU = kStreamStagedUnits;                  // units staged at a time
    constexpr int AREAS = SU * (NF + 1);                    // staging areas per wave (16 x 144 bytes each)
    extern __shared__ __attribute__((aligned(16))) unsigned char stream_smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fr = lane & 15, G = lane >> 4;
    const int wrow = lane >> 3, wchunk = lane & 7;
    const int n0 = blockIdx.x * (16 * NF);
    const int M = a.M, N = a.N, K = a.K;
    const int ngroups = K / (64 * UQ);
    half_t* wst = reinterpret_cast<half_t*>(stream_smem) + wave * (AREAS * 16 * kFlatStageRow);
    float* red = reinterpret_cast<float*>(stream_smem);

    if (a.bump_lens != nullptr && blockIdx.x == 0 && tid < a.bump_count) a.bump_lens[tid] += 1;

    // epilogue operands of the 64*NF threads that write the 16 x 16*NF outputs
    const int eml = tid / (4 * NF), enl = (tid % (4 * NF)) * 4, en = n0 + enl;
    const bool writer = tid < 64 * NF && eml < M && en < N;
    EpiOperands eo;
    if (writer) epilogue_fetch<EPI>(a, eml, en, eo);

    // per-lane byte offsets inside a group (loop invariant); the group itself moves the scalar base
    uint32_t woff[NF][2], xoff[XH];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            int wr = n0 + 16 * f + 8 * h + wrow;
            wr = wr < N ? wr : N - 1;
            woff[f][h] = ((uint32_t)(wr - n0) * (uint32_t)K + wchunk * 8) * 2u;
        }
#pragma unroll
    for (int h = 0; h < XH; ++h) {
        int xr = 8 * h + wrow;
        xr = xr < M ? xr : M - 1;
        xoff[h] = ((uint32_t)xr * (uint32_t)K + wchunk * 8) * 2u;
    }
    const char* wbase = reinterpret_cast<const char*>(a.w) + (size_t)n0 * K * 2;
    const char* xbase = reinterpret_cast<const char*>(a.x);

    // Workgroups start their walk over K in eight different places (workgroups are dealt round-robin to the eight XCDs, so
    // blockIdx.x / 8 counts inside an XCD) instead of all reading the same K offset of their rows, and of the shared
    // activation rows, at the same time (rows x N x K: 16 x 36864 x 12288 166 -> 157 us, 16 x 49152 x 12288 218 -> 208,
    // 16 x 12288 x 12288 50.4 -> 47.6, 4 x 4096 x 16384 28.0 -> 21.9, 4 x 16384 x 4096 22.6 -> 21.0; K = 49152 unchanged;
    // two phases were slower than one, thirty-two slower at K = 49152).  Only the order of a column's sum depends on it.
    const int phase = (int)((((unsigned)blockIdx.x >> 3) & 7u) * (unsigned)ngroups) >> 3;
    // LNS = 2: the producer's row statistics; thread t takes row t%16 and every 16th group from t/16 on, 16 groups at a time.
    // The first 16 (all of them up to 256 groups) are requested before anything else: loads return in issue order.
    constexpr int kStatBatch = 16;
    float2v stat[LNS == 2 ? kStatBatch : 1];
    float stat0 = 0.f;                                       // the first group's mean of this thread's row
    const float2v* stat_src = reinterpret_cast<const float2v*>(a.row_stats_in) + (tid & 15);
    auto request_stats = [&](int u0) {
#pragma unroll
        for (int u = 0; u < kStatBatch; ++u) {
            const int grp = (tid >> 4) + 16 * (u0 + u);
            if (grp < a.row_stats_groups) stat[u] = stat_src[grp * 16];
        }
    };
    if constexpr (LNS == 2) {
        stat0 = stat_src[0][0];
        request_stats(0);
    }
    constexpr int GB = LNS == 2 ? UQ : 1;
    half8v wA[UQ][NF][2], xA[UQ][XH], wB[UQ][NF][2], xB[UQ][XH], gA[GB], bA[GB], gB[GB], bB[GB];
    auto request = [&](half8v (&wr)[UQ][NF][2], half8v (&xr)[UQ][XH], half8v (&gr)[GB], half8v (&br)[GB], int g) {
        g = g < ngroups ? g : ngroups - 1;                    // look-ahead past the end: a valid group, never consumed
        g += phase;                                           // this workgroup's walk starts `phase` groups into K and wraps
        g = g >= ngroups ? g - ngroups : g;
        const char* wg = wbase + (size_t)g * (UQ * 128);
        const char* xg = xbase + (size_t)g * (UQ * 128);
#pragma unroll
        for (int q = 0; q < UQ; ++q) {
            if constexpr (LNS == 2) {                         // gamma and beta of the 8 columns this lane holds of unit q
                gr[q] = *reinterpret_cast<const half8v*>(reinterpret_cast<const char*>(a.ln_gamma) + (size_t)g * (UQ * 128) + q * 128 + wchunk * 16);
                br[q] = *reinterpret_cast<const half8v*>(reinterpret_cast<const char*>(a.ln_beta) + (size_t)g * (UQ * 128) + q * 128 + wchunk * 16);
            }
#pragma unroll
            for (int h = 0; h < XH; ++h) xr[q][h] = *reinterpret_cast<const half8v*>(xg + xoff[h] + q * 128);
        }
#pragma unroll
        for (int q = 0; q < UQ; ++q)
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const half8v* src = reinterpret_cast<const half8v*>(wg + woff[f][h] + q * 128);
                    if constexpr (NT) wr[q][f][h] = load_once(src); else wr[q][f][h] = *src;
                }
    };
    float4v acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = float4v{0.f, 0.f, 0.f, 0.f};
    const uint32_t st_w = (uint32_t)(wrow * kFlatStageRow + wchunk * 8);     // staging write (halves)
    const uint32_t st_r = (uint32_t)(fr * kFlatStageRow + G * 8);            // staging read
    float ln_mu[XH], ln_rs[XH];                               // LNS = 2: mean and 1/std of this lane's activation rows
    auto consume = [&](const half8v (&wr)[UQ][NF][2], const half8v (&xr)[UQ][XH], const half8v (&gr)[GB], const half8v (&br)[GB]) {
        // area (j*(NF+1) + 0) holds the activation unit j of the round, areas +1.. its weight units
#pragma unroll
        for (int q0 = 0; q0 < UQ; q0 += SU) {
#pragma unroll
            for (int j = 0; j < SU; ++j) {
#pragma unroll
                for (int h = 0; h < XH; ++h) {
                    half8v xv = xr[q0 + j][h];
                    if constexpr (LNS == 2) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const float sc = __builtin_fmaf((float)gr[q0 + j][e], ln_rs[h], 0.f);
                            const float sh = __builtin_fmaf(-ln_mu[h], sc, (float)br[q0 + j][e]);
                            xv[e] = (half_t)__builtin_fmaf((float)xv[e], sc, sh);
                        }
                    }
                    *reinterpret_cast<half8v*>(&wst[st_w + ((j * (NF + 1)) * 16 + 8 * h) * kFlatStageRow]) = xv;
                }
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        *reinterpret_cast<half8v*>(&wst[st_w + ((j * (NF + 1) + 1 + f) * 16 + 8 * h) * kFlatStageRow]) = wr[q0 + j][f][h];
            }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int j = 0; j < SU; ++j)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    // rows 8..15 of the activation area are stale when XH = 1: those outputs are never written
                    const half8v xf = *reinterpret_cast<const half8v*>(&wst[st_r + (j * (NF + 1)) * 16 * kFlatStageRow + 32 * u]);
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const half8v wf = *reinterpret_cast<const half8v*>(&wst[st_r + (j * (NF + 1) + 1 + f) * 16 * kFlatStageRow + 32 * u]);
                        acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_f16(wf, xf, acc[f], 0, 0, 0);
                    }
                }
            __builtin_amdgcn_wave_barrier();
        }
    };
    int g = wave;
    if (g < ngroups) request(wA, xA, gA, bA, g);
    if constexpr (LNS == 2) {
        // merge the groups: with q the first group's mean, A = sum(mean_g - q), B = sum((mean_g - q)^2), C = sum(M2_g);
        // mean = q + A/G, sum of squared deviations = C + cols * (B - A^2/G)
        float* sm = reinterpret_cast<float*>(stream_smem + 4 * AREAS * 16 * kFlatStageRow * 2);   // [4 waves][16 rows][3], then mean[16], 1/std[16]
        float A = 0.f, B = 0.f, C = 0.f;
        for (int u0 = 0; 16 * u0 < a.row_stats_groups; u0 += kStatBatch) {
            if (u0 > 0) request_stats(u0);                    // more than 256 groups: further trips, behind the first weights
#pragma unroll
            for (int u = 0; u < kStatBatch; ++u) {
                if ((tid >> 4) + 16 * (u0 + u) < a.row_stats_groups) {
                    const float dm = stat[u][0] - stat0;
                    A += dm;
                    B = __builtin_fmaf(dm, dm, B);
                    C += stat[u][1];
                }
            }
        }
        A = sum_xor32(sum_xor16(A)); B = sum_xor32(sum_xor16(B)); C = sum_xor32(sum_xor16(C));
        if (lane < 16) {
            sm[(wave * 16 + lane) * 3 + 0] = A;
            sm[(wave * 16 + lane) * 3 + 1] = B;
            sm[(wave * 16 + lane) * 3 + 2] = C;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");    // LDS only: the weight loads stay in flight across the barrier
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (tid < 16) {
            float At = 0.f, Bt = 0.f, Ct = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                At += sm[(w * 16 + tid) * 3 + 0];
                Bt += sm[(w * 16 + tid) * 3 + 1];
                Ct += sm[(w * 16 + tid) * 3 + 2];
            }
            const float G = (float)a.row_stats_groups, cols = (float)a.row_stats_cols;
            const float m2 = Ct + cols * fmaxf(Bt - At * At / G, 0.f);
            sm[192 + tid] = stat0 + At / G;
            sm[208 + tid] = rsqrtf(m2 / (G * cols) + a.ln_eps);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int h = 0; h < XH; ++h) {
            ln_mu[h] = sm[192 + 8 * h + wrow];
            ln_rs[h] = sm[208 + 8 * h + wrow];
        }
    }
    if (g < ngroups) {
        while (true) {
            request(wB, xB, gB, bB, g + 4);
            __builtin_amdgcn_sched_barrier(0);                // keep the look-ahead loads ahead of the arithmetic
            consume(wA, xA, gA, bA);
            g += 4;
            if (g >= ngroups) break;
            request(wA, xA, gA, bA, g + 4);
            __builtin_amdgcn_sched_barrier(0);
            consume(wB, xB, gB, bB);
            g += 4;
            if (g >= ngroups) break;
        }
    }
    // acc[f][r]: output column n0 + 16f + 4G + r, row fr.  The partial tiles go over the staging
    // space, which other waves may still be reading as theirs: barrier first.
    __syncthreads();
    constexpr int RT = 16 * (16 * NF + 4);                    // floats per wave tile: [16 rows][16*NF + 4]
#pragma unroll
    for (int f = 0; f < NF; ++f) *reinterpret_cast<float4v*>(&red[wave * RT + fr * (16 * NF + 4) + 16 * f + 4 * G]) = acc[f];
    __syncthreads();
    if (writer) {
        const float* rp = &red[eml * (16 * NF + 4) + enl];
        float4v v = *reinterpret_cast<const float4v*>(rp);
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const float4v pw = *reinterpret_cast<const float4v*>(rp + w * RT);
            v[0] += pw[0]; v[1] += pw[1]; v[2] += pw[2]; v[3] += pw[3];
        }
        const half4v o = epilogue_apply<EPI>(a, eml, en, v[0], v[1], v[2], v[3], eo);
        if constexpr (LNS == 1) {                             // this thread's four rounded outputs: mean and squared deviations
            const float o0 = (float)o[0], o1 = (float)o[1], o2 = (float)o[2], o3 = (float)o[3];
            const float mt = 0.25f * ((o0 + o1) + (o2 + o3));
            const float d0 = o0 - mt, d1 = o1 - mt, d2 = o2 - mt, d3 = o3 - mt;
            float* sp = red + 4 * RT + tid * 2;               // behind the four waves' partial tiles
            sp[0] = mt;
            sp[1] = (d0 * d0 + d1 * d1) + (d2 * d2 + d3 * d3);
        }
    }
    if constexpr (LNS == 1) {
        static_assert((4 * RT + 256 * 2) * 4 <= 4 * AREAS * 16 * kFlatStageRow * 2, "statistics behind the partial tiles, inside the staging space");
        __syncthreads();
        // the first of a row's 4*NF threads merges them (equal sizes: means average, squared deviations add up with the
        // spread of the means) and writes the row's pair for this workgroup
        if (writer && tid % (4 * NF) == 0) {
            const float* sp = red + 4 * RT + tid * 2;
            float ms = 0.f;
#pragma unroll
            for (int t = 0; t < 4 * NF; ++t) ms += sp[2 * t];
            const float mg = ms * (1.0f / (4 * NF));
            float m2 = 0.f;
#pragma unroll
            for (int t = 0; t < 4 * NF; ++t) {
                const float dm = sp[2 * t] - mg;
                m2 += sp[2 * t + 1] + 4.0f * dm * dm;
            }
            float* dst = a.row_stats_out + ((size_t)blockIdx.x * 16 + eml) * 2;
            dst[0] = mg;
            dst[1] = m2;
        }
    }
}

// --------------------------------------------------------------------------------------------
// dispatch
// --------------------------------------------------------------------------------------------
template <int WGM, int WGN, int BM = 256, int BN = 256, int NS = 2, int KS = 1, int SCHED = 0, bool NTS = false>
static void launch_dma64_cfg(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    const int tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
    const dim3 grid(tm * tn), block(WGM * WGN * KS * 64);
    switch (epi) {
        case EPI_BIAS: hipLaunchKernelGGL((gemm_mfma_dma64<BM, BN, WGM, WGN, EPI_BIAS, NS, KS, SCHED, NTS>), grid, block, 0, s, a, tm, tn); break;
        case EPI_BIAS_GELU: hipLaunchKernelGGL((gemm_mfma_dma64<BM, BN, WGM, WGN, EPI_BIAS_GELU, NS, KS, SCHED, NTS>), grid, block, 0, s, a, tm, tn); break;
        case EPI_BIAS_RES: hipLaunchKernelGGL((gemm_mfma_dma64<BM, BN, WGM, WGN, EPI_BIAS_RES, NS, KS, SCHED, NTS>), grid, block, 0, s, a, tm, tn); break;
        case EPI_QKV: hipLaunchKernelGGL((gemm_mfma_dma64<BM, BN, WGM, WGN, EPI_QKV, NS, KS, SCHED, NTS>), grid, block, 0, s, a, tm, tn); break;
    }
}

template <int NF, bool LN, int NW>
static void launch_skinny_nw(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    const dim3 grid((a.N + NF * 16 - 1) / (NF * 16), (a.M + 15) / 16), block(NW * 64);
    switch (epi) {
        case EPI_BIAS: hipLaunchKernelGGL((gemm_skinny<NF, EPI_BIAS, LN, NW>), grid, block, 0, s, a); break;
        case EPI_BIAS_GELU: hipLaunchKernelGGL((gemm_skinny<NF, EPI_BIAS_GELU, LN, NW>), grid, block, 0, s, a); break;
        case EPI_BIAS_RES: hipLaunchKernelGGL((gemm_skinny<NF, EPI_BIAS_RES, LN, NW>), grid, block, 0, s, a); break;
        case EPI_QKV: hipLaunchKernelGGL((gemm_skinny<NF, EPI_QKV, LN, NW>), grid, block, 0, s, a); break;
    }
}
template <int NF>
static void launch_skinny_cfg(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    if (a.ln_gamma != nullptr) launch_skinny_nw<NF, true, 4>(a, epi, s);
    else launch_skinny_nw<NF, false, 4>(a, epi, s);
}
constexpr int kFlatLdsLimit = 160 * 1024;                  // LDS of one CU

static void launch_flat_kernel(void (*kernel)(GemmArgs), const GemmArgs& a, dim3 grid, dim3 block, int lds, hipStream_t s) {
    // more than 64 KB of dynamic LDS has to be allowed once per kernel and device
    if (lds > 64 * 1024) {
        static std::mutex mu;
        static std::set<std::pair<const void*, int>> allowed;
        int dev = 0;
        (void)hipGetDevice(&dev);
        std::lock_guard<std::mutex> lock(mu);
        if (allowed.insert({reinterpret_cast<const void*>(kernel), dev}).second)
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kFlatLdsLimit);
    }
    hipLaunchKernelGGL(kernel, grid, block, lds, s, a);
}

template <int NW, int UPW, int TN, bool LN, bool SL>
static void launch_flat_sl(const GemmArgs& a, Epilogue epi, int lds, hipStream_t s) {
    const dim3 grid(a.N / TN + (a.pf.blocks > 0 ? a.pf.blocks : 0), SL ? (a.M + 15) / 16 : 1), block(NW * 64);
    switch (epi) {
        case EPI_BIAS: launch_flat_kernel(gemm_flat<NW, UPW, TN, EPI_BIAS, LN, SL>, a, grid, block, lds, s); break;
        case EPI_BIAS_GELU: launch_flat_kernel(gemm_flat<NW, UPW, TN, EPI_BIAS_GELU, LN, SL>, a, grid, block, lds, s); break;
        case EPI_BIAS_RES:
            if constexpr (!LN && !SL) {
                if (a.x_splits > 1) {
                    launch_flat_kernel(gemm_flat<NW, UPW, TN, EPI_BIAS_RES, false, false, true>, a, grid, block, lds, s);
                    break;
                }
            }
            launch_flat_kernel(gemm_flat<NW, UPW, TN, EPI_BIAS_RES, LN, SL>, a, grid, block, lds, s);
            break;
        case EPI_QKV: launch_flat_kernel(gemm_flat<NW, UPW, TN, EPI_QKV, LN, SL>, a, grid, block, lds, s); break;
    }
}
template <int NW, int UPW, int TN, bool LN>
static void launch_flat_epi(const GemmArgs& a, Epilogue epi, int lds, hipStream_t s) {
    if (!LN && a.M > 16) launch_flat_sl<NW, UPW, TN, false, true>(a, epi, lds, s);     // never with the fused LayerNorm
    else launch_flat_sl<NW, UPW, TN, LN, false>(a, epi, lds, s);
}
template <int NW, int TN, bool LN>
static void launch_flat(const GemmArgs& a, int upw, Epilogue epi, int lds, hipStream_t s) {
    switch (upw) {
        case 1: launch_flat_epi<NW, 1, TN, LN>(a, epi, lds, s); break;
        case 2: launch_flat_epi<NW, 2, TN, LN>(a, epi, lds, s); break;
        case 3: launch_flat_epi<NW, 3, TN, LN>(a, epi, lds, s); break;
        default: launch_flat_epi<NW, 4, TN, LN>(a, epi, lds, s); break;
    }
}
// true when the flat kernel took the problem: a few MB of weights, K = 64 * NW * UPW with
// NW in {4, 8, 16} and UPW in 1..4, N a multiple of 16, no row maps
static bool try_flat(const GemmArgs& a, Epilogue epi, hipStream_t s, bool ask_only = false) {
    constexpr int tn8_wgs = 128;                              // fewer 16-column workgroups than this: 8-column ones
    // (with the LayerNorm fused in front up to 20 MB: it replaces a launch)
    if ((int64_t)a.N * a.K * 2 > ((a.ln_gamma != nullptr ? 20 : 16) << 20) || a.N % 16 != 0 || a.K % 64 != 0) return false;
    if (a.res_row_map != nullptr || a.out_row_map != nullptr || a.tok_row_map != nullptr) return false;
    const bool ln = a.ln_gamma != nullptr;
    const int units = a.K / 64;
    auto fits = [&](int cand) { return units % cand == 0 && units / cand <= 4; };
    // fewest waves that hold K; with LN 8 waves when possible: the normalisation is vector
    // arithmetic spread over the threads
    int nw = 0;
    if (ln && fits(8)) nw = 8;
    for (int cand : {4, 8, 16})
        if (nw == 0 && fits(cand)) nw = cand;
    if (nw == 0 || (ln && nw == 16)) return false;
    const int upw = units / nw;
    const int lds = flat_lds_bytes(nw, upw, a.M <= 8 ? 8 : 16);
    if (lds > kFlatLdsLimit) return false;
    if (ask_only) return true;
    if (nw == 4) {
        // few columns: 8 per workgroup put twice the workgroups on the chip (output projection of hidden 1024: 64 -> 128 beside
        // its 128 prefetch workgroups, 324.9 -> 322.6 ms for 512 steps of 24 layers while such steps went launch by launch; wide
        // feed-forward parts and more than 16 rows still come here)
        if (ln) launch_flat<4, 16, true>(a, upw, epi, lds, s);
        else if (a.N / 16 < tn8_wgs) launch_flat<4, 8, false>(a, upw, epi, lds, s);
        else launch_flat<4, 16, false>(a, upw, epi, lds, s);
    } else if (nw == 8) {
        if (ln) launch_flat<8, 16, true>(a, upw, epi, lds, s); else launch_flat<8, 16, false>(a, upw, epi, lds, s);
    } else if (a.N / 16 < tn8_wgs) {
        launch_flat<16, 8, false>(a, upw, epi, lds, s);       // long rows, few columns: one CU cannot pull 16 rows fast enough
    } else {
        launch_flat<16, 16, false>(a, upw, epi, lds, s);
    }
    return true;
}

// LNS (see gemm_stream): 1 = leave row statistics (bias + residual), 2 = normalise the activations from them
static bool leaves_row_stats(const GemmArgs& a, Epilogue epi) { return a.row_stats_out != nullptr && epi == EPI_BIAS_RES && a.M <= 16; }
static bool takes_row_stats(const GemmArgs& a, Epilogue epi) {
    return a.row_stats_in != nullptr && a.ln_gamma != nullptr && epi == EPI_BIAS_GELU && a.M <= 16 && a.row_stats_groups >= 1 && a.row_stats_cols >= 1;
}

// at most 16 rows: one slice, with or without the non-temporal hint on the weights
template <int NF, int XH, bool NT>
static void launch_stream_rows(const GemmArgs& a, Epilogue epi, dim3 grid, dim3 block, int lds, hipStream_t s) {
    if (leaves_row_stats(a, epi)) {
        launch_flat_kernel(gemm_stream<NF, EPI_BIAS_RES, XH, false, 1, NT>, a, grid, block, lds, s);
        return;
    }
    if (takes_row_stats(a, epi)) {
        launch_flat_kernel(gemm_stream<NF, EPI_BIAS_GELU, XH, false, 2, NT>, a, grid, block, lds + kStreamStatsLds, s);
        return;
    }
    switch (epi) {
        case EPI_BIAS: launch_flat_kernel(gemm_stream<NF, EPI_BIAS, XH, false, 0, NT>, a, grid, block, lds, s); break;
        case EPI_BIAS_GELU: launch_flat_kernel(gemm_stream<NF, EPI_BIAS_GELU, XH, false, 0, NT>, a, grid, block, lds, s); break;
        case EPI_BIAS_RES: launch_flat_kernel(gemm_stream<NF, EPI_BIAS_RES, XH, false, 0, NT>, a, grid, block, lds, s); break;
        case EPI_QKV: launch_flat_kernel(gemm_stream<NF, EPI_QKV, XH, false, 0, NT>, a, grid, block, lds, s); break;
    }
}

template <int NF, int XH>
static void launch_stream(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    const int lds = 4 * kStreamStagedUnits * (NF + 1) * 16 * kFlatStageRow * 2;
    const dim3 block(256);
    if (a.M > 16) {                                           // rows in slices of 16 along gridDim.y
        const dim3 grid(a.N / (16 * NF), (a.M + 15) / 16);
        switch (epi) {
            case EPI_BIAS: launch_flat_kernel(gemm_stream<NF, EPI_BIAS, XH, true>, a, grid, block, lds, s); break;
            case EPI_BIAS_GELU: launch_flat_kernel(gemm_stream<NF, EPI_BIAS_GELU, XH, true>, a, grid, block, lds, s); break;
            case EPI_BIAS_RES: launch_flat_kernel(gemm_stream<NF, EPI_BIAS_RES, XH, true>, a, grid, block, lds, s); break;
            case EPI_QKV: launch_flat_kernel(gemm_stream<NF, EPI_QKV, XH, true>, a, grid, block, lds, s); break;
        }
        return;
    }
    const dim3 grid(a.N / (16 * NF));
    if (a.read_once) launch_stream_rows<NF, XH, true>(a, epi, grid, block, lds, s);
    else launch_stream_rows<NF, XH, false>(a, epi, grid, block, lds, s);
}

// Blocks of 16 columns the streaming kernel gives a workgroup for this problem; 0: not its problem (K a multiple of 256,
// whole column tiles, and no LayerNorm unless its statistics come with the call).
static int stream_column_blocks(const GemmArgs& a, Epilogue epi) {
    if ((a.ln_gamma != nullptr && !takes_row_stats(a, epi)) || a.K % 256 != 0 || a.N % 32 != 0) return 0;
    if ((int64_t)a.M * a.K * 2 >= ((int64_t)1 << 31) || (int64_t)32 * a.K * 2 >= ((int64_t)1 << 31)) return 0;   // 32-bit lane offsets
    // With 16 rows a workgroup pulls as many activation lines out of L2 as weight lines when it owns 16
    // columns, and the stream slows down with every distinct activation line (12288 x 49152: 208 us at 1 row, 211 at
    // 8, 222 at 9, 246 at 16).  48 columns per workgroup cut that to a third: 246 -> 209 us, 12288 x 12288 60 -> 50 us,
    // 36864 x 12288 179 -> 166 us, 49152 x 12288 226 -> 219 us (16 rows each).  Taken where 48 divides N and the
    // workgroups fill the CUs evenly (N = 12288: exactly one per CU).  Sharing the activation lines between the waves of
    // a workgroup through the CU's vector cache instead (waves side by side in N, all walking the same K) changed nothing.
    const int wg48 = a.N % 48 == 0 ? a.N / 48 : 0;
    if (a.M > 4 && wg48 >= 256 && (wg48 % 256 == 0 || wg48 >= 1024)) return 3;   // (8 rows: 49152 x 12288 209 -> 205 us; 4 rows: 12288 x 4096 16.7 -> 17.8 the other way, 2 rows: no difference)
    const int wg64 = a.N % 64 == 0 ? a.N / 64 : 0;             // N without a factor of 3: 64 columns (16 rows: 16384 x 4096 25.1 -> 23.0 us,
    if (a.M > 8 && wg64 >= 256 && (wg64 % 256 == 0 || wg64 >= 1024)) return 4;   // 32768 x 8192 129 -> 114 us; nothing to gain at 4 rows)
    // Up to 8 rows otherwise 16 columns per workgroup whatever N is (32 columns, once the rule for wide outputs, lost since the
    // workgroups walk K in phases: 1 row, 36864 x 12288 168 -> 153 us, 49152 x 12288 214 -> 201, 65536 x 4096 99 -> 88;
    // 4 and 8 rows, 32768 x 8192 101 -> 93); more rows and a wide output that takes neither 48 nor 64: 32 columns.
    if (a.M <= 8) return 1;
    return a.N / 32 >= 1024 ? 2 : 1;
}

// true when the streaming kernel took the problem
static bool try_stream(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    const int nf = stream_column_blocks(a, epi);
    if (nf == 0) return false;
    const bool few = a.M <= 8;                                // at most 8 rows: one half of the activation unit
    switch (nf) {
        case 1: if (few) launch_stream<1, 1>(a, epi, s); else launch_stream<1, 2>(a, epi, s); break;
        case 2: launch_stream<2, 2>(a, epi, s); break;
        case 3: if (few) launch_stream<3, 1>(a, epi, s); else launch_stream<3, 2>(a, epi, s); break;
        default: launch_stream<4, 2>(a, epi, s); break;
    }
    return true;
}

// --------------------------------------------------------------------------------------------
// 17 to 1024 rows: a weight stream through the tile kernel (which calls: tile_rules.hpp)
// --------------------------------------------------------------------------------------------
// no LayerNorm, prefetch or length update rides on the call (the weight-streaming kernels' business)
static bool is_plain(const GemmArgs& a) { return a.ln_gamma == nullptr && a.pf.blocks == 0 && a.bump_lens == nullptr; }
static bool rows_stream(const GemmArgs& a, Epilogue epi) {
    if (a.k_ranges > 1 && epi == EPI_BIAS_RES) return true;          // the caller asked gemm_cut_ranges
    return is_plain(a) && rows_stream_uncut(a.M, a.N, a.K, a.read_once != 0);
}

template <int BM, int WGM, int KS, bool NTW, bool ROT, int EPI>
static void launch_rows_epi(const GemmArgs& a, hipStream_t s) {
    const int tm = (a.M + BM - 1) / BM, tn = (a.N + 63) / 64;
    const dim3 grid(tm * tn * (EPI == EPI_PARTIAL ? a.k_ranges : 1)), block(WGM * KS * 64);
    hipLaunchKernelGGL((gemm_mfma_dma64<BM, 64, WGM, 1, EPI, 3, KS, 0, false, NTW, ROT>), grid, block, 0, s, a, tm, tn);
}
template <int BM, int WGM, int KS, bool NTW>
static void launch_rows_tile(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    if (a.k_ranges > 1) { launch_rows_epi<BM, WGM, KS, NTW, true, EPI_PARTIAL>(a, s); return; }
    switch (epi) {
        case EPI_BIAS: launch_rows_epi<BM, WGM, KS, NTW, true, EPI_BIAS>(a, s); break;
        case EPI_BIAS_GELU: launch_rows_epi<BM, WGM, KS, NTW, true, EPI_BIAS_GELU>(a, s); break;
        case EPI_BIAS_RES: launch_rows_epi<BM, WGM, KS, NTW, true, EPI_BIAS_RES>(a, s); break;
        case EPI_QKV: launch_rows_epi<BM, WGM, KS, NTW, true, EPI_QKV>(a, s); break;
    }
}
template <bool NTW>
static void launch_rows_nt(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    if (a.M <= 32 && a.K % 256 == 0) launch_rows_tile<32, 1, 4, NTW>(a, epi, s);
    else if (a.M <= 64) launch_rows_tile<64, 2, 2, NTW>(a, epi, s);
    else launch_rows_tile<128, 2, 2, NTW>(a, epi, s);
}
static hipError_t launch_rows(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    if (a.M > kRowsStreamMaxM) launch_rows_epi<128, 4, 2, false, false, EPI_PARTIAL>(a, s);
    else if (a.read_once) launch_rows_nt<true>(a, epi, s);
    else launch_rows_nt<false>(a, epi, s);
    const hipError_t e = hipGetLastError();
    return a.k_ranges > 1 && e == hipSuccess ? launch_finish_rows(a, s) : e;
}

bool gemm_hands_row_stats(const GemmArgs& producer, const GemmArgs& consumer, Epilogue consumer_epi, int& groups, int& cols) {
    GemmArgs p = producer, c = consumer;
    p.row_stats_out = reinterpret_cast<float*>(16);              // any non-null value: only asked, never launched
    c.row_stats_in = reinterpret_cast<const float*>(16);
    c.row_stats_groups = c.row_stats_cols = 1;
    if (p.M < 1 || p.M > 16 || c.M != p.M || c.K != p.N || c.ln_gamma == nullptr || p.ln_gamma != nullptr || p.x_splits > 1) return false;
    if (try_flat(p, EPI_BIAS_RES, nullptr, true) || try_flat(c, consumer_epi, nullptr, true)) return false;
    const int nf = stream_column_blocks(p, EPI_BIAS_RES), nfc = takes_row_stats(c, consumer_epi) ? stream_column_blocks(c, consumer_epi) : 0;
    if (nf == 0 || p.N % (16 * nf) != 0 || nfc == 0) return false;
    // Every workgroup of the consumer merges the producer's groups before its first multiply: that pays where a workgroup
    // then streams a megabyte of weights or more and one trip brings all groups (hidden 12288 at 16 rows: 48 columns x 24 KB
    // each, 256 groups: 826 -> 818 us per step); with short-lived workgroups the launch it saves is cheaper (hidden 4096
    // at 4 rows, 16 columns x 8 KB each: 106.7 -> 108.7 us per step; hidden 12288 at 1 row, 768 groups: 638 -> 652 us).
    if ((int64_t)16 * nfc * c.K * 2 < (1 << 20) || p.N / (16 * nf) > 256) return false;
    groups = p.N / (16 * nf);
    cols = 16 * nf;
    return true;
}

bool gemm_takes_layernorm(const GemmArgs& a) { return a.M >= 1 && a.M <= 16 && a.ln_gamma != nullptr && try_flat(a, EPI_BIAS, nullptr, true); }
bool gemm_takes_prefetch(const GemmArgs& a) { return a.M >= 1 && a.M <= 16 && try_flat(a, EPI_BIAS_RES, nullptr, true); }

bool gemm_merges_attention_ranges(const GemmArgs& a) {
    return a.M >= 1 && a.M <= 16 && a.ln_gamma == nullptr && a.d >= 8 && a.d % 8 == 0 && a.heads * a.d == a.K &&
           try_flat(a, EPI_BIAS_RES, nullptr, true);
}

// true when launch_gemm gives this problem to an MFMA tile kernel.  Only those take row strides (lda, ldy), and a
// problem that comes with strides never goes to the row slices.
static bool is_strided(const GemmArgs& a) { return (a.lda != 0 && a.lda != a.K) || (a.ldy != 0 && a.ldy != a.N); }
static bool goes_to_tile_kernel(const GemmArgs& a) {
    const bool sliced = a.M > 16 && !is_strided(a) && a.res_row_map == nullptr && a.out_row_map == nullptr && a.tok_row_map == nullptr &&
                        is_plain(a) && slices_beat_tiles(a.M, a.N, a.K);
    return a.M > 16 && !sliced;
}
bool gemm_takes_row_strides(const GemmArgs& a) { return a.M > 16 && a.x_splits <= 1; }
int gemm_cut_ranges(const GemmArgs& a) {
    return a.res_row_map != nullptr || a.out_row_map != nullptr ? prompt_k_ranges(a.M, a.N, a.K) : gemm_k_ranges(a.M, a.N, a.K);
}

// The same problem without its first m0 rows (EPI_QKV: the prefill form, whose rows carry their sequence and position in
// tok_row_map; the decode form takes the sequence from the row number and is never cut).
static GemmArgs rows_from(const GemmArgs& a, Epilogue epi, int m0) {
    GemmArgs r = a;
    r.M = a.M - m0;
    r.x = a.x + (size_t)m0 * (a.lda ? a.lda : a.K);
    if (epi == EPI_QKV) {
        r.y = a.y + (size_t)m0 * a.hidden;
        r.tok_row_map = a.tok_row_map + m0;
        return r;
    }
    if (a.out_row_map) r.out_row_map = a.out_row_map + m0;
    else r.y = a.y + (size_t)m0 * (a.ldy ? a.ldy : a.N);
    if (a.res) {
        if (a.res_row_map) r.res_row_map = a.res_row_map + m0;
        else r.res = a.res + (size_t)m0 * a.N;
    }
    return r;
}

hipError_t launch_gemm(const GemmArgs& a, Epilogue epi, hipStream_t s) {
    if (a.M <= 0) return hipSuccess;
    const bool bad_stride = (a.lda != 0 && (a.lda < a.K || a.lda % 8 != 0)) || (a.ldy != 0 && (a.ldy < a.N || a.ldy % 8 != 0));
    if (bad_stride || (is_strided(a) && (!gemm_takes_row_strides(a) || epi == EPI_QKV))) return hipErrorInvalidValue;
    if (a.x_splits > 1 && (epi != EPI_BIAS_RES || !gemm_merges_attention_ranges(a))) return hipErrorInvalidValue;
    // row statistics are between two launches of the weight-streaming kernel: asked for anywhere else, refuse
    if (a.row_stats_out != nullptr && !(leaves_row_stats(a, epi) && !try_flat(a, epi, nullptr, true) && stream_column_blocks(a, epi) != 0 &&
                                        a.N % (16 * stream_column_blocks(a, epi)) == 0)) return hipErrorInvalidValue;
    if (a.row_stats_in != nullptr && !(takes_row_stats(a, epi) && !try_flat(a, epi, nullptr, true) && stream_column_blocks(a, epi) != 0)) return hipErrorInvalidValue;
    // the cut along K is the caller's choice, and its operands are its own
    if (a.k_ranges > 1 && (epi != EPI_BIAS_RES || a.part == nullptr || a.k_ranges != gemm_cut_ranges(a) || (a.ldy != 0 && a.ldy != a.N) || a.ln_gamma != nullptr || a.pf.blocks != 0)) return hipErrorInvalidValue;
    if (a.fin_gamma != nullptr && a.k_ranges <= 1) return hipErrorInvalidValue;
    if (a.M > 16 && rows_stream(a, epi)) return launch_rows(a, epi, s);
    if (epi == EPI_BIAS && is_plain(a) && short_k_wide(a.M, a.N, a.K)) {
        const int tn = (a.N + 127) / 128;
        hipLaunchKernelGGL((gemm_mfma_dma64<64, 128, 2, 2, EPI_BIAS, 3, 1, 0>), dim3(tn), dim3(256), 0, s, a, 1, tn);
        return hipGetLastError();
    }
    // A few more rows than the weight-streaming kernels take at once (a decode step of more than 16 sequences, a very
    // short prompt): the same kernels with the rows cut into slices of 16 along gridDim.y, where that beats a tile kernel
    // that would run a handful of workgroups through the whole K loop (decode layer-step of the hidden-1024 layer at 32
    // sequences: 91 us with the tile kernels, 38 us so; 128 sequences: 136 -> 73 us).
    if (!goes_to_tile_kernel(a)) {
        // enough workgroups to cover the chip first, then wider slices to amortise the activations
        if (try_flat(a, epi, s)) return hipGetLastError();
        if (try_stream(a, epi, s)) return hipGetLastError();
        if (a.N >= 64 * 1024) launch_skinny_cfg<4>(a, epi, s);
        else if (a.N >= 32 * 1024) launch_skinny_cfg<2>(a, epi, s);
        else launch_skinny_cfg<1>(a, epi, s);
    } else {
        const bool divisible = epi != EPI_QKV || a.tok_row_map != nullptr;       // see rows_from
        if (const int m_whole = divisible ? rows_in_whole_rounds(a.M, a.N) : 0) {
            // whole rounds of large tiles first, then the last few hundred rows as a problem of their own
            GemmArgs head = a;
            head.M = m_whole;
            hipError_t e = launch_gemm(head, epi, s);
            if (e != hipSuccess) return e;
            return launch_gemm(rows_from(a, epi, m_whole), epi, s);
        }
        // Four waves with 128 x 128 each in the 256 x 256 tile: a third less LDS read traffic per flop than eight waves of 128 x 64 (25082 x 49152 x 12288
        // 1.16 -> 1.23 PFLOP/s, 8192 x 16384 x 12288 1.20 -> 1.33, 2951 x 16384 x 4096 1.13 -> 1.24), at every K and row stride since the loads of a
        // step are spread over both of its halves (against eight waves with an early release of the stage, us: 3000 x 4096 x 32768 799 -> 661, 2048 x
        // 12288 x 49152 2518 -> 2149, its rows 128 bytes further apart 2379 -> 2077, 5000 x 10240 x 40960 4307 -> 3704).
        auto tile256 = [&] {
            if ((size_t)a.M * a.N * sizeof(half_t) >= kMemorySideCacheBytes) launch_dma64_cfg<2, 2, 256, 256, 2, 1, 1, true>(a, epi, s);
            else launch_dma64_cfg<2, 2, 256, 256, 2, 1, 1>(a, epi, s);
        };
        switch (full_tile(a.M, a.N, a.K)) {
        case kFull256: tile256(); return hipGetLastError();
        case kFull224x256: launch_dma64_cfg<2, 2, 224, 256, 2, 1, 1>(a, epi, s); return hipGetLastError();
        case kFull192x256: launch_dma64_cfg<2, 2, 192, 256, 2, 1, 1>(a, epi, s); return hipGetLastError();
        case kFull160x256: launch_dma64_cfg<2, 2, 160, 256, 3, 1, 2>(a, epi, s); return hipGetLastError();
        case kFull128x256: launch_dma64_cfg<2, 2, 128, 256, 3, 1, 2>(a, epi, s); return hipGetLastError();
        case kFull192: launch_dma64_cfg<2, 2, 192, 128, 3, 1, 2>(a, epi, s); return hipGetLastError();
        case kFull128: launch_dma64_cfg<2, 2, 128, 128, 3, 1, 2>(a, epi, s); return hipGetLastError();
        case kFull96: launch_dma64_cfg<2, 2, 96, 128, 4, 1, 2>(a, epi, s); return hipGetLastError();
        case kFullNone: break;
        }
        switch (tile_for(a.M, a.N, a.K)) {
        case kTile64: launch_dma64_cfg<2, 1, 64, 64, 3, 1, 2>(a, epi, s); break;
        case kTile64Split:
            if (reads_weights_past_l2(a.M, a.N, a.K, 64)) launch_dma64_cfg<2, 1, 64, 64, 3, 2, 0>(a, epi, s);
            else launch_dma64_cfg<2, 1, 64, 64, 3, 2, 2>(a, epi, s);
            break;
        case kTile128x64Split:
            if (reads_weights_past_l2(a.M, a.N, a.K, 128)) launch_dma64_cfg<4, 1, 128, 64, 3, 2, 0>(a, epi, s);
            else launch_dma64_cfg<4, 1, 128, 64, 3, 2, 2>(a, epi, s);
            break;
        case kTile128x64: launch_dma64_cfg<4, 1, 128, 64, 3>(a, epi, s); break;
        case kTile192Pair: launch_dma64_cfg<2, 2, 192, 128, 2, 1, 0>(a, epi, s); break;
        case kTile128PairShared: launch_dma64_cfg<2, 2, 128, 128>(a, epi, s); break;
        case kTile128Pair: launch_dma64_cfg<2, 2, 128, 128, 2, 1, 1>(a, epi, s); break;
        case kTile96: launch_dma64_cfg<2, 2, 96, 128, 4, 1, 2>(a, epi, s); break;
        case kTile128: launch_dma64_cfg<2, 2, 128, 128, 3, 1, 2>(a, epi, s); break;
        case kTile192: launch_dma64_cfg<2, 2, 192, 128, 3, 1, 2>(a, epi, s); break;
        case kTile128x256: launch_dma64_cfg<2, 2, 128, 256, 3, 1, 2>(a, epi, s); break;
        case kTile256: tile256(); break;
        }
    }
    return hipGetLastError();
}

}  // namespace eet
