// Row-wise kernels: LayerNorm, add-bias+GELU, add-bias+residual, the mask-free softmax of
// Algorithm 1 as a stand-alone operator, and the index set-up of a prefill.
//
// The paper extends these kernels past 1024-wide rows by folding a virtual thread block into
// several real ones (Section 2.2).  On CDNA the same goal is met by folding in time: a fixed
// 256-thread workgroup (or one 64-lane wave for softmax rows) walks the row in 16-byte vectors,
// keeps the row in registers between the reduction and the write when it fits, and re-reads it
// (from L2) when it does not.  Any width works; widths that are a multiple of 8 take the
// vector path.  All of them are HBM-bound: bytes per row = 2 * width * sizeof(fp16).
#include "kernels.hpp"

namespace eet {

// ============================================================================================
// LayerNorm
// ============================================================================================
// NV > 0: each thread caches NV vectors of 8 halfs (width <= NV*2048, width % 8 == 0).
// EARLY: gamma and beta are requested with the row and not after the two reductions, where they are a second trip to memory for
// the few rows of a decode step (16 steps of a hidden-4096 layer, two such launches each: 1501 -> 1494 us; 3262 x 4096 10.9 -> 10.2).
// With many rows they are in the caches anyway, and the registers that hold them cost waves in flight (22640 x 4352 81 -> 94 us,
// 25311 x 12288 252 -> 274): up to 4096 rows only.
template <int NV, bool EARLY>
__global__ __launch_bounds__(256) void layernorm_cached(const half_t* __restrict__ x,
                                                        const int32_t* __restrict__ in_row_map,
                                                        const half_t* __restrict__ gamma,
                                                        const half_t* __restrict__ beta,
                                                        half_t* __restrict__ y, int width, float eps,
                                                        int32_t* bump_lens, int bump_count, ClearLines clear) {
    if (blockIdx.x == 0 && (int)threadIdx.x < clear.lines) clear.at[threadIdx.x * kClearStride] = 0u;
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const int64_t src = in_row_map ? (int64_t)in_row_map[row] : row;
    const half8v* xr = reinterpret_cast<const half8v*>(x + src * width);
    const int nvec = width >> 3;
    const int tid = threadIdx.x;

    const half8v* g8 = reinterpret_cast<const half8v*>(gamma);
    const half8v* b8 = reinterpret_cast<const half8v*>(beta);
    half8v v[NV], g[EARLY ? NV : 1], b[EARLY ? NV : 1];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = tid + i * 256;
        if (idx < nvec) {
            v[i] = xr[idx];
            if constexpr (EARLY) {
                g[i] = g8[idx];
                b[i] = b8[idx];
            }
        }
    }
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        if (tid + i * 256 < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += (float)v[i][e];
        }
    }
    const float mean = block_sum<4>(sum, red) / (float)width;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = tid + i * 256;
        if (idx < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float dlt = (float)v[i][e] - mean;
                sq += dlt * dlt;
            }
        }
    }
    const float var = block_sum<4>(sq, red) / (float)width;
    const float rstd = rsqrtf(var + eps);

    half8v* yr = reinterpret_cast<half8v*>(y + row * width);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = tid + i * 256;
        if (idx < nvec) {
            const int k = EARLY ? i : 0;
            if constexpr (!EARLY) {
                g[0] = g8[idx];
                b[0] = b8[idx];
            }
            half8v o;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                o[e] = (half_t)(((float)v[i][e] - mean) * rstd * (float)g[k][e] + (float)b[k][e]);
            yr[idx] = o;
        }
    }
    if (bump_lens != nullptr && tid == 0 && row < bump_count) bump_lens[row] += 1;
}

constexpr int kLayerNormWaveRows = 64;
// Many narrow rows (width <= 2048, width % 8 == 0; kLayerNormWaveRows and more): one wave per row, four rows per workgroup.  The row sits in NV
// 16-byte vectors per lane, both reductions are lane exchanges, and there is no barrier and no LDS, so a prompt's few
// thousand rows are all in flight at once instead of queueing behind 256-thread workgroups that each wait twice.  Scale and
// shift come with the row at every row count: against loads after the reductions 16000 x 768 10.4 -> 9.2 us, 64000 x 512 22.2 ->
// 21.1, 32000 x 2048 41.3 -> 39.0, at worst 8000 x 1536 9.65 -> 9.97 (54 sizes, up to 64000 rows).
//
// BLOCK_ORDER: the two reductions add in the order of layernorm_cached (one exchange per 512 columns, as one of its waves does,
// then those sums in turn), so that a row comes out with the same bits as there.  The launch that also sets up a prefill takes
// it below 64 rows, where launch_layernorm takes the 256-thread kernel: a layer's result does not depend on which of the two
// launches normalised its rows (the layers of a stack take one or the other).
template <int NV, bool BLOCK_ORDER>
__device__ __forceinline__ float sum_of_row(const float (&part)[NV]) {
    float t = 0.f;
    if constexpr (BLOCK_ORDER) {
#pragma unroll
        for (int i = 0; i < NV; ++i) t += wave_sum(part[i]);
    } else {
        t = wave_sum(part[NV - 1]);                           // part[i] goes on from part[i - 1]
    }
    return t;
}
template <int NV, bool BLOCK_ORDER = false>
__device__ __forceinline__ void layernorm_row_of_wave(const half_t* xrow, const half_t* __restrict__ gamma, const half_t* __restrict__ beta,
                                                      half_t* yrow, int width, float eps, int lane) {
    const half8v* xr = reinterpret_cast<const half8v*>(xrow);
    const half8v* g8 = reinterpret_cast<const half8v*>(gamma);
    const half8v* b8 = reinterpret_cast<const half8v*>(beta);
    const int nvec = width >> 3;
    half8v v[NV], g[NV], b[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            v[i] = xr[idx];
            g[i] = g8[idx];
            b[i] = b8[idx];
        }
    }
    float part[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        part[i] = BLOCK_ORDER || i == 0 ? 0.f : part[i - 1];
        if (lane + i * 64 < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) part[i] += (float)v[i][e];
        }
    }
    const float mean = sum_of_row<NV, BLOCK_ORDER>(part) / (float)width;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        part[i] = BLOCK_ORDER || i == 0 ? 0.f : part[i - 1];
        if (lane + i * 64 < nvec) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float dlt = (float)v[i][e] - mean;
                part[i] += dlt * dlt;
            }
        }
    }
    const float rstd = rsqrtf(sum_of_row<NV, BLOCK_ORDER>(part) / (float)width + eps);
    half8v* yr = reinterpret_cast<half8v*>(yrow);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = lane + i * 64;
        if (idx < nvec) {
            half8v o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (half_t)(((float)v[i][e] - mean) * rstd * (float)g[i][e] + (float)b[i][e]);
            yr[idx] = o;
        }
    }
}
template <int NV>
__global__ __launch_bounds__(256) void layernorm_wave(const half_t* __restrict__ x, const int32_t* __restrict__ in_row_map,
                                                      const half_t* __restrict__ gamma, const half_t* __restrict__ beta,
                                                      half_t* __restrict__ y, int rows, int width, float eps,
                                                      int32_t* bump_lens, int bump_count) {
    const int lane = threadIdx.x & 63;
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;                                  // whole waves leave; nothing below synchronises
    const int64_t src = in_row_map ? (int64_t)in_row_map[row] : (int64_t)row;
    layernorm_row_of_wave<NV>(x + src * width, gamma, beta, y + (int64_t)row * width, width, eps, lane);
    if (bump_lens != nullptr && lane == 0 && row < bump_count) bump_lens[row] += 1;
}

// Any width, any alignment: three scalar passes over the row (re-read through L2).
__global__ __launch_bounds__(256) void layernorm_generic(const half_t* __restrict__ x,
                                                         const int32_t* __restrict__ in_row_map,
                                                         const half_t* __restrict__ gamma,
                                                         const half_t* __restrict__ beta,
                                                         half_t* __restrict__ y, int width, float eps,
                                                         int32_t* bump_lens, int bump_count) {
    __shared__ float red[4];
    const int64_t row = blockIdx.x;
    const int64_t src = in_row_map ? (int64_t)in_row_map[row] : row;
    const half_t* xr = x + src * width;
    const int tid = threadIdx.x;
    float sum = 0.f;
    for (int c = tid; c < width; c += 256) sum += (float)xr[c];
    const float mean = block_sum<4>(sum, red) / (float)width;
    float sq = 0.f;
    for (int c = tid; c < width; c += 256) {
        const float dlt = (float)xr[c] - mean;
        sq += dlt * dlt;
    }
    const float var = block_sum<4>(sq, red) / (float)width;
    const float rstd = rsqrtf(var + eps);
    half_t* yr = y + row * width;
    for (int c = tid; c < width; c += 256)
        yr[c] = (half_t)(((float)xr[c] - mean) * rstd * (float)gamma[c] + (float)beta[c]);
    if (bump_lens != nullptr && tid == 0 && row < bump_count) bump_lens[row] += 1;
}

// The K ranges of a projection whose narrow output was cut along K (gemm_mfma_dma64 with EPI_PARTIAL): y = sum over the
// ranges, in order, + bias + residual, rounded once; and, with `gamma`, the LayerNorm that follows, of the row as stored.
// One workgroup per row, the row in registers: what it costs is one trip for the partial sums (out of L2 or the memory-side
// cache) and, with the LayerNorm, two block reductions, instead of a launch of its own for it.  n_b += 1 as in the kernels above.
template <int NT, int NV>
__global__ __launch_bounds__(NT) void finish_rows(const float* __restrict__ part, int ranges, int64_t range_stride, const half_t* __restrict__ bias,
                                                  const half_t* res, const int32_t* __restrict__ res_row_map, half_t* y,
                                                  const int32_t* __restrict__ out_row_map, const half_t* __restrict__ gamma,
                                                  const half_t* __restrict__ beta, half_t* __restrict__ ln_y, float eps, int width,
                                                  int32_t* bump_lens, int bump_count) {
    __shared__ float red[NT / kWave];
    const int row = blockIdx.x, tid = threadIdx.x, nvec = width >> 3;
    const int64_t rres = res_row_map ? (int64_t)res_row_map[row] : (int64_t)row;
    const int64_t rout = out_row_map ? (int64_t)out_row_map[row] : (int64_t)row;
    const float* pr = part + (int64_t)row * width;
    half8v v[NV], lg[NV], lb[NV];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int idx = tid + i * NT;
        if (idx >= nvec) continue;
        if (gamma != nullptr) {
            lg[i] = reinterpret_cast<const half8v*>(gamma)[idx];
            lb[i] = reinterpret_cast<const half8v*>(beta)[idx];
        }
        const half8v b = reinterpret_cast<const half8v*>(bias)[idx];
        const half8v r = reinterpret_cast<const half8v*>(res + rres * width)[idx];
        const float* pv = pr + idx * 8;
        float4v lo = *reinterpret_cast<const float4v*>(pv), hi = *reinterpret_cast<const float4v*>(pv + 4);
#pragma unroll 4
        for (int k = 1; k < ranges; ++k) {
            lo += *reinterpret_cast<const float4v*>(pv + k * range_stride);
            hi += *reinterpret_cast<const float4v*>(pv + k * range_stride + 4);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            v[i][e] = (half_t)((e < 4 ? lo[e & 3] : hi[e & 3]) + (float)b[e] + (float)r[e]);
            sum += (float)v[i][e];
        }
        reinterpret_cast<half8v*>(y + rout * width)[idx] = v[i];
    }
    if (gamma != nullptr) {                                    // uniform over the launch
        const float mean = block_sum<NT / kWave>(sum, red) / (float)width;
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            if (tid + i * NT >= nvec) continue;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float dlt = (float)v[i][e] - mean;
                sq += dlt * dlt;
            }
        }
        const float rstd = rsqrtf(block_sum<NT / kWave>(sq, red) / (float)width + eps);
        half8v* yr = reinterpret_cast<half8v*>(ln_y + (int64_t)row * width);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + i * NT;
            if (idx >= nvec) continue;
            half8v o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (half_t)(((float)v[i][e] - mean) * rstd * (float)lg[i][e] + (float)lb[i][e]);
            yr[idx] = o;
        }
    }
    if (bump_lens != nullptr && tid == 0 && row < bump_count) bump_lens[row] += 1;
}

hipError_t launch_finish_rows(const GemmArgs& a, hipStream_t s) {
    const dim3 grid(a.M);
#define EET_FINISH(NT, NV)                                                                                                       \
    hipLaunchKernelGGL((finish_rows<NT, NV>), grid, dim3(NT), 0, s, a.part, a.k_ranges, (int64_t)a.M * a.N, a.bias, a.res,       \
                       a.res_row_map, a.y, a.out_row_map, a.fin_gamma, a.fin_beta, a.fin_y, a.fin_eps, a.N, a.bump_lens, a.bump_count)
    if (a.fin_gamma != nullptr && a.fin_as_launch && a.N <= 2048 && a.M >= kLayerNormWaveRows) {       // layernorm_wave: one wave per row
        if (a.N <= 512) EET_FINISH(64, 1);
        else if (a.N <= 1024) EET_FINISH(64, 2);
        else EET_FINISH(64, 4);
    } else if (a.fin_gamma != nullptr && a.fin_as_launch && a.N > 2048) {                               // layernorm_cached: 256 threads
        if (a.N <= 4096) EET_FINISH(256, 2);
        else if (a.N <= 8192) EET_FINISH(256, 4);
        else if (a.N <= kFinishRowsMaxWidth) EET_FINISH(256, 8);
        else return hipErrorInvalidValue;
    } else if (a.N <= 1024) EET_FINISH(128, 1);
    else if (a.N <= 2048) EET_FINISH(256, 1);
    else if (a.N <= 4096) EET_FINISH(512, 1);
    else if (a.N <= 8192) EET_FINISH(512, 2);
    else if (a.N <= kFinishRowsMaxWidth) EET_FINISH(512, 4);
    else return hipErrorInvalidValue;
#undef EET_FINISH
    return hipGetLastError();
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// (rows and width of a layer's own activations: aligned)
bool layernorm_clears(int64_t rows, int width, int lines) {
    return lines <= 256 && width % 8 == 0 && width <= 16384 && (width > 2048 || rows < kLayerNormWaveRows);
}
hipError_t launch_layernorm(const half_t* x, const int32_t* in_row_map, const half_t* gamma,
                            const half_t* beta, half_t* y, int64_t rows, int width, float eps,
                            int32_t* bump_lens, int bump_count, hipStream_t s, ClearLines clear) {
    if (rows <= 0) return hipSuccess;
    if (clear.lines > 0 && !layernorm_clears(rows, width, clear.lines)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)rows), block(256);
    const bool vec = (width % 8 == 0) && aligned16(x) && aligned16(y) && aligned16(gamma) && aligned16(beta);
#define EET_LN_AT(NV, EARLY) hipLaunchKernelGGL((layernorm_cached<NV, EARLY>), grid, block, 0, s, x, in_row_map, gamma, beta, y, width, eps, bump_lens, bump_count, clear)
#define EET_LN(NV) do { if (rows <= 4096) EET_LN_AT(NV, true); else EET_LN_AT(NV, false); } while (0)
#define EET_LNW(NV) hipLaunchKernelGGL(layernorm_wave<NV>, dim3((unsigned)((rows + 3) / 4)), block, 0, s, x, in_row_map, gamma, beta, y, (int)rows, width, eps, bump_lens, bump_count)
    if (vec && width <= 2048 && rows >= kLayerNormWaveRows) { // a prompt's rows: one wave each
        if (width <= 512) EET_LNW(1);
        else if (width <= 1024) EET_LNW(2);
        else EET_LNW(4);
    } else if (vec && width <= 2048) EET_LN(1);
    else if (vec && width <= 4096) EET_LN(2);
    else if (vec && width <= 8192) EET_LN(4);
    else if (vec && width <= 16384) EET_LN(8);
    else
        hipLaunchKernelGGL(layernorm_generic, grid, block, 0, s, x, in_row_map, gamma, beta, y, width, eps,
                           bump_lens, bump_count);
#undef EET_LN
#undef EET_LN_AT
#undef EET_LNW
    return hipGetLastError();
}

// ============================================================================================
// add-bias + GELU, add-bias + residual   (4*width resp. 6*width bytes per row)
// ============================================================================================
// grid = (column chunks, row groups); each thread handles one 8-wide vector of a row.
template <bool RES>
__global__ __launch_bounds__(256) void bias_act_vec(const half_t* __restrict__ x, const half_t* __restrict__ bias,
                                                    const half_t* __restrict__ res, half_t* __restrict__ y,
                                                    int64_t rows, int width) {
    const int nvec = width >> 3;
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= nvec) return;
    const half8v b = reinterpret_cast<const half8v*>(bias)[c];
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
        const int64_t off = r * nvec + c;
        const half8v v = reinterpret_cast<const half8v*>(x)[off];
        half8v o;
        if (RES) {
            const half8v rr = reinterpret_cast<const half8v*>(res)[off];
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (half_t)((float)v[e] + (float)b[e] + (float)rr[e]);
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (half_t)gelu_tanh((float)v[e] + (float)b[e]);
        }
        reinterpret_cast<half8v*>(y)[off] = o;
    }
}

template <bool RES>
__global__ __launch_bounds__(256) void bias_act_scalar(const half_t* __restrict__ x, const half_t* __restrict__ bias,
                                                       const half_t* __restrict__ res, half_t* __restrict__ y,
                                                       int64_t rows, int width) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= width) return;
    const float b = (float)bias[c];
    for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
        const int64_t off = r * width + c;
        const float v = (float)x[off] + b;
        y[off] = (half_t)(RES ? v + (float)res[off] : gelu_tanh(v));
    }
}

template <bool RES>
static hipError_t launch_bias_act(const half_t* x, const half_t* bias, const half_t* res, half_t* y,
                                  int64_t rows, int width, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const unsigned gy = (unsigned)(rows < 32768 ? rows : 32768);
    const bool vec = (width % 8 == 0) && aligned16(x) && aligned16(y) && aligned16(bias) && (!RES || aligned16(res));
    if (vec) {
        const dim3 grid((width / 8 + 255) / 256, gy);
        hipLaunchKernelGGL(bias_act_vec<RES>, grid, dim3(256), 0, s, x, bias, res, y, rows, width);
    } else {
        const dim3 grid((width + 255) / 256, gy);
        hipLaunchKernelGGL(bias_act_scalar<RES>, grid, dim3(256), 0, s, x, bias, res, y, rows, width);
    }
    return hipGetLastError();
}

hipError_t launch_bias_gelu(const half_t* x, const half_t* bias, half_t* y, int64_t rows, int width, hipStream_t s) {
    return launch_bias_act<false>(x, bias, nullptr, y, rows, width, s);
}
hipError_t launch_bias_residual(const half_t* x, const half_t* bias, const half_t* res, half_t* y, int64_t rows,
                                int width, hipStream_t s) {
    return launch_bias_act<true>(x, bias, res, y, rows, width, s);
}

// ============================================================================================
// Mask-free softmax (Algorithm 1), in place on scores [batch, heads, S, S]
// ============================================================================================
// One wave per query row.  Row i of sequence b is visited only if i < len[b] (pad queries are
// skipped); its window is keys 0..i -- the comparison of key index against query index that
// replaces the attention mask -- and entries i+1..S-1 of a visited row are set to zero.
// NV = 8-wide vectors cached per lane (S <= NV*512, S % 8 == 0).
template <int NV>
__global__ __launch_bounds__(256) void softmax_maskfree_vec(half_t* __restrict__ scores, SeqLens lens, int heads,
                                                            int S, float scale_log2e, int left) {
    const int lane = threadIdx.x % kWave;
    const int i = blockIdx.x * 4 + threadIdx.x / kWave;   // query row
    const int bh = blockIdx.y;
    const int b = bh / heads;
    const int first = left ? S - lens.len[b] : 0;          // Algorithm 1's padLen when the pads lead: first non-pad position
    if (i < first || i >= first + lens.len[b]) return;     // pad rows; also covers i >= S
    half8v* row = reinterpret_cast<half8v*>(scores + ((size_t)bh * S + i) * S);
    const int nvec = S >> 3;
    const int nwin = (i >> 3) + 1;                         // vectors up to the end of the window first..i
    const int vwin = first >> 3;                           // ... and from its start

    float t[NV][8];
    float m = -INFINITY;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int idx = lane + c * kWave;
        if (idx >= vwin && idx < nwin) {
            const half8v v = row[idx];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const bool ok = idx * 8 + e <= i && idx * 8 + e >= first;
                t[c][e] = ok ? (float)v[e] * scale_log2e : -INFINITY;
                m = fmaxf(m, t[c][e]);
            }
        }
    }
    m = wave_max(m);                                       // the first key is always in the window: m is finite
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int idx = lane + c * kWave;
        if (idx >= vwin && idx < nwin) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                t[c][e] = exp2f(t[c][e] - m);              // exp2(-inf) = 0 for masked entries
                sum += t[c][e];
            }
        }
    }
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;
#pragma unroll
    for (int c = 0; c < NV; ++c) {
        const int idx = lane + c * kWave;
        if (idx < nvec) {
            half8v o;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (idx >= vwin && idx < nwin) ? (half_t)(t[c][e] * inv) : (half_t)0.f;
            row[idx] = o;
        }
    }
}

// Any S: scalar three-pass version, one wave per row.
__global__ __launch_bounds__(256) void softmax_maskfree_generic(half_t* __restrict__ scores, SeqLens lens,
                                                                int heads, int S, float scale_log2e, int left) {
    const int lane = threadIdx.x % kWave;
    const int i = blockIdx.x * 4 + threadIdx.x / kWave;
    const int bh = blockIdx.y;
    const int b = bh / heads;
    const int first = left ? S - lens.len[b] : 0;
    if (i < first || i >= first + lens.len[b]) return;
    half_t* row = scores + ((size_t)bh * S + i) * S;
    float m = -INFINITY;
    for (int j = first + lane; j <= i; j += kWave) m = fmaxf(m, (float)row[j] * scale_log2e);
    m = wave_max(m);
    float sum = 0.f;
    for (int j = first + lane; j <= i; j += kWave) sum += exp2f((float)row[j] * scale_log2e - m);
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;
    for (int j = lane; j < S; j += kWave)
        row[j] = (j >= first && j <= i) ? (half_t)(exp2f((float)row[j] * scale_log2e - m) * inv) : (half_t)0.f;
}

hipError_t launch_softmax_maskfree(half_t* scores, const SeqLens& lens, int batch, int heads, int S, float scale,
                                   hipStream_t s, bool left_padded) {
    const int left = left_padded ? 1 : 0;
    const dim3 grid((S + 3) / 4, batch * heads), block(256);
    const float sl2 = scale * 1.4426950408889634f;
    const bool vec = (S % 8 == 0) && aligned16(scores);
#define EET_SM(NV) hipLaunchKernelGGL(softmax_maskfree_vec<NV>, grid, block, 0, s, scores, lens, heads, S, sl2, left)
    if (vec && S <= 512) EET_SM(1);
    else if (vec && S <= 1024) EET_SM(2);
    else if (vec && S <= 2048) EET_SM(4);
    else if (vec && S <= 4096) EET_SM(8);
    else if (vec && S <= 8192) EET_SM(16);
    else hipLaunchKernelGGL(softmax_maskfree_generic, grid, block, 0, s, scores, lens, heads, S, sl2, left);
#undef EET_SM
    return hipGetLastError();
}

// ============================================================================================
// Prefill index set-up: the padding offsets become integers on the device, nothing else.
// ============================================================================================
// One block per padded row r = b*S + i.  Valid row: record packed->padded map.  Pad row: zero
// the output row.  Block 0 also publishes the lengths and their prefix sums.
__global__ __launch_bounds__(64) void prefill_setup(SeqLens lens, int batch, int S, int width,
                                                    int32_t* __restrict__ cache_lens, int32_t* __restrict__ cu_seqlens,
                                                    int32_t* __restrict__ row_map, half_t* __restrict__ out, int left) {
    const int r = blockIdx.x;
    const int b = r / S, i = r % S;
    const int cu = tokens_before(lens, b, threadIdx.x);
    const int first = left ? S - lens.len[b] : 0;          // position of the sequence's token 0 in its padded row block
    if (i >= first && i < first + lens.len[b]) {
        if (threadIdx.x == 0) row_map[cu + i - first] = r;
    } else {
        half_t* o = out + (size_t)r * width;
        if ((width & 7) == 0) {
            half8v z;
#pragma unroll
            for (int e = 0; e < 8; ++e) z[e] = (half_t)0.f;
            for (int c = threadIdx.x; c < (width >> 3); c += 64) reinterpret_cast<half8v*>(o)[c] = z;
        } else {
            for (int c = threadIdx.x; c < width; c += 64) o[c] = (half_t)0.f;
        }
    }
    if (r == 0) {
        int acc = 0;
        for (int k = threadIdx.x; k < batch; k += 64) cache_lens[k] = lens.len[k];
        if (threadIdx.x == 0) {
            for (int k = 0; k < batch; ++k) {
                cu_seqlens[k] = acc;
                acc += lens.len[k];
            }
            cu_seqlens[batch] = acc;
        }
    }
}

// Part `part` of `parts` of the exchange area of a decode step (kernels.hpp: StepArea), `nthreads` threads
__device__ __forceinline__ void set_up_step_area(const StepArea& st, int part, int parts, int tid, int nthreads) {
    const uint32_t words = st.words * (uint32_t)st.groups;
    for (uint32_t i = part * nthreads + tid; i < words; i += parts * nthreads) st.ctl[i] = i % st.words < (uint32_t)kStepCtlWords ? 0ull : ~0ull;
}
static int step_area_blocks(const StepArea& st, int nthreads) { return (int)((st.words * (uint32_t)st.groups + 4 * nthreads - 1) / (4 * nthreads)); }

// The same set-up and the first LayerNorm of a prefill in one launch, rows of up to 2048 (width % 8 == 0): one wave per padded
// row, which is either zeroed in `out` or normalised into its packed place in `y`.  A short prompt is a chain of dependent
// launches, and this is one of eight less (4 prompts of 16 to 64 tokens, hidden 768: 51.5 -> 49.6 us for the layer).
template <int NV, bool FEW>
__global__ __launch_bounds__(256) void prefill_setup_layernorm(SeqLens lens, int batch, int S, int width, int32_t* __restrict__ cache_lens,
                                                               int32_t* __restrict__ cu_seqlens, int32_t* __restrict__ row_map, half_t* out,
                                                               int left, const half_t* x, const half_t* __restrict__ gamma,
                                                               const half_t* __restrict__ beta, half_t* __restrict__ y, float eps, StepArea step) {
    const int lane = threadIdx.x & 63;
    const int row_blocks = (batch * S + 3) / 4;
    if ((int)blockIdx.x >= row_blocks) {                      // workgroups past the rows: the exchange area of the decode steps to come
        set_up_step_area(step, (int)blockIdx.x - row_blocks, (int)gridDim.x - row_blocks, threadIdx.x, 256);
        return;
    }
    const int r = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r == 0) {
        static_assert(kMaxBatch == 2 * kWave, "two lengths per lane");
        int before = 0;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = h * kWave + lane;
            int n = k < batch ? lens.len[k] : 0;
            if (k < batch) cache_lens[k] = n;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int up = __shfl_up(n, o, kWave);
                if (lane >= o) n += up;
            }
            if (k < batch) cu_seqlens[k + 1] = before + n;
            before += __shfl(n, kWave - 1, kWave);
        }
        if (lane == 0) cu_seqlens[0] = 0;
    }
    if (r >= batch * S) return;                               // whole waves leave; nothing below synchronises
    const int b = r / S, i = r - b * S;
    const int len = lens.len[b], first = left ? S - len : 0;
    if (i >= first && i < first + len) {
        const int t = tokens_before(lens, b, lane) + i - first;
        if (lane == 0) row_map[t] = r;
        layernorm_row_of_wave<NV, FEW>(x + (int64_t)r * width, gamma, beta, y + (int64_t)t * width, width, eps, lane);
    } else {
        half8v z;
#pragma unroll
        for (int e = 0; e < 8; ++e) z[e] = (half_t)0.f;
        for (int c = lane; c < (width >> 3); c += 64) reinterpret_cast<half8v*>(out + (int64_t)r * width)[c] = z;
    }
}

bool prefill_setup_takes_layernorm(int width) { return width % 8 == 0 && width <= 2048; }
hipError_t launch_prefill_setup_layernorm(const SeqLens& lens, int batch, int S, int width, int32_t* cache_lens, int32_t* cu_seqlens,
                                          int32_t* row_map, half_t* out, bool left_padded, const half_t* x, const half_t* gamma,
                                          const half_t* beta, half_t* y, float eps, StepArea step, hipStream_t s) {
    const dim3 grid((batch * S + 3) / 4 + step_area_blocks(step, 256));
    int64_t rows = 0;
    for (int b = 0; b < batch; ++b) rows += lens.len[b];
#define EET_SETUP_LN_AT(NV, FEW) hipLaunchKernelGGL((prefill_setup_layernorm<NV, FEW>), grid, dim3(256), 0, s, lens, batch, S, width, cache_lens, cu_seqlens, row_map, out, left_padded ? 1 : 0, x, gamma, beta, y, eps, step)
#define EET_SETUP_LN(NV) do { if (rows < kLayerNormWaveRows) EET_SETUP_LN_AT(NV, true); else EET_SETUP_LN_AT(NV, false); } while (0)
    if (width <= 512) EET_SETUP_LN(1);
    else if (width <= 1024) EET_SETUP_LN(2);
    else EET_SETUP_LN(4);
#undef EET_SETUP_LN
#undef EET_SETUP_LN_AT
    return hipGetLastError();
}

// The device-side cache lengths set from the host (resuming from a saved K/V cache): one small fill kernel, so the
// call can sit in a stream or a captured graph like every other.
__global__ __launch_bounds__(kMaxBatch) void set_cache_lens(SeqLens lens, int batch, int32_t* __restrict__ cache_lens, StepArea step) {
    if (blockIdx.x > 0) set_up_step_area(step, (int)blockIdx.x - 1, (int)gridDim.x - 1, threadIdx.x, kMaxBatch);
    else if ((int)threadIdx.x < batch) cache_lens[threadIdx.x] = lens.len[threadIdx.x];
}

hipError_t launch_set_cache_lens(const SeqLens& lens, int batch, int32_t* cache_lens, StepArea step, hipStream_t s) {
    hipLaunchKernelGGL(set_cache_lens, dim3(1 + step_area_blocks(step, kMaxBatch)), dim3(kMaxBatch), 0, s, lens, batch, cache_lens, step);
    return hipGetLastError();
}

hipError_t launch_prefill_setup(const SeqLens& lens, int batch, int S, int width, int32_t* cache_lens,
                                int32_t* cu_seqlens, int32_t* row_map, half_t* out, hipStream_t s, bool left_padded) {
    hipLaunchKernelGGL(prefill_setup, dim3(batch * S), dim3(64), 0, s, lens, batch, S, width, cache_lens,
                       cu_seqlens, row_map, out, left_padded ? 1 : 0);
    return hipGetLastError();
}

}  // namespace eet
