// Shared device-side vocabulary for the gfx950 kernels: vector types, wave64 reductions,
// fp16 <-> fp32 helpers.  Everything here is inline device code; no host logic.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace eet {

typedef _Float16 half_t;
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef _Float16 half4v __attribute__((ext_vector_type(4)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;  // CDNA wavefront width

// Per-sequence lengths of one call, passed by value as a kernel argument (the only
// host->device metadata of a prefill: no mask tensor exists, Section 2.1 of the paper).
constexpr int kMaxBatch = 128;
struct SeqLens {
    int32_t len[kMaxBatch];
};

// ---- lane exchanges without the LDS --------------------------------------------------------------
// A shuffle goes through the LDS unit (ds_bpermute: some 100 cycles until its result is there), and a reduction over a wave is six of
// them behind one another; as data-parallel primitives and row swaps the same six steps are a few cycles each.  One LayerNorm row has twelve
// of them in its chain.
template <int CTRL>
__device__ __forceinline__ int dpp_word(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, false); }
template <int CTRL, class T>
__device__ __forceinline__ T dpp(T x) { return __builtin_bit_cast(T, dpp_word<CTRL>(__builtin_bit_cast(int, x))); }
// A lane's value and that of lane ^ 16 (^ 32), in the same order in both lanes: a swap of a register with itself leaves both in
// each.  The two elements are copied into scalars before the bit casts: __builtin_bit_cast applied to the vector element r[1]
// directly reads element 0 with this compiler, which silently turned a maximum into "the value of the lower lane" (a reference of the
// exponentials that ignored half of each row's keys: exact results until a row's scores span more than the 16 bits of
// headroom fp16 has above one, then infinities).
template <class T>
struct LanePair {
    T lower, upper;
};
template <class T>
__device__ __forceinline__ LanePair<T> pair_xor16(T x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    return {__builtin_bit_cast(T, r0), __builtin_bit_cast(T, r1)};
}
template <class T>
__device__ __forceinline__ LanePair<T> pair_xor32(T x) {
    const unsigned u = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    return {__builtin_bit_cast(T, r0), __builtin_bit_cast(T, r1)};
}
__device__ __forceinline__ float sum_xor16(float x) { const auto p = pair_xor16(x); return p.lower + p.upper; }
__device__ __forceinline__ float sum_xor32(float x) { const auto p = pair_xor32(x); return p.lower + p.upper; }
__device__ __forceinline__ float max_xor16(float x) { const auto p = pair_xor16(x); return fmaxf(p.lower, p.upper); }
__device__ __forceinline__ float max_xor32(float x) { const auto p = pair_xor32(x); return fmaxf(p.lower, p.upper); }

// Over the lane's 16: partners ^ 8, ^ 4, ^ 2, ^ 1, as a shuffle loop has them (4 by a rotation: after the first step lanes 8 apart agree)
template <class T, class Op>
__device__ __forceinline__ T reduce16(T v, Op op) {
    v = op(v, dpp<0x128>(v));
    v = op(v, dpp<0x124>(v));
    v = op(v, dpp<0x4e>(v));
    return op(v, dpp<0xb1>(v));
}
// Over the wave, ^ 32 and ^ 16 first; every lane calls it and gets the result
template <class T, class Op>
__device__ __forceinline__ T reduce_wave(T v, Op op) {
    const auto a = pair_xor32(v);
    v = op(a.lower, a.upper);
    const auto b = pair_xor16(v);
    return reduce16(op(b.lower, b.upper), op);
}
__device__ __forceinline__ float wave_sum(float v) {
    return reduce_wave(v, [](float x, float y) { return x + y; });
}
__device__ __forceinline__ float wave_max(float v) {
    return reduce_wave(v, [](float x, float y) { return fmaxf(x, y); });
}

// Over aligned groups of 8 lanes
__device__ __forceinline__ float sum8(float v) {
    v += dpp<0xb1>(v);
    v += dpp<0x4e>(v);
    return v + dpp<0x141>(v);
}
// x - m of two halfs in float, the operands taken as they are (a conversion is a half-rate instruction, and the compiler makes a
// conversion and an addition of a multiply-add by one)
__device__ __forceinline__ void minus_mean(half2v x, float m, float& d0, float& d1) {
    asm("v_fma_mix_f32 %0, %2, 1.0, -%3 op_sel_hi:[1,0,0]\n\tv_fma_mix_f32 %1, %2, 1.0, -%3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=&v"(d0), "=v"(d1) : "v"(x), "v"(m));
}
// LDS transpose read (gfx950): within 16 lanes, lane r supplies the address of 4 consecutive halfs "row r"; lane l
// receives element l%4 of rows l/4, l/4+4, l/4+8, l/4+12.
__device__ __forceinline__ half4v lds_read_tr16(const char* p) {
    typedef short short4v __attribute__((ext_vector_type(4)));
    const short4v v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((short4v __attribute__((address_space(3)))*)p);
    return __builtin_bit_cast(half4v, v);
}

// total / n (the same n in all lanes), inv_n = 1 / n as it is in float: the product, which is exact for a power of two, else corrected once by what it
// leaves over
__device__ __forceinline__ float mean_of(float total, int n, float inv_n) {
    float m = total * inv_n;
    if ((n & (n - 1)) != 0) m = __builtin_fmaf(__builtin_fmaf(-m, (float)n, total), inv_n, m);
    return m;
}

// Tokens of the sequences before sequence b: two loads and six lane exchanges whatever b is (a loop over the kernel argument
// is a scalar load and a wait per sequence).  Every lane of the wave calls it and gets the sum.
__device__ __forceinline__ int tokens_before(const SeqLens& lens, int b, int lane) {
    int n = (lane < b ? lens.len[lane] : 0) + (lane + 64 < b ? lens.len[lane + 64] : 0);
    return __builtin_amdgcn_readfirstlane(reduce_wave(n, [](int x, int y) { return x + y; }));
}

// Sum over a workgroup of NW waves; every thread gets the result.  `red` is LDS scratch of
// at least NW floats, reusable after the call returns.
template <int NW>
__device__ __forceinline__ float block_sum(float v, float* red) {
    v = wave_sum(v);
    if (NW == 1) return v;
    const int w = threadIdx.x / kWave, l = threadIdx.x % kWave;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < NW; ++i) t += red[i];
    return t;
}

// Load of data that a launch reads once (the weights of a decode step, the K/V rows of a decode attention): the
// non-temporal hint.  A read-only stream of 1-2 GB runs at 6.6-6.9 TB/s with it and at 5.5-6.05 TB/s without (16-byte
// loads, 8 or 16 in flight per lane, any grid), and the decode kernels gain the same tenth: cfg5b's attention 202 -> 180
// us, its FFN-2 weight stream 206 -> 187 us.  Operands that other workgroups read again (activation rows) keep plain loads.
template <class T>
__device__ __forceinline__ T load_once(const T* p) {
    return __builtin_nontemporal_load(p);
}

// tanh-form GELU in fp32 (the GPT-2 activation): 0.5 x (1 + tanh(u)), u = sqrt(2/pi) (x + 0.044715 x^3), written as
// x * sigmoid(2u) = x / (1 + 2^(-x (A + B x^2))) with A = 2 sqrt(2/pi) log2(e), B = 0.044715 A: seven vector
// instructions (one v_exp_f32, one v_rcp_f32), exact limits at +-inf (x * 0 and x * 1), no cancellation.
__device__ __forceinline__ float gelu_tanh(float x) {
    constexpr float A = 2.3022081985f, B = 0.10294323952f;
    const float t = __builtin_fmaf(x * x, B, A);
    const float e = __builtin_amdgcn_exp2f(-x * t);
    return x * __builtin_amdgcn_rcpf(e + 1.0f);
}

// The work of one prefetch workgroup (see PrefetchArgs in kernels.hpp): part `part` of `parts`, `nthreads` threads.
// One 4-byte load per 128-byte line.  The loads are ordinary loads whose values are xor-ed into a register that an
// empty asm statement "uses" at the end: nothing is stored, the compiler cannot drop the loads, and it keeps track
// of the registers they land in (a load whose destination the compiler believes dead would write that register
// later, after it has been given to something else).
// lines [lo, hi) of `base`, thread tid of nthreads: eight independent loads in flight per thread
__device__ __forceinline__ int touch_lines(const char* base, uint32_t lo, uint32_t hi, int tid, int nthreads) {
    int acc = 0;
    for (uint32_t i = lo + tid; i < hi; i += 8u * nthreads) {
        int v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t j = i + (uint32_t)u * nthreads;
            v[u] = j < hi ? *reinterpret_cast<const int*>(base + (size_t)j * 128) : 0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= v[u];
    }
    return acc;
}
template <class PF>
__device__ __forceinline__ void run_prefetch(const PF& p, int part, int parts, int tid, int nthreads) {
    int acc = 0;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint32_t lines = p.lin_lines[r];
        const uint32_t per = (lines + parts - 1) / parts, lo = part * per;
        const uint32_t hi = lo + per < lines ? lo + per : lines;
        if (lo < hi) acc ^= touch_lines(static_cast<const char*>(p.lin[r]), lo, hi, tid, nthreads);
    }
    if (p.k_cache != nullptr) {
        const int pairs = p.kv_batch * p.kv_heads;
        for (int bh = part; bh < pairs; bh += parts) {
            int rows = p.lens[bh / p.kv_heads];
            rows = rows < 0 ? 0 : (rows > p.kv_capacity ? p.kv_capacity : rows);                  // never past the pair's slots
            const uint32_t lines = (uint32_t)rows * (uint32_t)(p.kv_d * 2 / 128);                  // a row is 128 or 256 bytes
            const size_t off = (size_t)bh * p.kv_capacity * p.kv_d * 2;
            acc ^= touch_lines(reinterpret_cast<const char*>(p.k_cache) + off, 0, lines, tid, nthreads);
            acc ^= touch_lines(reinterpret_cast<const char*>(p.v_cache) + off, 0, lines, tid, nthreads);
        }
    }
    asm volatile("" ::"v"(acc));
}

}  // namespace eet
