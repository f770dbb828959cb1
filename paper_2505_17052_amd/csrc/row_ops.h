// Device helpers for activation rows, shared by the plan (which gathers the embeddings) and the matrix-core path.
#pragma once
#include "sev_internal.h"

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t b) { return __uint_as_float(b << 16); }

// hi/lo split of two floats at once with the packed hardware conversion (round to nearest even):
// hi = {bf16(a), bf16(b)}, lo = {bf16(a - hi_a), bf16(b - hi_b)}, element 0 in the low half.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_pack2(float a, float b, uint32_t &hi, uint32_t &lo) {
    const f32x2 v = {a, b};
    const bf16x2 h = __builtin_convertvector(v, bf16x2);
    const bf16x2 l = __builtin_convertvector(v - __builtin_convertvector(h, f32x2), bf16x2);
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, l);
}

// Writes 8 consecutive-k activations of row m (k0 a multiple of 8) as hi and lo fragments.
__device__ __forceinline__ void store_split8(uint16_t *xp, int m, int k0, int units, const float *v) {
    uint32_t h[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) split_pack2(v[2 * i], v[2 * i + 1], h[i], l[i]);
    *(uint4 *)(xp + xpack_index(m, k0, 0, units)) = make_uint4(h[0], h[1], h[2], h[3]);
    *(uint4 *)(xp + xpack_index(m, k0, 1, units)) = make_uint4(l[0], l[1], l[2], l[3]);
}

template <int THREADS>
__device__ __forceinline__ float block_sum(float v, float *red) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) s += red[w];
    __syncthreads();
    return s;
}

// Sums of squares of the residual rows are accumulated by many blocks; they are kept as 64-bit
// fixed point (2^-20 units) so that the atomic additions commute and the result is reproducible.
// One contribution (32 rows x <= 256 columns) is clamped to 1e10, so up to 1024 of them cannot wrap;
// what is lost below 2^-20 is far under the norm's epsilon once divided by the row width.
#define SSQ_SCALE 1048576.0f
__device__ __forceinline__ unsigned long long ssq_fix(float v) { return (unsigned long long)(fminf(v, 1.0e10f) * SSQ_SCALE); }
__device__ __forceinline__ float rms_scale(unsigned long long q, float inv_d, float eps) {
    return 1.0f / sqrtf((float)((double)q * (1.0 / 1048576.0)) * inv_d + eps);
}

// Where the embedding of a call's rows goes (plan_kernel's last blocks, one per row).
struct EmbedArgs {
    const void *E;             // [vocab][d], float32 or bfloat16
    float *h;                  // residual stream [rows][d]
    int d;
    // bfloat16 models: the first norm's gains, the operand split(h * g) of the first QKV GEMM (which applies the row's RMS scale
    // in its epilogue) and the rows' sums of squares
    const float *g;
    uint16_t *xa;
    unsigned long long *ssq_out, *ssq_clear;
    int units;
};

// Row m of the residual stream = E[tok]; 256 threads.
template <bool BF16>
__device__ __forceinline__ void embed_row(const EmbedArgs &e, int m, int tok, float *red) {
    float *hr = e.h + (size_t)m * e.d;
    if constexpr (!BF16) {
        const float *src = (const float *)e.E + (size_t)tok * e.d;
        for (int i = threadIdx.x; i < e.d; i += 256) hr[i] = src[i];
    } else {
        const uint16_t *src = (const uint16_t *)e.E + (size_t)tok * e.d;
        float ss = 0.f;
        for (int c = threadIdx.x; c < e.d / 8; c += 256) {
            const uint4 raw = *(const uint4 *)(src + c * 8);
            const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
            float v[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                v[2 * i] = bf16_bits_to_f32(w[i] & 0xffffu);
                v[2 * i + 1] = bf16_bits_to_f32(w[i] >> 16);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) ss += v[i] * v[i];
            *(float4 *)(hr + c * 8) = make_float4(v[0], v[1], v[2], v[3]);
            *(float4 *)(hr + c * 8 + 4) = make_float4(v[4], v[5], v[6], v[7]);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] *= e.g[c * 8 + i];
            store_split8(e.xa, m, c * 8, e.units, v);
        }
        ss = block_sum<256>(ss, red);
        if (threadIdx.x == 0) {
            e.ssq_out[m] = ssq_fix(ss);
            e.ssq_clear[m] = 0ull;
        }
    }
}
