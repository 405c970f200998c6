// Activation quantizer: fp16 -> int8 symmetric, one scale per token or per (token, group).
// Sec. 2 quantizer formula with z = 0; 8-bit symmetric activations, Sec. 3.1.2.
// HBM-streaming kernel: 2 B read + 1 B written per element.
#include "internal.h"

namespace mixllm {

// Exhaustive check of quotient(): for every positive finite fp16 scale (one block each) and every
// finite fp16 value the int8 code from quotient() against the code from the IEEE division.
__global__ __launch_bounds__(256) void check_fast_division_kernel(unsigned long long *mismatches)
{
    const uint16_t sb = (uint16_t)(blockIdx.x + 1);   // 0x0001 .. 0x7BFF
    const float s = (float)__builtin_bit_cast(half_t, sb);
    const float r = recip(s);
    unsigned long long bad = 0;
    for (int xb = threadIdx.x; xb < 65536; xb += 256) {
        if ((xb & 0x7C00) == 0x7C00) continue;   // infinities and NaNs
        const half_t x = __builtin_bit_cast(half_t, (uint16_t)xb);
        bad += (quant_bits(x, s, r) & 0xffu) != quant_code_ieee(x, s);
        // the 4-bit weight quantizer rounds the same quotient without the int8 clamp
        bad += __builtin_rintf(quotient((float)x, s, r)) != __builtin_rintf((float)x / s);
    }
    if (bad) atomicAdd(mismatches, bad);
}

// One block per token, the row held in registers between the absmax pass and the quantizing
// pass (NV vectors of 8 per thread: K <= 8 * NV * THREADS): one trip to memory instead of two,
// which is most of the duration of this kernel when M is small.
template <int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void act_quant_per_token_regs(const half_t *__restrict__ x,
                                                                    int8_t *__restrict__ xq,
                                                                    half_t *__restrict__ xs, int K)
{
    __shared__ float red[THREADS / 64];
    const int m = blockIdx.x;
    const h8 *row = (const h8 *)(x + (size_t)m * K);
    const int nvec = K / 8;
    h8 d[NV];
    u16x2 am = {0, 0};
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int v = threadIdx.x + THREADS * j;
        if (v < nvec) d[j] = row[v];
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
        if ((int)threadIdx.x + THREADS * j < nvec) absmax8(d[j], am);
    float amax = wave_max(absmax_of(am));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) amax = fmaxf(amax, red[w]);
    half_t s16 = store_scale(amax / 127.0f);
    const float s = (float)s16, r = recip(s);
    if (threadIdx.x == 0) xs[m] = s16;
    uint2 *out = (uint2 *)(xq + (size_t)m * K);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int v = threadIdx.x + THREADS * j;
        if (v < nvec) out[v] = quant8(d[j], s, r);
    }
}

// One block per token, any K; the row is read twice (the second read hits L2).
__global__ __launch_bounds__(1024) void act_quant_per_token(const half_t *__restrict__ x,
                                                            int8_t *__restrict__ xq,
                                                            half_t *__restrict__ xs, int K)
{
    __shared__ float red[16];
    const int m = blockIdx.x;
    const h8 *row = (const h8 *)(x + (size_t)m * K);
    const int nvec = K / 8;
    u16x2 am = {0, 0};
    for (int v = threadIdx.x; v < nvec; v += 1024) absmax8(row[v], am);
    float amax = wave_max(absmax_of(am));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 16; ++w) amax = fmaxf(amax, red[w]);
    half_t s16 = store_scale(amax / 127.0f);
    const float s = (float)s16, r = recip(s);
    if (threadIdx.x == 0) xs[m] = s16;
    uint2 *out = (uint2 *)(xq + (size_t)m * K);
    for (int v = threadIdx.x; v < nvec; v += 1024) out[v] = quant8(row[v], s, r);
}

// 16 lanes per quantization group of 128; a block covers 16 groups of one token.
__global__ __launch_bounds__(256) void act_quant_per_group(const half_t *__restrict__ x,
                                                           int8_t *__restrict__ xq,
                                                           half_t *__restrict__ xs, int K, int ng)
{
    const int m = blockIdx.x;
    const int g = blockIdx.y * 16 + (threadIdx.x >> 4);
    if (g >= ng) return;   // whole 16-lane groups leave together; no block barrier below
    const size_t off = (size_t)m * K + (size_t)g * G + (threadIdx.x & 15) * 8;
    h8 d = *(const h8 *)(x + off);
    u16x2 am = {0, 0};
    absmax8(d, am);
    const float amax = row16_max(absmax_of(am));
    half_t s16 = store_scale(amax / 127.0f);
    const float s = (float)s16;
    if ((threadIdx.x & 15) == 0) xs[(size_t)m * ng + g] = s16;
    *(uint2 *)(xq + off) = quant8(d, s, recip(s));
}

int launch_check_fast_division(unsigned long long *mismatches, hipStream_t st)
{
    hipLaunchKernelGGL(check_fast_division_kernel, dim3(0x7BFF), dim3(256), 0, st, mismatches);
    return (int)hipGetLastError();
}

int launch_quantize_activations(const mixllm_desc &d, const void *x, int8_t *xq, void *xs,
                                hipStream_t st)
{
    if (d.M == 0) return hipSuccess;
    if (d.act_group == d.K) {
        // A block as wide as its row: few tokens wait for one load instead of up to seven in a row
        // (K = 14336, 16 tokens: 4.3 us in 256 threads, 3.1 in 1024; K = 28672: 9.8 in the form that reads
        // the row twice, 4.4 here), many tokens are indifferent (K = 14336, 2048 tokens: 20.3 / 19.4) until
        // the block has threads without work (K = 4096, 8192 tokens: 20.3 us in 256 threads, 33 in 1024).
        // Before the packed maximum and the shorter rounding K = 14336 took 94 us at 8192 tokens, now 65
        // (5.4 TB/s), and 25 at 2048, now 19.
        auto go = [&](auto kernel, int threads) {
            hipLaunchKernelGGL(kernel, dim3(d.M), dim3(threads), 0, st, (const half_t *)x, xq, (half_t *)xs, d.K);
        };
        if (d.K <= 4096) go(act_quant_per_token_regs<2, 256>, 256);
        else if (d.K <= 8192) go(act_quant_per_token_regs<2, 512>, 512);
        else if (d.K <= 16384) go(act_quant_per_token_regs<2, 1024>, 1024);
        else if (d.K <= 32768) go(act_quant_per_token_regs<4, 1024>, 1024);
        else go(act_quant_per_token, 1024);
    } else {
        const int ng = d.K / G;
        hipLaunchKernelGGL(act_quant_per_group, dim3(d.M, (ng + 15) / 16), dim3(256), 0, st,
                           (const half_t *)x, xq, (half_t *)xs, d.K, ng);
    }
    return (int)hipGetLastError();
}

}  // namespace mixllm
