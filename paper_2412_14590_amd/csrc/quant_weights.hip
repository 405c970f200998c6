// Offline weight path: quantize fp16 weights straight into the packed layouts, and convert
// between canonical (one code per byte, row-major) and packed arrays.
// Quantizer: Sec. 2 formula; 8-bit symmetric / 4-bit asymmetric group-wise, Sec. 3.1.2 and 4.1.
// The packed layouts are the ahead-of-time prepacking of Sec. 3.3, chosen for gfx950:
// every 16-byte slot is exactly what one lane feeds to an int8 MFMA as its B operand.
#include "internal.h"

namespace mixllm {

// ------------------------------------------------- order of the concatenated rows --
// feature_perm from a DEVICE list of the 8-bit channels (Sec. 3.4: the two parts own different
// channel indices; Alg. 1's per-layer slice arrives on the device from mixllm_select_salient):
// the listed channels ascending, then all others ascending.  No scratch memory: while the order
// is being built, bit 31 of perm[c] says "channel c is in the list" and the low 31 bits are the
// entry under construction (channel numbers are below 2^24).

__global__ __launch_bounds__(256) void perm_clear_kernel(int32_t *__restrict__ perm, int N)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c < N) perm[c] = 0;
}

// An index outside [0, N) is ignored; a channel listed twice is marked once.
__global__ __launch_bounds__(256) void perm_mark_kernel(const int32_t *__restrict__ idx, int n8, int32_t *__restrict__ perm,
                                                        int N)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n8) {
        const int c = idx[i];
        if (c >= 0 && c < N) perm[c] = (int32_t)0x80000000u;
    }
}

// One block walks the channels in order, 1024 at a time: a marked channel goes to the next free
// position of the first part, an unmarked one to the next free position of the second part.
// Position and channel of a write differ, so a write keeps the mark bit of the word it lands in
// (only the thread that owns a position writes its low bits; the mark bit is only ever read).
// With fewer than n8 distinct valid indices in the list the second part would run past N: those
// writes are dropped (the call's contract is a list of n8 distinct channels; a bad list gives an
// unspecified order, never an access out of bounds).
__global__ __launch_bounds__(1024) void perm_scan_kernel(int32_t *__restrict__ perm, int N, int n8)
{
    __shared__ int wave_tot[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int marked_before = 0;   // marked channels in the chunks already walked
    for (int c0 = 0; c0 < N; c0 += 1024) {
        const int c = c0 + tid;
        const int flag = (c < N && perm[c] < 0) ? 1 : 0;
        int inc = flag;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o, 64);
            if (lane >= o) inc += t;
        }
        if (lane == 63) wave_tot[wave] = inc;
        __syncthreads();   // every flag of the chunk has been read; wave totals are visible
        int base = 0, total = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            if (w < wave) base += wave_tot[w];
            total += wave_tot[w];
        }
        const int a = marked_before + base + inc - flag;   // marked channels before c
        if (c < N) {
            const int pos = flag ? a : n8 + (c - a);
            if (pos < N) perm[pos] = (perm[pos] & (int32_t)0x80000000u) | c;
        }
        marked_before += total;
        __syncthreads();   // wave_tot is rewritten by the next chunk; this chunk's writes are done
    }
    for (int c = tid; c < N; c += 1024) perm[c] &= 0x7fffffff;
}

// The same for up to PERM_CHANNELS channels in one launch, with the marks as a bitmap in LDS: every block
// builds the whole bitmap and the running count of marks per word for itself (the list is some
// thousand entries) and places a share of the channels.  Three dependent launches, the last of them one
// block walking 28 chunks of 1024 channels, took 16 us for 28672 channels,
// this one 5.
constexpr int PERM_CHANNELS = 1 << 17, PERM_SHARE = 4096;
__global__ __launch_bounds__(1024) void perm_bitmap_kernel(const int32_t *__restrict__ idx, int n8, int32_t *__restrict__ perm, int N)
{
    __shared__ uint32_t bits[PERM_CHANNELS / 32];
    __shared__ int before[PERM_CHANNELS / 32];   // marked channels in the words before
    __shared__ int wave_tot[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwords = (N + 31) / 32, per = (nwords + 1023) / 1024, w0 = tid * per, w1 = min(w0 + per, nwords);
    for (int w = tid; w < nwords; w += 1024) bits[w] = 0;
    __syncthreads();
    for (int i = tid; i < n8; i += 1024) {
        const int c = idx[i];
        if (c >= 0 && c < N) atomicOr(&bits[c >> 5], 1u << (c & 31));
    }
    __syncthreads();
    int mine = 0;
    for (int w = w0; w < w1; ++w) mine += __popc(bits[w]);
    int inc = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    int run = inc - mine, marked = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < wave) run += wave_tot[w];
        marked += wave_tot[w];
    }
    for (int w = w0; w < w1; ++w) {
        before[w] = run;
        run += __popc(bits[w]);
    }
    __syncthreads();
    const int c_end = min(((int)blockIdx.x + 1) * PERM_SHARE, N);
    for (int c = blockIdx.x * PERM_SHARE + tid; c < c_end; c += 1024) {
        const uint32_t word = bits[c >> 5];
        const int a = before[c >> 5] + __popc(word & ((1u << (c & 31)) - 1u));
        const int pos = (word >> (c & 31)) & 1u ? a : n8 + (c - a);
        if (pos < N) perm[pos] = c;
    }
    // (a list with fewer than n8 distinct valid channels leaves places free: still a channel number)
    if (blockIdx.x == 0)
        for (int i = marked + tid; i < n8; i += 1024) perm[i] = 0;
}

int launch_build_feature_perm(int N, int n8, const int32_t *salient_idx_dev, int32_t *perm, hipStream_t st)
{
    if (N <= 0) return (int)hipSuccess;
    if (N <= PERM_CHANNELS) {
        hipLaunchKernelGGL(perm_bitmap_kernel, dim3((N + PERM_SHARE - 1) / PERM_SHARE), dim3(1024), 0, st, salient_idx_dev, n8, perm, N);
        return (int)hipGetLastError();
    }
    hipLaunchKernelGGL(perm_clear_kernel, dim3((N + 255) / 256), dim3(256), 0, st, perm, N);
    if (n8 > 0)
        hipLaunchKernelGGL(perm_mark_kernel, dim3((n8 + 255) / 256), dim3(256), 0, st, salient_idx_dev, n8, perm, N);
    hipLaunchKernelGGL(perm_scan_kernel, dim3(1), dim3(1024), 0, st, perm, N, n8);
    return (int)hipGetLastError();
}

// ------------------------------------------------------------------ quantize + pack --
// Bound by HBM: two bytes in, half a byte (or one) out per weight.  The lanes of a wave are lanes of the
// packed layout: lane = row of the tile + 16 * k-slot, a wave reads 16 rows x 256 bytes of one group and writes
// the group's packed block as one contiguous KB (one block per row, writing 4-byte pieces 256 bytes apart,
// took 88 us for the 300 MB of K = 4096, N = 28672; this form 58).  Two things make a short launch longer than its
// bytes: blocks that walk too much in sequence and too few of them, hence the second form of the 8-bit part
// and the two sizes of a unit of the 4-bit part (rules at the launch).

constexpr int QP_THREADS = 512, QP_WAVES = QP_THREADS / 64;

static __device__ inline void absmax16(const h8 &a, const h8 &b, float &amax)
{
#pragma unroll
    for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fmaxf(fabsf((float)a[i]), fabsf((float)b[i])));
}
static __device__ inline uint4 codes8x16(const h8 &a, const h8 &b, float s, float r)
{
    uint32_t w[4];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        uint32_t v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = quant_bits(d < 2 ? a[4 * d + i] : b[4 * (d - 2) + i], s, r);
        w[d] = pack_low_bytes(v[0], v[1], v[2], v[3]);
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// One tile of 16 8-bit rows.  One scale per channel: each wave finds the maxima of two rows, the second read
// of the tile comes from the L2; then every wave takes every QP_WAVES-th group.
static __device__ inline void quantize_tile8(const half_t *__restrict__ W, const int32_t *__restrict__ perm, int K, int n8, int ng, int ngp,
                                             int w8_per_channel, int block, int8_t *__restrict__ w8, half_t *__restrict__ s8, float *row_scale)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r16 = lane & 15, ks = lane >> 4;
    const h8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
    const int r0 = block * TILE_N;
    if (w8_per_channel) {
        for (int i = wave; i < TILE_N; i += QP_WAVES) {
            const bool real = r0 + i < n8;
            float amax = 0.0f;
            if (real) {
                const half_t *row = W + (size_t)perm[r0 + i] * K;
                for (int k = lane * 16; k < K; k += 1024) absmax16(*(const h8 *)(row + k), *(const h8 *)(row + k + 8), amax);
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
            if (lane == 0) {
                const half_t s16 = real ? store_scale(amax / 127.0f) : (half_t)0.0f;
                s8[r0 + i] = s16;
                row_scale[i] = (float)s16;
            }
        }
        __syncthreads();
    }
    const int r = r0 + r16;
    const bool real = r < n8;
    const half_t *row = W + (size_t)(real ? perm[r] : 0) * K;
    float s = w8_per_channel ? row_scale[r16] : 0.0f, rs = recip(s);
    uint4 *out = (uint4 *)w8 + (size_t)block * (K / 64) * 64 + lane;
    for (int g = wave; g < (w8_per_channel ? ng : ngp); g += QP_WAVES) {
        if (g >= ng) {   // padding of the per-group scales
            if (ks == 0) s8[(size_t)r * ngp + g] = (half_t)0.0f;
            continue;
        }
        const half_t *src = row + g * G + ks * 16;   // 16 values in each half of the group
        h8 v[4] = {zero8, zero8, zero8, zero8};
        if (real) {
            v[0] = *(const h8 *)src;
            v[1] = *(const h8 *)(src + 8);
            v[2] = *(const h8 *)(src + 64);
            v[3] = *(const h8 *)(src + 72);
        }
        if (!w8_per_channel) {
            float amax = 0.0f;
            absmax16(v[0], v[1], amax);
            absmax16(v[2], v[3], amax);
            amax = fmaxf(amax, __shfl_xor(amax, 16, 64));
            amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
            const half_t s16 = real ? store_scale(amax / 127.0f) : (half_t)0.0f;
            if (ks == 0) s8[(size_t)r * ngp + g] = s16;
            s = (float)s16;
            rs = recip(s);
        }
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
            out[(size_t)(2 * g + hf) * 64] = real ? codes8x16(v[2 * hf], v[2 * hf + 1], s, rs) : make_uint4(0, 0, 0, 0);
    }
}

// A block's 2^lr (at most 8) 8-bit rows, r0 and on, where there are too few tiles for the chip: lane = row +
// 2^lr * slot, a slot being 16 consecutive k, so that a load of a wave always holds whole groups of the rows it
// touches.  The waves take the row's chunks (one load of a wave each) in turn, QP_AHEAD of them requested together.
// With one scale per channel the rows are walked twice (the second read comes from the L2 or the memory-side cache).
constexpr int QP_AHEAD = 4;
static __device__ inline void quantize_rows8(const half_t *__restrict__ W, const int32_t *__restrict__ perm, int K, int n8, int ng, int ngp,
                                             int w8_per_channel, int r0, int lr, int8_t *__restrict__ w8, half_t *__restrict__ s8,
                                             float *wave_max8)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rows = 1 << lr, slot = lane >> lr, r = r0 + (lane & (rows - 1));
    const bool real = r < n8;
    const half_t *row = W + (size_t)perm[min(r, n8 - 1)] * K;   // (a row of the padding reads the last one; its codes and scales are zero)
    const int nslots = K / 16, per = 64 >> lr, nchunks = (nslots + per - 1) / per;
    // chunk c of this lane: the slot past the end re-reads the last one (it changes no maximum and is not stored)
    auto load = [&](int c, h8 &a, h8 &b) {
        const half_t *src = row + min(c * per + slot, nslots - 1) * 16;
        a = *(const h8 *)src;
        b = *(const h8 *)(src + 8);
    };
    float s = 0.0f;
    if (w8_per_channel) {
        float amax = 0.0f;
        for (int c0 = wave; c0 < nchunks; c0 += QP_AHEAD * QP_WAVES) {
            h8 a[QP_AHEAD], b[QP_AHEAD];
#pragma unroll
            for (int j = 0; j < QP_AHEAD; ++j) load(c0 + j * QP_WAVES, a[j], b[j]);
#pragma unroll
            for (int j = 0; j < QP_AHEAD; ++j) absmax16(a[j], b[j], amax);
        }
        for (int o = 32; o >= rows; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
        if (slot == 0) wave_max8[wave * 8 + lane] = amax;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < QP_WAVES; ++w) amax = fmaxf(amax, wave_max8[w * 8 + (lane & (rows - 1))]);
        const half_t s16 = real ? store_scale(amax / 127.0f) : (half_t)0.0f;
        if (tid < rows) s8[r] = s16;
        s = (float)s16;
    } else if (wave == 0) {
        for (int g = ng + slot; g < ngp; g += per) s8[(size_t)r * ngp + g] = (half_t)0.0f;   // padding of the per-group scales
    }
    float rs = recip(s);
    uint4 *out = (uint4 *)w8 + (size_t)(r / TILE_N) * (K / 64) * 64 + r % TILE_N;
    for (int c0 = wave; c0 < nchunks; c0 += QP_AHEAD * QP_WAVES) {
        h8 a[QP_AHEAD], b[QP_AHEAD];
#pragma unroll
        for (int j = 0; j < QP_AHEAD; ++j) load(c0 + j * QP_WAVES, a[j], b[j]);
#pragma unroll
        for (int j = 0; j < QP_AHEAD; ++j) {
            const int q = (c0 + j * QP_WAVES) * per + slot;
            if (!w8_per_channel) {   // the 8 slots of a group lie in 8 lanes of the same row (a group is valid as a whole)
                float amax = 0.0f;
                absmax16(a[j], b[j], amax);
                for (int o = rows; o < 8 * rows; o <<= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
                const half_t s16 = real ? store_scale(amax / 127.0f) : (half_t)0.0f;
                if (q < nslots && (slot & 7) == 0) s8[(size_t)r * ngp + (q >> 3)] = s16;
                s = (float)s16;
                rs = recip(s);
            }
            const uint4 codes = codes8x16(a[j], b[j], s, rs);
            if (q < nslots) out[(size_t)(q >> 2) * 64 + 16 * (q & 3)] = real ? codes : make_uint4(0, 0, 0, 0);
        }
    }
}

// blocks [0, nblk8): one tile of 8-bit rows each (TILE8), or 2^lr of them; the others: QP_WAVES units of the 4-bit part each, a unit being
// one tile of 16 rows x U groups (U = 8 or 2; two groups are requested together)
template <bool TILE8, int U>
__global__ __launch_bounds__(QP_THREADS) void quantize_pack_kernel(
    const half_t *__restrict__ W, const int32_t *__restrict__ perm, int K, int n8, int n4, int nblk8, int lr, int n4p,
    int ng, int ngp, int w8_per_channel, int8_t *__restrict__ w8, uint8_t *__restrict__ w4,
    half_t *__restrict__ s8, half_t *__restrict__ s4, uint8_t *__restrict__ z4)
{
    __shared__ float maxima[TILE8 ? TILE_N : QP_WAVES * 8];
    if ((int)blockIdx.x < nblk8) {
        if constexpr (TILE8) quantize_tile8(W, perm, K, n8, ng, ngp, w8_per_channel, blockIdx.x, w8, s8, maxima);
        else quantize_rows8(W, perm, K, n8, ng, ngp, w8_per_channel, (int)blockIdx.x << lr, lr, w8, s8, maxima);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r16 = lane & 15, ks = lane >> 4;
    const int upt = ngp / U;   // units per tile
    const int unit = ((int)blockIdx.x - nblk8) * QP_WAVES + wave;
    if (unit >= n4p / TILE_N * upt) return;
    const int tile = unit / upt, g0 = (unit - tile * upt) * U;
    const int r = tile * TILE_N + r16;
    const bool real = r < n4;
    const half_t *row = W + (size_t)perm[n8 + min(r, n4 - 1)] * K + ks * 16;   // (padding rows read the last one, see quantize_rows8)
    uint4 *out = (uint4 *)w4 + ((size_t)tile * ng + g0) * 64 + lane;
    uint32_t scales[U / 2], zeros = 0;
#pragma unroll
    for (int i = 0; i < U / 2; ++i) scales[i] = 0;
#pragma unroll
    for (int u0 = 0; u0 < U; u0 += 2) {
        if (g0 + u0 >= ng) break;   // (the metadata of these padding groups is zero)
        h8 v[2][4];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const half_t *src = row + min(g0 + u0 + j, ng - 1) * G;
            v[j][0] = *(const h8 *)src;
            v[j][1] = *(const h8 *)(src + 8);
            v[j][2] = *(const h8 *)(src + 64);
            v[j][3] = *(const h8 *)(src + 72);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int u = u0 + j;
            if (g0 + u >= ng) break;
            float mn = 0.0f, mx = 0.0f;   // the range always contains 0
#pragma unroll
            for (int d = 0; d < 4; ++d)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    mn = fminf(mn, (float)v[j][d][i]);
                    mx = fmaxf(mx, (float)v[j][d][i]);
                }
#pragma unroll
            for (int o = 16; o < 64; o <<= 1) {
                mn = fminf(mn, __shfl_xor(mn, o, 64));
                mx = fmaxf(mx, __shfl_xor(mx, o, 64));
            }
            const half_t s16 = store_scale((mx - mn) / 15.0f);
            const float sc = (float)s16, rsc = recip(sc);
            const float zf = fminf(fmaxf(__builtin_rintf(quotient(-mn, sc, rsc)), 0.0f), 15.0f);
            const int z = (int)zf;
            // code = clamp(round(v / s) + z, 0, 15), the limits moved to the other side of the sum; the
            // eight biases of a dword are taken off (and z added) in one addition modulo 2^32
            const uint32_t fix = ((uint32_t)z - ROUND_BIAS) * 0x11111111u;
            uint32_t w[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                w[d] = fix;
#pragma unroll
                for (int i = 0; i < 8; ++i)   // byte b of a dword: k-local b in the low nibble, b + 4 in the high one
                    w[d] += rounded_bits(v[j][d][i], sc, rsc, -zf, 15.0f - zf) << (8 * (i & 3) + (i & 4));
            }
            out[u * 64] = real ? make_uint4(w[0], w[1], w[2], w[3]) : make_uint4(0, 0, 0, 0);
            if (real) {
                scales[u >> 1] |= (uint32_t)__builtin_bit_cast(uint16_t, s16) << (16 * (u & 1));
                zeros |= (uint32_t)z << (4 * u);
            }
        }
    }
    if (ks == 0) {
        half_t *so = s4 + (size_t)r * ngp + g0;
        uint8_t *zo = z4 + (size_t)r * (ngp / 2) + g0 / 2;
        if constexpr (U == 8) {
            *(uint4 *)so = make_uint4(scales[0], scales[1], scales[2], scales[3]);
            *(uint32_t *)zo = zeros;
        } else {
            *(uint32_t *)so = scales[0];
            *zo = (uint8_t)zeros;
        }
    }
}

int launch_quantize_weights(const mixllm_desc &d, const void *W, void *w8, void *w4, void *s8,
                            void *s4, void *z4, const int32_t *perm, hipStream_t st)
{
    const int n4 = d.N - d.n8, n8p = round_up(d.n8, TILE_N), n4p = round_up(n4, TILE_N);
    const int ng = d.K / G, ngp = round_up(ng, 8);
    if (n8p + n4p == 0) return hipSuccess;
    // Rows of a block of the 8-bit part.  Its two passes over 2^lr rows are a chain, and a launch with few other blocks
    // waits for it (one block per tile of 16 rows: K = 28672, N = 1024 with 102 8-bit channels 59 us, row order
    // included, K = 131072, N = 64 with 32 of them 229; here 24 and 24): it is hidden while the rows are at most
    // 1/600 of the layer's, and does not matter once the 8-bit blocks alone cover three quarters of the CUs; otherwise
    // the rows are halved, down to one.  (8 / 4 / 2 / 1 rows, K = 28672: N = 1024 with 102 8-bit channels
    // 49 / 34 / 22 / 23 us, with 1024 48 / 34 / 33 / 41, N = 8192 with 819 128 / 134 / 136 / 142; K = 4096, N = 6144
    // with 614 20 / 20 / 22 / 24.)  Whole tiles where there is one per CU (K = 4096, N = 28672, all channels 8-bit, a scale
    // per group: 102 us, in blocks of 8 rows 112) and on wide layers of short rows (K = 1152, N = 28672: 25, 30).
    const int cus = cu_count();
    const bool tile8 = n8p / TILE_N >= cus || (ng <= 16 && d.N >= 600 * TILE_N);
    int lr = tile8 ? 4 : 3;
    while (!tile8 && lr > 0 && 600 << lr > d.N && 4 * (n8p >> lr) < 3 * cus) --lr;
    // Groups of a unit of the 4-bit part: 2, requested together (units of 8: K = 1152, N = 300 15 us, here 9, K = N = 4096
    // 18.4, 14.5, K = 8192, N = 57344 263, 249), unless most of a row's units would be padding (K = 384, N = 28672 12.7 us, in
    // units of 2 14.2; K = 128, N = 131072 17, 28).
    const bool u8 = ng < 4;
    const int units = n4p / TILE_N * (ngp / (u8 ? 8 : 2)), nblk8 = n8p >> lr;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nblk8 + (units + QP_WAVES - 1) / QP_WAVES), dim3(QP_THREADS), 0, st, (const half_t *)W, perm,
                           d.K, d.n8, n4, nblk8, lr, n4p, ng, ngp, d.w8_group == d.K ? 1 : 0, (int8_t *)w8, (uint8_t *)w4, (half_t *)s8,
                           (half_t *)s4, (uint8_t *)z4);
    };
    if (tile8) u8 ? go(quantize_pack_kernel<true, 8>) : go(quantize_pack_kernel<true, 2>);
    else u8 ? go(quantize_pack_kernel<false, 8>) : go(quantize_pack_kernel<false, 2>);
    return (int)hipGetLastError();
}

// ------------------------------------------------------------ canonical -> packed --

__global__ __launch_bounds__(256) void pack_w4_kernel(const uint8_t *__restrict__ q4, int n4, int n4p,
                                                      int K, int ng, uint32_t *__restrict__ w4)
{
    const size_t total = (size_t)n4p * K / 8;   // packed dwords
    for (size_t o = (size_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (size_t)gridDim.x * 256) {
        const int dw = o & 3, l = (o >> 2) & 63;
        const size_t tg = o >> 8;                // tile * ng + g
        const int g = (int)(tg % ng), tile = (int)(tg / ng);
        const int r = tile * TILE_N + (l & 15), ks = l >> 4;
        const int k0 = g * G + (dw >> 1) * 64 + ks * 16 + (dw & 1) * 8;
        uint32_t packed = 0;
        if (r < n4) {
            const uint8_t *src = q4 + (size_t)r * K + k0;
#pragma unroll
            for (int b = 0; b < 4; ++b)
                packed |= ((uint32_t)(src[b] & 15) | ((uint32_t)(src[b + 4] & 15) << 4)) << (8 * b);
        }
        w4[o] = packed;
    }
}

__global__ __launch_bounds__(256) void pack_w8_kernel(const int8_t *__restrict__ q8, int n8, int n8p,
                                                      int K, uint4 *__restrict__ w8)
{
    const int nsteps = K / 64;
    const size_t total = (size_t)n8p * K / 16;   // 16-byte slots
    for (size_t o = (size_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (size_t)gridDim.x * 256) {
        const int l = o & 63;
        const size_t ts = o >> 6;
        const int step = (int)(ts % nsteps), tile = (int)(ts / nsteps);
        const int r = tile * TILE_N + (l & 15), ks = l >> 4;
        uint4 v = make_uint4(0, 0, 0, 0);
        if (r < n8) v = *(const uint4 *)(q8 + (size_t)r * K + step * 64 + ks * 16);
        w8[o] = v;
    }
}

// scales (fp16 [rows][ncan] -> [rowsp][nstride], zero padded); also used with ncan = nstride = 1
__global__ __launch_bounds__(256) void pack_scales_kernel(const half_t *__restrict__ src, int rows,
                                                          int rowsp, int ncan, int nstride,
                                                          half_t *__restrict__ dst)
{
    const size_t total = (size_t)rowsp * nstride;
    for (size_t o = (size_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (size_t)gridDim.x * 256) {
        const int r = (int)(o / nstride), g = (int)(o % nstride);
        dst[o] = (r < rows && g < ncan) ? src[(size_t)r * ncan + g] : (half_t)0.0f;
    }
}

__global__ __launch_bounds__(256) void pack_zeros_kernel(const uint8_t *__restrict__ z4c, int n4,
                                                         int n4p, int ng, int ngp,
                                                         uint8_t *__restrict__ z4)
{
    const size_t total = (size_t)n4p * (ngp / 2);
    for (size_t o = (size_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (size_t)gridDim.x * 256) {
        const int r = (int)(o / (ngp / 2)), g = 2 * (int)(o % (ngp / 2));
        uint32_t lo = 0, hi = 0;
        if (r < n4) {
            if (g < ng) lo = z4c[(size_t)r * ng + g] & 15;
            if (g + 1 < ng) hi = z4c[(size_t)r * ng + g + 1] & 15;
        }
        z4[o] = (uint8_t)(lo | (hi << 4));
    }
}

static inline int grid_for(size_t total)
{
    size_t b = (total + 255) / 256;
    return (int)(b < 1 ? 1 : (b > 65536 ? 65536 : b));
}

int launch_pack_weights(const mixllm_desc &d, const int8_t *q8, const void *s8c, const uint8_t *q4,
                        const void *s4c, const uint8_t *z4c, void *w8, void *w4, void *s8, void *s4,
                        void *z4, hipStream_t st)
{
    const int n4 = d.N - d.n8, n8p = round_up(d.n8, TILE_N), n4p = round_up(n4, TILE_N);
    const int ng = d.K / G, ngp = round_up(ng, 8);
    if (n4p) {
        hipLaunchKernelGGL(pack_w4_kernel, dim3(grid_for((size_t)n4p * d.K / 8)), dim3(256), 0, st, q4,
                           n4, n4p, d.K, ng, (uint32_t *)w4);
        hipLaunchKernelGGL(pack_scales_kernel, dim3(grid_for((size_t)n4p * ngp)), dim3(256), 0, st,
                           (const half_t *)s4c, n4, n4p, ng, ngp, (half_t *)s4);
        hipLaunchKernelGGL(pack_zeros_kernel, dim3(grid_for((size_t)n4p * ngp / 2)), dim3(256), 0, st,
                           z4c, n4, n4p, ng, ngp, (uint8_t *)z4);
    }
    if (n8p) {
        hipLaunchKernelGGL(pack_w8_kernel, dim3(grid_for((size_t)n8p * d.K / 16)), dim3(256), 0, st, q8,
                           d.n8, n8p, d.K, (uint4 *)w8);
        const int ncan = d.w8_group == d.K ? 1 : ng, nstride = d.w8_group == d.K ? 1 : ngp;
        hipLaunchKernelGGL(pack_scales_kernel, dim3(grid_for((size_t)n8p * nstride)), dim3(256), 0, st,
                           (const half_t *)s8c, d.n8, n8p, ncan, nstride, (half_t *)s8);
    }
    return (int)hipGetLastError();
}

// ------------------------------------------------------------ packed -> canonical --
// Bound by HBM (half a byte or one in, one out per weight).  Lanes and units are those of
// quantize_pack_kernel: a wave reads packed blocks as they lie, 1 KB at a time, and writes 16 bytes per
// lane, both halves of every 128-byte piece of a row.  One launch for codes, scales, zero points and the
// row order of both parts.  (A thread per packed dword with byte stores took 50 us for the 4-bit part of
// K = 4096, N = 28672, 158 MB, and the five launches beside it 35; this launch 39, 4.8 TB/s.)

template <bool ALIGNED>   // of the 4-bit codes, the one array of codes that may start at any byte
__global__ __launch_bounds__(256) void unpack_kernel(const uint4 *__restrict__ w8, const uint4 *__restrict__ w4,
                                                     const half_t *__restrict__ s8, const half_t *__restrict__ s4,
                                                     const uint8_t *__restrict__ z4, const int32_t *__restrict__ feature_perm, int K, int N,
                                                     int n8, int n4, int ng, int ngp, int w8_per_channel, int units8, int units4,
                                                     int8_t *__restrict__ q8, half_t *__restrict__ s8c, uint8_t *__restrict__ q4,
                                                     half_t *__restrict__ s4c, uint8_t *__restrict__ z4c, int32_t *__restrict__ perm)
{
    const int lane = threadIdx.x & 63, r16 = lane & 15, ks = lane >> 4, upt = ngp / 8;
    int unit = (int)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (unit < units8) {
        const int tile = unit / upt, g0 = (unit - tile * upt) * 8, r = tile * TILE_N + r16;
        if (r >= n8) return;
        const uint4 *src = w8 + ((size_t)tile * ng + g0) * 128 + lane;
        int8_t *dst = q8 + (size_t)r * K + g0 * G + ks * 16;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (g0 + u < ng) {
                *(uint4 *)(dst + u * G) = src[u * 128];
                *(uint4 *)(dst + u * G + 64) = src[u * 128 + 64];
            }
        if (w8_per_channel) {
            if (g0 == 0 && ks == 0) s8c[r] = s8[r];
        } else
            for (int g = g0 + 2 * ks; g < min(g0 + 2 * ks + 2, ng); ++g) s8c[(size_t)r * ng + g] = s8[(size_t)r * ngp + g];
        return;
    }
    unit -= units8;
    if (unit < units4) {
        const int tile = unit / upt, g0 = (unit - tile * upt) * 8, r = tile * TILE_N + r16;
        if (r >= n4) return;
        const uint4 *src = w4 + ((size_t)tile * ng + g0) * 64 + lane;
        uint8_t *dst = q4 + (size_t)r * K + g0 * G + ks * 16;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (g0 + u < ng) {
                const uint4 v = src[u * 64];
                const uint32_t lo = 0x0F0F0F0Fu;
                const uint4 c[2] = {make_uint4(v.x & lo, (v.x >> 4) & lo, v.y & lo, (v.y >> 4) & lo),
                                    make_uint4(v.z & lo, (v.z >> 4) & lo, v.w & lo, (v.w >> 4) & lo)};
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    uint8_t *o = dst + u * G + hf * 64;
                    if (ALIGNED) *(uint4 *)o = c[hf];
                    else {
                        const uint32_t d[4] = {c[hf].x, c[hf].y, c[hf].z, c[hf].w};
#pragma unroll
                        for (int i = 0; i < 16; ++i) o[i] = (uint8_t)(d[i >> 2] >> (8 * (i & 3)));
                    }
                }
            }
        for (int g = g0 + 2 * ks; g < min(g0 + 2 * ks + 2, ng); ++g) {
            s4c[(size_t)r * ng + g] = s4[(size_t)r * ngp + g];
            z4c[(size_t)r * ng + g] = (uint8_t)z4_load(z4, r, g, ngp);
        }
        return;
    }
    const int j = (unit - units4) * 64 + lane;
    if (perm && j < N) perm[j] = feature_perm[j];
}

int launch_unpack_weights(const mixllm_desc &d, const void *w8, const void *w4, const void *s8, const void *s4, const void *z4,
                          const int32_t *feature_perm, int8_t *q8, void *s8c, uint8_t *q4, void *s4c, uint8_t *z4c, int32_t *perm,
                          hipStream_t st)
{
    const int n4 = d.N - d.n8, ng = d.K / G, ngp = round_up(ng, 8), upt = ngp / 8;
    const int units8 = round_up(d.n8, TILE_N) / TILE_N * upt, units4 = round_up(n4, TILE_N) / TILE_N * upt;
    const int units = units8 + units4 + (perm ? (d.N + 63) / 64 : 0);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((units + 3) / 4), dim3(256), 0, st, (const uint4 *)w8, (const uint4 *)w4, (const half_t *)s8,
                           (const half_t *)s4, (const uint8_t *)z4, feature_perm, d.K, d.N, d.n8, n4, ng, ngp, d.w8_group == d.K ? 1 : 0,
                           units8, units4, q8, (half_t *)s8c, q4, (half_t *)s4c, z4c, perm);
    };
    if (((uintptr_t)q4 & 15u) == 0) go(unpack_kernel<true>);
    else go(unpack_kernel<false>);
    return (int)hipGetLastError();
}

}  // namespace mixllm
