// Global precision search (Sec. 3.2): the salience of every output channel of a layer
// (Eq. 4) and the choice of the T most salient channels over all layers (Alg. 1).
// Offline, off the timed path of the linear; the salience kernel is a plain streaming
// reduction over W and G (4 bytes per weight), the selection a radix select over the
// saliences' bit patterns followed by an ordered compaction.
#include <algorithm>

#include "internal.h"

namespace mixllm {

namespace {

// ---- channel salience -------------------------------------------------------------------
// One block of 4 waves per output channel.  A wave-wide 16-byte load covers 4 quantization
// groups (16 lanes x 8 values each); the group's range, scale and zero point are found inside
// the 16-lane segment exactly as the weight quantizer finds them, so the codes are the ones
// mixllm_quantize_weights would store for this row as a 4-bit row.
__global__ __launch_bounds__(256) void channel_salience_kernel(const half_t *__restrict__ W, const half_t *__restrict__ Gr,
                                                               int K, float weight, int accumulate,
                                                               float *__restrict__ salience)
{
    __shared__ float part[4];
    const int n = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const half_t *w_row = W + (size_t)n * K, *g_row = Gr + (size_t)n * K;
    float acc = 0.0f;
    // 512 values per wave and iteration, 2048 per block
    for (int k0 = wave * 512 + lane * 8; k0 < K; k0 += 2048) {
        const h8 w = *(const h8 *)(w_row + k0);
        const h8 g = *(const h8 *)(g_row + k0);
        float mn = 0.0f, mx = 0.0f;   // the range always contains 0
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mn = fminf(mn, (float)w[i]);
            mx = fmaxf(mx, (float)w[i]);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            mn = fminf(mn, __shfl_xor(mn, o, 16));
            mx = fmaxf(mx, __shfl_xor(mx, o, 16));
        }
        const float sc = (float)store_scale((mx - mn) / 15.0f);
        const float rsc = recip(sc);
        const float zf = fminf(fmaxf(__builtin_rintf(quotient(-mn, sc, rsc)), 0.0f), 15.0f);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float wf = (float)w[i];
            const float code = fminf(fmaxf(__builtin_rintf(quotient(wf, sc, rsc)) + zf, 0.0f), 15.0f);
            const float delta = (code - zf) * sc - wf;   // quantize(W) - W
            acc = __builtin_fmaf((float)g[i], delta, acc);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) part[wave] = acc;
    __syncthreads();
    if (tid == 0) {
        const float s1 = (part[0] + part[1]) + (part[2] + part[3]);
        const float s = fabsf(s1 + 0.5f * s1 * s1);
        salience[n] = (accumulate ? salience[n] : 0.0f) + weight * s;
    }
}

// ---- global selection -------------------------------------------------------------------
// Saliences are non-negative floats, so their bit patterns order like the values.  Three
// histogram passes over digits of 11, 11 and 10 bits (most significant first) find the bit pattern
// of the T-th largest salience and how many channels with exactly that value still belong to the
// chosen set; equal values are taken in the order of the concatenation (earlier layer, then lower
// channel).  The keys of a whole model are a megabyte or two: what bounds the selection is the
// number of dependent launches and, inside one, atomics on the same global address (one per block
// and occupied bin, about 20 ns each: the first pass of 1344 blocks of 256 threads took 28 us for
// 344064 keys).  So the blocks are few and large, every block works out the previous pass's digit
// for itself from the finished histogram instead of a launch of one thread doing so (4-9 us each),
// and the lists are written from the ranks that tiles of the CONCATENATION have - a block per layer
// walking its channels in order took 32 us to count and 117 us to write.  Seven launches where there were
// thirteen; the search over 32 layers of 344064 channels with two gradient samples of a 4096 x 28672
// layer (2 x 78 us of salience kernels) went from 493 to 262 us.

constexpr int SEL_THREADS = 1024;
constexpr int SEL_PASSES = 3;
constexpr int SEL_BINS = 2048;        // 11 bits; the last digit has 10 and uses the lower half
constexpr int SEL_OFFSETS = 1024;     // layer offsets the emitting block keeps in LDS
constexpr int SEL_MAX_TILES = 1024;   // tiles of the concatenation: one per thread of the block that adds up their counts

// digit of a pass: bits [shift, shift + width)
__host__ __device__ constexpr int sel_shift(int pass) { return pass == 0 ? 21 : pass == 1 ? 10 : 0; }
__host__ __device__ constexpr uint32_t sel_mask(int pass) { return pass == 2 ? 1023u : 2047u; }

struct SelectRank {
    uint32_t prefix;      // digits of the threshold found so far
    uint32_t remaining;   // rank still to be found among the keys with that prefix; after the last pass:
                          // number of channels equal to the threshold that are chosen
};
struct SelectState {
    SelectRank rank[SEL_PASSES + 1];   // [i]: before pass i.  Written by one block of the launch after that pass
    uint32_t hist[SEL_PASSES][SEL_BINS];
    uint32_t tile_gt[SEL_MAX_TILES], tile_eq[SEL_MAX_TILES];
};

// exclusive prefix sum of one value per thread over a block of 1024 (wave scans, then the 16 wave totals)
__device__ inline uint32_t block_exclusive_scan(uint32_t v, uint32_t *wave_tot, uint32_t &block_total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o, 64);
        if (lane >= o) inc += t;
    }
    __syncthreads();   // wave_tot may still be read from the previous call
    if (lane == 63) wave_tot[wave] = inc;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
        const uint32_t t = wave_tot[w];
        base += w < wave ? t : 0u;
        total += t;
    }
    block_total = total;
    return base + inc - v;
}

// The rank after pass `pass`, from its finished histogram: the largest digit with at least `remaining`
// keys at or above it.  Every block computes it (thread t looks at the t-th pair of bins from the top);
// block 0 leaves it for the next launch.
__device__ inline SelectRank pick_digit(SelectState *st, int pass, uint32_t *wave_tot, SelectRank *found)
{
    const SelectRank r = st->rank[pass];
    const int d = SEL_BINS - 1 - 2 * (int)threadIdx.x;
    const uint32_t hi = st->hist[pass][d], lo = st->hist[pass][d - 1];
    if (threadIdx.x == 0) *found = r;
    uint32_t total;
    const uint32_t above = block_exclusive_scan(hi + lo, wave_tot, total);   // keys with a digit above d (its barriers order *found)
    if (above < r.remaining && r.remaining <= above + hi + lo) {             // true in one thread
        const bool upper = r.remaining <= above + hi;
        found->prefix = r.prefix | ((uint32_t)(upper ? d : d - 1) << sel_shift(pass));
        found->remaining = r.remaining - above - (upper ? 0u : hi);
    }
    __syncthreads();
    const SelectRank out = *found;
    if (blockIdx.x == 0 && threadIdx.x == 0) st->rank[pass + 1] = out;
    return out;
}

// The layer offsets come from a host array that may be gone when the call returns, and the call
// must neither block nor stage a copy: they travel as kernel arguments, 128 at a time.
struct OffsetChunk {
    int64_t v[128];
};
__global__ void select_offsets_kernel(int64_t *dst, int n, OffsetChunk c)
{
    const int t = threadIdx.x;
    if (t < n) dst[t] = c.v[t];
}

// clears the counters and starts the ranks; the layers' counts start at zero; the first `n` layer offsets (a launch of
// their own in front of the first histogram cost a search over 32 layers 4 us)
__global__ __launch_bounds__(256) void select_init_kernel(SelectState *st, uint32_t T, int32_t *layer_counts, int L, int64_t *offsets, int n, OffsetChunk c)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 1 && (int)threadIdx.x < n) offsets[threadIdx.x] = c.v[threadIdx.x];
    if (i < SEL_PASSES * SEL_BINS) (&st->hist[0][0])[i] = 0;
    if (i == 0) st->rank[0] = SelectRank{0, T};
    for (int l = i; l < L; l += gridDim.x * 256) layer_counts[l] = 0;
}

// histogram of digit PASS over the keys whose higher digits equal the prefix
template <int PASS>
__global__ __launch_bounds__(SEL_THREADS) void select_hist_kernel(const uint32_t *__restrict__ keys, int64_t total, SelectState *st)
{
    __shared__ uint32_t h[SEL_BINS];
    __shared__ uint32_t wave_tot[SEL_THREADS / 64];
    __shared__ SelectRank found;
    h[threadIdx.x] = 0;
    h[threadIdx.x + SEL_THREADS] = 0;
    // The first four keys of a thread (all it has on up to a million channels) are requested before the digit is picked:
    // two trips to memory at a time instead of one after the other.
    constexpr int FIRST = 4;
    const int64_t i0 = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x, step = (int64_t)gridDim.x * SEL_THREADS;
    uint32_t first[FIRST];
#pragma unroll
    for (int j = 0; j < FIRST; ++j) first[j] = keys[min(i0 + j * step, total - 1)];
    uint32_t prefix = 0;
    if constexpr (PASS > 0) prefix = pick_digit(st, PASS - 1, wave_tot, &found).prefix;
    __syncthreads();
    constexpr int above = PASS == 0 ? 31 : sel_shift(PASS > 0 ? PASS - 1 : 0);
    auto take = [&](uint32_t k) {
        if (PASS == 0 || (k >> above) == (prefix >> above)) atomicAdd(&h[(k >> sel_shift(PASS)) & sel_mask(PASS)], 1u);
    };
#pragma unroll
    for (int j = 0; j < FIRST; ++j)
        if (i0 + j * step < total) take(first[j]);
    for (int64_t i = i0 + FIRST * step; i < total; i += step) take(keys[i]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int d = threadIdx.x + j * SEL_THREADS;
        if (h[d]) atomicAdd(&st->hist[PASS][d], h[d]);
    }
}

// per tile of the concatenation: channels above the threshold, channels equal to it
__global__ __launch_bounds__(SEL_THREADS) void select_count_kernel(const uint32_t *__restrict__ keys, int64_t total, int tile, SelectState *st)
{
    __shared__ uint32_t wave_tot[SEL_THREADS / 64];
    __shared__ SelectRank found;
    __shared__ uint32_t s_gt, s_eq;
    const int64_t lo = (int64_t)blockIdx.x * tile, hi = min(lo + tile, total);
    uint32_t next = keys[min(lo + (int64_t)threadIdx.x, total - 1)];   // (requested before the threshold is known)
    const uint32_t thr = pick_digit(st, SEL_PASSES - 1, wave_tot, &found).prefix;
    if (threadIdx.x == 0) s_gt = s_eq = 0;
    __syncthreads();
    uint32_t a = 0, b = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += SEL_THREADS) {
        const uint32_t k = next;
        next = keys[min(i + SEL_THREADS, total - 1)];
        a += k > thr;
        b += k == thr;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        a += __shfl_xor(a, o, 64);
        b += __shfl_xor(b, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        atomicAdd(&s_gt, a);
        atomicAdd(&s_eq, b);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st->tile_gt[blockIdx.x] = s_gt;
        st->tile_eq[blockIdx.x] = s_eq;
    }
}

// Layers and their channels are consecutive in the concatenation, so a chosen channel's place in
// `selected` is the number of chosen ones before it: those above the threshold, and of those equal to
// it the first `remaining`.  A tile's start comes from the counts of the tiles before it.
__global__ __launch_bounds__(SEL_THREADS) void select_emit_kernel(const uint32_t *__restrict__ keys, int64_t total, int tile,
                                                                  const int64_t *__restrict__ offsets, int L, const SelectState *st,
                                                                  int32_t *__restrict__ selected, int32_t *__restrict__ layer_counts)
{
    __shared__ uint32_t wave_tot[SEL_THREADS / 64];
    __shared__ int64_t s_off[SEL_OFFSETS];
    const int tid = threadIdx.x, lane = tid & 63;
    // the search for a channel's layer is a chain of dependent reads: from LDS unless there are very many layers
    const bool in_lds = L < SEL_OFFSETS;
    // everything the block starts from is requested at once
    const int64_t lo = (int64_t)blockIdx.x * tile, hi = min(lo + tile, total);
    uint32_t next = keys[min(lo + (int64_t)tid, total - 1)];
    const uint32_t gt_before = tid < (int)blockIdx.x ? st->tile_gt[tid] : 0u, eq_before = tid < (int)blockIdx.x ? st->tile_eq[tid] : 0u;
    if (in_lds && tid <= L) s_off[tid] = offsets[tid];
    auto layer_of = [&](int64_t c) {   // the last layer that starts at or before c (an empty one starts where the next does)
        int l = 0, r = L;              // offset of l <= c < offset of r
        while (r - l > 1) {
            const int m = (l + r) >> 1;
            if ((in_lds ? s_off[m] : offsets[m]) <= c) l = m;
            else r = m;
        }
        return l;
    };
    const uint32_t thr = st->rank[SEL_PASSES].prefix, take = st->rank[SEL_PASSES].remaining;
    uint32_t gt_seen, eq_seen;
    block_exclusive_scan(gt_before, wave_tot, gt_seen);
    block_exclusive_scan(eq_before, wave_tot, eq_seen);
    uint32_t written = gt_seen + min(eq_seen, take);
    for (int64_t c0 = lo; c0 < hi; c0 += SEL_THREADS) {
        const int64_t c = c0 + tid;
        const uint32_t k = c < hi ? next : 0u;
        next = keys[min(c + SEL_THREADS, total - 1)];
        const uint32_t is_eq = (c < hi && k == thr) ? 1u : 0u;
        // both counts of a chunk fit 16 bits: one scan finds them together
        const uint32_t is_gt = (c < hi && k > thr) ? 1u : 0u;
        uint32_t chunk;
        const uint32_t before = block_exclusive_scan(is_gt | (is_eq << 16), wave_tot, chunk);
        const uint32_t eq_rank = eq_seen + (before >> 16);
        const bool sel = is_gt || (is_eq && eq_rank < take);
        const uint32_t eq_here = min(eq_rank, take) - min(eq_seen, take);   // chosen equal ones of this chunk before this key
        const int first_l = layer_of(c0), last_l = layer_of(min(c0 + SEL_THREADS, hi) - 1);
        const uint32_t chosen = (chunk & 0xffffu) + min(eq_seen + (chunk >> 16), take) - min(eq_seen, take);
        const int l = first_l == last_l ? first_l : layer_of(min(c, hi - 1));
        if (sel) selected[written + (before & 0xffffu) + eq_here] = (int32_t)(c - (in_lds ? s_off[l] : offsets[l]));
        // how many of each layer: one addition where the whole chunk is one layer's (every wave of a wide
        // layer adding to its one address would queue up there), else one per wave and layer in it
        if (first_l == last_l) {
            if (tid == 0 && chosen) atomicAdd(&layer_counts[first_l], (int32_t)chosen);
        } else {
            for (uint64_t left = __ballot(sel); left;) {
                const int of = __shfl(l, __ffsll((unsigned long long)left) - 1, 64);
                const uint64_t same = __ballot(sel && l == of) & left;
                if (lane == 0) atomicAdd(&layer_counts[of], (int32_t)__popcll(same));
                left &= ~same;
            }
        }
        written += chosen;
        eq_seen += chunk >> 16;
    }
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

}  // namespace

int launch_channel_salience(const void *W, const void *Gr, int N, int K, float weight, int accumulate, float *salience,
                            hipStream_t st)
{
    if (N == 0) return (int)hipSuccess;
    hipLaunchKernelGGL(channel_salience_kernel, dim3(N), dim3(256), 0, st, (const half_t *)W, (const half_t *)Gr, K, weight,
                       accumulate, salience);
    return (int)hipGetLastError();
}

size_t select_salient_workspace_bytes(int L)
{
    return align_up(sizeof(SelectState), 256) + align_up(sizeof(int64_t) * (size_t)(L + 1), 256);
}

int launch_select_salient(const float *salience, const int64_t *layer_offsets_host, int L, int64_t T, int32_t *selected,
                          int32_t *layer_counts, void *workspace, hipStream_t st)
{
    SelectState *state = (SelectState *)workspace;
    int64_t *offsets = (int64_t *)((uint8_t *)workspace + align_up(sizeof(SelectState), 256));
    const int64_t total = layer_offsets_host[L];
    for (int o = 0; o <= L; o += 128) {
        OffsetChunk c;
        const int n = std::min(128, L + 1 - o);
        for (int i = 0; i < 128; ++i) c.v[i] = i < n ? layer_offsets_host[o + i] : 0;
        if (o == 0) {
            hipLaunchKernelGGL(select_init_kernel, dim3((SEL_PASSES * SEL_BINS + 255) / 256), dim3(256), 0, st, state, (uint32_t)T,
                               layer_counts, L, offsets, n, c);
            if (T == 0) return (int)hipGetLastError();   // every list is empty
        } else
            hipLaunchKernelGGL(select_offsets_kernel, dim3(1), dim3(128), 0, st, offsets + o, n, c);
    }
    const uint32_t *keys = (const uint32_t *)salience;
    const dim3 threads(SEL_THREADS);
    // four keys a thread and at most one block per CU: more blocks are more atomics on one address, fewer
    // leave the reads of a large model to too few CUs
    const dim3 blocks((unsigned)std::min<int64_t>(256, (total + 4 * SEL_THREADS - 1) / (4 * SEL_THREADS)));
    hipLaunchKernelGGL(select_hist_kernel<0>, blocks, threads, 0, st, keys, total, state);
    hipLaunchKernelGGL(select_hist_kernel<1>, blocks, threads, 0, st, keys, total, state);
    hipLaunchKernelGGL(select_hist_kernel<2>, blocks, threads, 0, st, keys, total, state);
    // tiles of whole chunks of 1024 keys, at most SEL_MAX_TILES of them
    const int64_t chunks = (total + SEL_THREADS - 1) / SEL_THREADS;
    const int tile = (int)((chunks + SEL_MAX_TILES - 1) / SEL_MAX_TILES) * SEL_THREADS;
    const dim3 tiles((unsigned)((total + tile - 1) / tile));
    hipLaunchKernelGGL(select_count_kernel, tiles, threads, 0, st, keys, total, tile, state);
    hipLaunchKernelGGL(select_emit_kernel, tiles, threads, 0, st, keys, total, tile, offsets, L, state, selected, layer_counts);
    return (int)hipGetLastError();
}

}  // namespace mixllm
