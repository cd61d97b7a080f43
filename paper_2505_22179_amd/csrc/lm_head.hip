// lm_head_topk: the draft model's fp16 language-model head (a GEMV-shaped fp16 x fp16 product over a
// vocabulary-sized weight, HBM-bound), the log-softmax of its logits and their top-k.  Contract in
// include/w4a16.h.
#include <type_traits>

#include "internal.h"
#include "devscope.h"

namespace w4 {

typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kLmDepth = 4;        // macro steps of weights in flight per wavefront
constexpr int kLmStepK = 128;      // k per macro step: 256 contiguous bytes of every weight row
constexpr int kLmChunk = 512;      // logits per wavefront of the statistics pass (small workspaces)
constexpr int kLmThreads = 256;
constexpr int kLmMaxTopK = 64;

// Packed LM-head weight: the vocabulary (padded to a multiple of 16 with zero rows) is cut into tiles
// of 16 tokens; tile t is one contiguous run of K / 32 blocks of 1 KB, block s holding W[16 t + c]
// [32 s + 8 r .. + 7] at byte (16 r + c) * 16 -- the first operand of one 16x16x32 MFMA for lane
// (r, c), so a wavefront's loads are 1 KB contiguous each and its whole tile is one linear stream.
__global__ void lm_head_pack_kernel(const _Float16 *__restrict__ W, u32x4 *__restrict__ packed, int V, int K,
                                    long long total)
{
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte piece each
    if (idx >= total) return;
    const int lane = (int)(idx & 63);
    const long long blk = idx >> 6;
    const int steps = K / 32;
    const int s = (int)(blk % steps);
    const int tile = (int)(blk / steps);
    const int r = lane >> 4, c = lane & 15;
    const int v = tile * 16 + c;
    u32x4 piece = {0u, 0u, 0u, 0u};
    if (v < V) piece = *reinterpret_cast<const u32x4 *>(W + (size_t)v * K + 32 * s + 8 * r);
    packed[idx] = piece;
}

// Statistics of the logits a workgroup has just produced, one entry per row and workgroup (a granule of NW * TWL * 16
// tokens): the largest logit and the sum of exp(logit - largest).  With them the softmax needs no pass of its own over the logits, and
// the top tokens of a row are known to lie in the granules with the largest maxima.  A granule without a finite logit
// sums relative to 0; a NaN never is a maximum and makes the sum a NaN.
struct LmStat {
    float max, sum;
};
constexpr float kNegInf = -__builtin_inff();
__device__ __forceinline__ float sum_base(float max) { return max == kNegInf ? 0.f : max; }

// a wavefront's part, and the workgroup's from those of NW wavefronts
template <int TWL, int MTL>
__device__ __forceinline__ void wave_stats(const float4v (&acc)[TWL][MTL], LmStat (&part)[MTL * 16], int tile0, int V)
{
    const int lane = threadIdx.x & 63;
    const int r = lane >> 4, c = lane & 15;
#pragma unroll
    for (int mt = 0; mt < MTL; ++mt) {
        float v[TWL][4], mx = kNegInf, se = 0.f;
#pragma unroll
        for (int t = 0; t < TWL; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {   // tokens past the vocabulary (padding, and tiles past the end) count for nothing
                v[t][i] = (tile0 + t) * 16 + 4 * r + i < V ? acc[t][mt][i] : kNegInf;
                mx = fmaxf(mx, v[t][i]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
        mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
        const float base = sum_base(mx);
#pragma unroll
        for (int t = 0; t < TWL; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) se += __expf(v[t][i] - base);
        se += __shfl_xor(se, 16, 64);
        se += __shfl_xor(se, 32, 64);
        if (r == 0) part[mt * 16 + c] = {mx, se};
    }
}
template <int ROWS, int NW>
__device__ __forceinline__ void store_stats(const LmStat (*part)[ROWS], LmStat *__restrict__ stats, int M)
{
    __syncthreads();
    const int row = threadIdx.x;
    if (row < M) {   // M <= ROWS <= the workgroup's threads
        float mx = kNegInf, se = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) mx = fmaxf(mx, part[w][row].max);
        const float base = sum_base(mx);
#pragma unroll
        for (int w = 0; w < NW; ++w) se += part[w][row].sum * __expf(part[w][row].max - base);
        stats[(size_t)row * gridDim.x + blockIdx.x] = {mx, se};
    }
}

// Logits.  A wavefront owns one vocabulary tile (16 tokens = the rows of the MFMA result, the up to 16
// hidden-state rows its columns) and streams the tile's K / 32 blocks with a ring of kLmDepth macro
// steps (4 blocks = 4 KB each) in flight; the x fragments (at most 16 x K fp16, L2-resident) are
// re-read per wavefront, which works on two neighbouring tiles at once so that each fragment serves
// both.  Tiles lie K * 32 bytes apart, a power of two for the usual hidden sizes:
// wavefronts that all walked k from 0 would ask the same few memory channels at any moment, so each
// starts at macro step (tile mod steps) and wraps around.
template <bool EVEN, int TWL, int MTL, int DEPTH>
__global__ __launch_bounds__(256) void lm_head_logits_kernel(const _Float16 *__restrict__ x,
                                                             const u32x4 *__restrict__ packed,
                                                             float *__restrict__ logits, LmStat *__restrict__ stats, int M, int V,
                                                             int K, int tiles)
{
    __shared__ LmStat part[4][MTL * 16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane >> 4, c = lane & 15;
    const int tile0 = (blockIdx.x * 4 + wave) * TWL;   // TWL consecutive tiles share every x fragment
    // a wavefront past the last tile repeats it: its logits are not stored, but it takes part in the statistics' barrier
    const int steps = K / kLmStepK;
    const u32x4 *wp[TWL];
#pragma unroll
    for (int t = 0; t < TWL; ++t)   // a tile past the end repeats the last one; its logits are not stored
        wp[t] = packed + (size_t)min(tile0 + t, tiles - 1) * (K / 32) * 64 + lane;
    const u32x4 *xp[MTL];           // MTL row tiles of 16 hidden-state rows; rows >= M repeat row M-1, never stored
#pragma unroll
    for (int mt = 0; mt < MTL; ++mt) xp[mt] = reinterpret_cast<const u32x4 *>(x + (size_t)min(mt * 16 + c, M - 1) * K + 8 * r);
    u32x4 w[DEPTH][TWL][4], xf[DEPTH][MTL][4];
    const int rot = (min(tile0, tiles - 1) / TWL) % steps;
    auto load = [&](int s, int slot) {
        int sr = s + rot;              // uniform
        sr = sr >= steps ? sr - steps : sr;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int t = 0; t < TWL; ++t) w[slot][t][j] = __builtin_nontemporal_load(wp[t] + (sr * 4 + j) * 64);
#pragma unroll
            for (int mt = 0; mt < MTL; ++mt) xf[slot][mt][j] = xp[mt][(sr * 4 + j) * 4];
        }
    };
    float4v acc[TWL][MTL];
#pragma unroll
    for (int t = 0; t < TWL; ++t)
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) acc[t][mt] = (float4v){0.f, 0.f, 0.f, 0.f};
    auto compute = [&](int slot) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int t = 0; t < TWL; ++t)
#pragma unroll
                for (int mt = 0; mt < MTL; ++mt)
                    acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, w[slot][t][j]),
                                                                        __builtin_bit_cast(half8v, xf[slot][mt][j]),
                                                                        acc[t][mt], 0, 0, 0);
    };
    if constexpr (EVEN) {   // steps is a multiple of the ring depth: every load of the steady state is unconditional
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) load(u, u);
        int s0 = 0;
        for (; s0 + DEPTH < steps; s0 += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                compute(u);
                load(s0 + u + DEPTH, u);
            }
        }
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) compute(u);
    } else {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u)
            if (u < steps) load(u, u);
        for (int s0 = 0; s0 < steps; s0 += DEPTH) {
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                if (s0 + u < steps) {   // uniform
                    compute(u);
                    if (s0 + u + DEPTH < steps) load(s0 + u + DEPTH, u);
                }
            }
        }
    }
    // lane (r, c) holds the logits of tokens 16 tile + 4 r .. + 3 for hidden-state row 16 mt + c
#pragma unroll
    for (int t = 0; t < TWL; ++t)
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) {
            const int v0 = (tile0 + t) * 16 + 4 * r, row = mt * 16 + c;
            if (row < M && tile0 + t < tiles) {
                float *dst = logits + (size_t)row * V + v0;
                if ((V & 3) == 0 && v0 + 3 < V) {
                    *reinterpret_cast<float4v *>(dst) = acc[t][mt];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (v0 + i < V) dst[i] = acc[t][mt][i];
                }
            }
        }
    if (stats) {   // uniform
        wave_stats<TWL, MTL>(acc, part[wave], tile0, V);
        store_stats<MTL * 16, 4>(part, stats, M);
    }
}

// Logits where the vocabulary is too small to fill the chip with wavefronts of whole walks.  A workgroup takes four tiles (64 tokens, the least
// granule) with kLmKeptSets wavefronts on each, which deal the macro steps out among them and meet in LDS, in order.  The hidden-state rows are copied
// to LDS before the walk, whole cache lines straight there, in as few phases as LDS holds their x tiles in, so the walk asks for weights only: in the
// kernel above x fragments are as many loads as weights, sixteen rows x 64 bytes each, and a wavefront's walk is a chain of K / 512 round
// trips; in the kernel below a step has a barrier.  Block (step, jp, hb) of 1 KB holds rows 8 hb .. + 7 times the 128 bytes of blocks 2 jp and 2 jp + 1 of the
// step, chunks swizzled as there.  HB = 1: at most eight rows, for which the lanes of rows 8 .. 15 read the first eight again (never stored).
// What bounds it: what one compute unit takes in (some 35 - 50 B/ns here) while V / 64 of them work, then launch, the x copies and the finishing
// kernel.  Whole call, top 8, us, before -> now: 16 rows, V = 4000, K = 2048 22.8 -> 13.6, 5120 48.0 -> 22.2, 8192 69.0 -> 29.9; V = 16000, K = 3200 38.5 -> 24.8;
// 6 rows, V = 10000, K = 1408 16.9 -> 12.9; 4 rows, V = 4000, K = 8192 31.9 -> 27.8; 40 rows, V = 5000, K = 8192 49.5 -> 39.7, K = 2048 18.8 -> 17.1.
constexpr int kLmKeptSets = 4, kLmKeptWaves = 4 * kLmKeptSets;
constexpr int kLmKeptLds = 144 * 1024;   // x tiles that fit beside the statistics
template <int HB, int DEPTH>
__global__ __launch_bounds__(64 * kLmKeptWaves) void lm_head_logits_kept_kernel(const _Float16 *__restrict__ x, const u32x4 *__restrict__ packed,
                                                                                float *__restrict__ logits, LmStat *__restrict__ stats, int M, int V,
                                                                                int K, int tiles, int phases, int phase_q, int phase_rem)
{
    constexpr int MTL = (HB + 1) / 2;
    extern __shared__ u32x4 xt[];   // [step of the phase][jp][hb][64]; afterwards the sums
    __shared__ LmStat part[4][MTL * 16];
    fetch_arguments_together(x, packed, logits, stats, M, V, K, tiles, phases, phase_q, phase_rem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane >> 4, c = lane & 15;
    const int t = wave & 3, set = wave >> 2;
    const int tile0 = blockIdx.x * 4 + t;   // a wavefront past the last tile repeats it; its logits are not stored
    const Stretch xs = stretch(x, (uint32_t)M * (uint32_t)K * 2);
    const Stretch ws = stretch(packed + (size_t)min(tile0, tiles - 1) * (K / 32) * 64, (uint32_t)K * 32);
    const auto xoff = [&](int hb) {   // byte offset of what this lane copies of block hb
        const int row8 = lane >> 3, row = min(hb * 8 + row8, M - 1);
        return ((uint32_t)row * (uint32_t)K + (uint32_t)(((lane & 7) ^ (4 * (hb & 1) + (row8 >> 1))) * 8)) * 2;
    };
    const uint32_t lane_off = (uint32_t)lane * 16;
    uint32_t xfrag[2];
    {
        const int h = HB == 1 ? 0 : c >> 3, row8 = c & 7, sw = 4 * h + (row8 >> 1);
        xfrag[0] = (uint32_t)(h * 64 + row8 * 8 + (r ^ sw));
        xfrag[1] = (uint32_t)(h * 64 + row8 * 8 + ((4 + r) ^ sw));
    }
    float4v acc[1][MTL];
#pragma unroll
    for (int mt = 0; mt < MTL; ++mt) acc[0][mt] = (float4v){0.f, 0.f, 0.f, 0.f};
    u32x4 w[DEPTH][4];
    for (int ph = 0; ph < phases; ++ph) {   // as many steps at a time as LDS holds x tiles of; uniform over the grid
        const int begin = ph * phase_q + min(ph, phase_rem), steps = phase_q + (ph < phase_rem ? 1 : 0);
        const int mine = (steps - set + kLmKeptSets - 1) / kLmKeptSets;   // >= DEPTH (checked by the host)
        if (ph > 0) __syncthreads();   // everybody has left the last phase's x tiles
        const uint32_t own = xoff(wave % HB);
        for (int b = wave; b < steps * 2 * HB; b += kLmKeptWaves)   // b = (step * 2 + jp) * HB + hb
            quad_to_lds(xs, xt + b * 64, kLmKeptWaves % HB == 0 ? own : xoff(b % HB), (uint32_t)(begin * 2 + b / HB) * 128);
        __builtin_amdgcn_sched_barrier(0);   // x before the weights: the wait below counts on it
        // tiles lie K * 32 bytes apart: each workgroup starts its walk at another step (see above)
        const int rot = (int)(blockIdx.x % (unsigned)mine);
        const auto step_of = [&](int i) {   // uniform, i < 2 * mine - rot
            const int k = i + rot;
            return (uint32_t)(set + kLmKeptSets * (k >= mine ? k - mine : k));
        };
        const auto load = [&](int i, int slot) {
#pragma unroll
            for (int j = 0; j < 4; ++j) w[slot][j] = stream_quad(ws, lane_off + (uint32_t)j * 1024, ((uint32_t)begin + step_of(i)) * 4096);
        };
        const auto compute = [&](int i, int slot) {
            const u32x4 *const tile = xt + step_of(i) * (2 * HB * 64);
            u32x4 xf[MTL][4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < MTL; ++mt) xf[mt][j] = tile[((j >> 1) * HB + 2 * mt) * 64 + xfrag[j & 1]];
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int mt = 0; mt < MTL; ++mt)
                    acc[0][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, w[slot][j]), __builtin_bit_cast(half8v, xf[mt][j]),
                                                                        acc[0][mt], 0, 0, 0);
        };
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) load(u, u);
        asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(4 * DEPTH) : "memory");   // everybody's x has landed
        int i = 0;
        for (; i + 2 * DEPTH <= mine; i += DEPTH) {   // uniform over the wavefront; no barrier inside
#pragma unroll
            for (int u = 0; u < DEPTH; ++u) {
                compute(i + u, u);
                load(i + u + DEPTH, u);
            }
        }
#pragma unroll
        for (int u = 0; u < 2 * DEPTH - 1; ++u)
            if (i + u < mine) {   // uniform
                compute(i + u, u % DEPTH);
                if (i + u + DEPTH < mine) load(i + u + DEPTH, u % DEPTH);
            }
    }
    // the sets of a tile meet, in order
    __syncthreads();   // everybody has left the x tiles
    float4v *const sums = reinterpret_cast<float4v *>(xt);
    if (set > 0)
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) sums[(wave * MTL + mt) * 64 + lane] = acc[0][mt];
    __syncthreads();
    if (set == 0) {
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) {
#pragma unroll
            for (int q = 1; q < kLmKeptSets; ++q) acc[0][mt] += sums[((q * 4 + t) * MTL + mt) * 64 + lane];
            const int v0 = tile0 * 16 + 4 * r, row = mt * 16 + c;
            if (row < M && tile0 < tiles) {
                float *dst = logits + (size_t)row * V + v0;
                if ((V & 3) == 0 && v0 + 3 < V) {
                    *reinterpret_cast<float4v *>(dst) = acc[0][mt];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (v0 + e < V) dst[e] = acc[0][mt][e];
                }
            }
        }
        if (stats) wave_stats<1, MTL>(acc, part[t], tile0, V);   // uniform
    }
    if (stats) store_stats<MTL * 16, 4>(part, stats, M);   // uniform
}

// Logits of more than 16 rows.  There the x fragments, not the weights, filled the load path of the kernel above: every
// wavefront fetched its own (sixteen rows x 64 bytes a load, the costliest pattern for a compute unit's address path,
// as many loads as for the weights).  Here the NW wavefronts of a workgroup walk k together on TWL tiles each and
// share the x tile of a macro step through LDS: whole cache lines, global -> LDS directly, requested two steps ahead into
// three buffers (and waited for one step later, see below), one barrier per step.  The tile is kept as MTL * 4 blocks of 1 KB, block (mt, jp, h) = rows 16 mt + 8 h .. + 7
// times the 128 bytes of blocks 2 jp and 2 jp + 1 of the step; the eight 16-byte chunks of a row sit at
// chunk ^ (4 h + row / 2), which spreads a fragment read over all LDS banks.  Workgroups start their k walk at
// different steps, as above.  What bounds it is the weight stream where it is long (V = 128256, K = 8192, 60 rows: 6.6 TB/s of weights);
// shorter walks also wait for their first tiles and at the barriers.  Whole call, top 1, V = 128256, against the kernel
// above: 60 rows, K = 8192 476 -> 333 us, K = 4096 250 -> 185; 24 rows, K = 8192 358 -> 328, K = 4096 183 -> 177.
constexpr int kLmSharedMaxK = 1 << 20;   // its descriptors and offsets are 32-bit (M * K * 2 and TWL * K * 32 bytes); wider heads take the kernel above
template <int MTL, int NW, int TWL, int DEPTH>
__global__ __launch_bounds__(64 * NW, 2) void lm_head_logits_shared_kernel(const _Float16 *__restrict__ x,
                                                                                    const u32x4 *__restrict__ packed,
                                                                                    float *__restrict__ logits,
                                                                                    LmStat *__restrict__ stats, int M, int V,
                                                                                    int K, int tiles)
{
    constexpr int kTileQuads = MTL * 4 * 64;   // 16-byte pieces of one step's x tile
    constexpr int kCopies = (MTL * 4 + NW - 1) / NW;
    __shared__ u32x4 xa[3][kTileQuads];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane >> 4, c = lane & 15;
    const int tile0 = (blockIdx.x * NW + wave) * TWL;
    const int steps = K / kLmStepK;
    // a tile past the end repeats the last one; its logits are not stored
    const uint32_t tile_bytes = (uint32_t)K * 32;
    const int first = min(tile0, tiles - 1);
    const Stretch ws = stretch(packed + (size_t)first * (K / 32) * 64, (uint32_t)TWL * tile_bytes);
    uint32_t tile_off[TWL];
#pragma unroll
    for (int t = 0; t < TWL; ++t) tile_off[t] = (uint32_t)(min(tile0 + t, tiles - 1) - first) * tile_bytes;
    const Stretch xs = stretch(x, (uint32_t)M * (uint32_t)K * 2);
    uint32_t xoff[kCopies];
#pragma unroll
    for (int i = 0; i < kCopies; ++i) {
        const int blk = wave + NW * i;
        const int mt = blk >> 2, jp = (blk >> 1) & 1, h = blk & 1, row8 = lane >> 3;
        const int chunk = (lane & 7) ^ (4 * h + (row8 >> 1));
        const int row = min(mt * 16 + h * 8 + row8, M - 1);   // rows >= M repeat row M - 1; their products are never stored
        xoff[i] = ((uint32_t)row * (uint32_t)K + (uint32_t)(jp * 64 + chunk * 8)) * 2;
    }
    const int rot = (int)(blockIdx.x % (unsigned)steps);
    auto wrapped = [&](int s) {   // uniform: the step of k that step s of the walk takes, s < 2 * steps - rot
        const int k = s + rot;
        return (uint32_t)(k >= steps ? k - steps : k);
    };
    auto copy_x = [&](int s, int buf) {
        const uint32_t from = wrapped(s) * (kLmStepK * 2);
#pragma unroll
        for (int i = 0; i < kCopies; ++i)
            if (wave + NW * i < MTL * 4)   // uniform
                quad_to_lds(xs, xa[buf] + (wave + NW * i) * 64, xoff[i], from);
    };
    u32x4 w[DEPTH][TWL][4];
    const uint32_t lane_off = (uint32_t)lane * 16;
    auto load_w = [&](int s, int slot, int t, int j) {
        w[slot][t][j] = stream_quad(ws, lane_off + (uint32_t)j * 1024, tile_off[t] + wrapped(s) * 4096);
    };
    // fragment (mt, j): lane (r, c) reads row 16 mt + c, elements 32 j + 8 r .. + 7 of the step
    uint32_t xfrag[2];
    {
        const int h = c >> 3, row8 = c & 7, sw = 4 * h + (row8 >> 1);
        xfrag[0] = (uint32_t)(h * 64 + row8 * 8 + (r ^ sw));
        xfrag[1] = (uint32_t)(h * 64 + row8 * 8 + ((4 + r) ^ sw));
    }
    float4v acc[TWL][MTL];
#pragma unroll
    for (int t = 0; t < TWL; ++t)
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) acc[t][mt] = (float4v){0.f, 0.f, 0.f, 0.f};
    copy_x(0, 0);
    if (steps > 1) copy_x(1, 1);
    __builtin_amdgcn_sched_barrier(0);   // the counted waits below rely on the order of these requests, here and in step()
#pragma unroll
    for (int d = 0; d < DEPTH; ++d)
        if (d < steps)   // uniform
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < TWL; ++t) load_w(d, d, t, j);
    int b_now = 0, b_next = 1, b_free = 2;   // tile s + 2 goes where tile s - 1 was: everybody has read that by the barrier of step s
    auto step = [&](int s, int slot, bool more_w, bool more_x) {
        __syncthreads();
        if (more_x) copy_x(s + 2, b_free);
        __builtin_amdgcn_sched_barrier(0);   // x before the weights of this step: kNewer counts on it
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32x4 xf[MTL];
#pragma unroll
            for (int mt = 0; mt < MTL; ++mt) xf[mt] = xa[b_now][mt * 256 + (j >> 1) * 128 + xfrag[j & 1]];
#pragma unroll
            for (int t = 0; t < TWL; ++t) {
#pragma unroll
                for (int mt = 0; mt < MTL; ++mt)
                    acc[t][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, w[slot][t][j]), __builtin_bit_cast(half8v, xf[mt]),
                                                                        acc[t][mt], 0, 0, 0);
                if (more_w) load_w(s + DEPTH, slot, t, j);
            }
        }
        const int b = b_now;
        b_now = b_next;
        b_next = b_free;
        b_free = b;
    };
    // A step's barrier says that its x tile is complete, so every wavefront first waits for its own share of it.  Newer
    // than that share are, from the third step on, the weights requested in the two steps before and one x share; in
    // the first two steps at least the DEPTH steps of weights the walk starts with.  These counts are the least that is
    // needed.  What runs is stricter: __syncthreads is a fence of the workgroup, and the compiler waits there for every copy into
    // LDS that it sees under way, vmcnt(0) at the first step of a trip of the loop and vmcnt(4 TWL) at the others, so
    // at most one step of weights stays in flight across a barrier.
    constexpr int kStepLoads = 4 * TWL, kNewer = 2 * kStepLoads + MTL * 4 / NW;
    static_assert(kNewer < 64 && DEPTH * kStepLoads < 64, "the wait counter has six bits");
    constexpr int kAhead = DEPTH > 2 ? DEPTH : 2;   // how far the requests of a step reach
    int s = 0;
    if (steps >= DEPTH) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DEPTH * kStepLoads) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma clang loop unroll(disable)
    for (; s + DEPTH - 1 + kAhead < steps; s += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (s + u > 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kNewer) : "memory");   // uniform
            step(s + u, u, true, true);
        }
    }
#pragma unroll
    for (int u = 0; u < DEPTH - 1 + kAhead; ++u)
        if (s + u < steps) {   // uniform
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            step(s + u, u % DEPTH, s + u + DEPTH < steps, s + u + 2 < steps);
        }
    // lane (r, c) holds the logits of tokens 16 tile + 4 r .. + 3 for hidden-state row 16 mt + c
#pragma unroll
    for (int t = 0; t < TWL; ++t)
#pragma unroll
        for (int mt = 0; mt < MTL; ++mt) {
            const int v0 = (tile0 + t) * 16 + 4 * r, row = mt * 16 + c;
            if (row < M && tile0 + t < tiles) {
                float *dst = logits + (size_t)row * V + v0;
                if ((V & 3) == 0 && v0 + 3 < V) {
                    *reinterpret_cast<float4v *>(dst) = acc[t][mt];
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (v0 + i < V) dst[i] = acc[t][mt][i];
                }
            }
        }
    // b_now is the buffer after the last tile's: nothing was copied to it, and its readers have passed the last step's barrier
    static_assert(NW * MTL * 16 * sizeof(LmStat) <= sizeof(xa[0]), "the statistics of the wavefronts fit a buffer");
    if (stats) {   // uniform
        LmStat(*const part)[MTL * 16] = reinterpret_cast<LmStat(*)[MTL * 16]>(xa[b_now]);
        wave_stats<TWL, MTL>(acc, part[wave], tile0, V);
        store_stats<MTL * 16, NW>(part, stats, M);
    }
}

// (value, token) pairs ordered by value, equal values by ascending token
struct Cand {
    float val;
    int idx;
};
// (bitwise operators on purpose: no short-circuit branches in the scan loops)
__device__ __forceinline__ bool better(const Cand &a, const Cand &b) { return (a.val > b.val) | ((a.val == b.val) & (a.idx < b.idx)); }

// Wavefront-wide maximum, returned to every lane, on the data-parallel-primitive path of the
// vector ALU (no LDS round trips): quad butterflies, rotations inside each row of 16 lanes, then the
// four row results are read into scalars.
template <int CTRL>
__device__ __forceinline__ int dpp_move(int v)
{
    return __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false);
}
constexpr int kQuadXor1 = 0xB1, kQuadXor2 = 0x4E, kRowRor4 = 0x124, kRowRor8 = 0x128, kWaveShr1 = 0x138;

__device__ __forceinline__ float wave_max(float v)
{
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<kQuadXor1>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<kQuadXor2>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<kRowRor4>(__builtin_bit_cast(int, v))));
    v = fmaxf(v, __builtin_bit_cast(float, dpp_move<kRowRor8>(__builtin_bit_cast(int, v))));
    const int iv = __builtin_bit_cast(int, v);
    const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 0));
    const float b = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16));
    const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32));
    const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
    return fmaxf(fmaxf(a, b), fmaxf(c, d));
}

__device__ __forceinline__ float lane_value(float v, int lane)   // lane uniform
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
// set bits of a ballot below this lane
__device__ __forceinline__ int lanes_below(uint64_t which)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(which >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)which, 0));
}

// butterfly sum over the wavefront (fixed order), returned to every lane
__device__ __forceinline__ float wave_sum(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

constexpr int kNoToken = 0x7FFFFFFF;

// The statistics as a pass over the logits, for workspaces that hold one entry per 512 tokens only: one wavefront per chunk of
// 512 logits of one row.
__global__ __launch_bounds__(kLmThreads) void lm_head_stats_kernel(const float *__restrict__ logits, LmStat *__restrict__ stats, int V, int chunks)
{
    constexpr int kPerLane = kLmChunk / 64;
    const int lane = threadIdx.x & 63;
    const int chunk = blockIdx.x * (kLmThreads / 64) + (threadIdx.x >> 6), m = blockIdx.y;
    if (chunk >= chunks) return;
    const float *row = logits + (size_t)m * V;
    const int base = chunk * kLmChunk + lane;
    float val[kPerLane], mx = kNegInf, se = 0.f;
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
        val[i] = base + 64 * i < V ? row[base + 64 * i] : kNegInf;
        mx = fmaxf(mx, val[i]);
    }
    mx = wave_max(mx);
    const float from = sum_base(mx);
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) se += __expf(val[i] - from);
    se = wave_sum(se);
    if (lane == 0) stats[(size_t)m * chunks + chunk] = {mx, se};
}

// The best pairs seen so far, best first: lane l holds the l-th.
struct Best {
    Cand c = {kNegInf, kNoToken};
    // takes in the pairs of the lanes that offer one; `worst`: lane of the pair that a new one has to beat
    __device__ __forceinline__ void offer(Cand mine, bool offers, int worst)
    {
        const int lane = threadIdx.x & 63;
        for (;;) {
            const Cand last = {lane_value(c.val, worst), __builtin_amdgcn_readlane(c.idx, worst)};
            const uint64_t todo = __ballot(offers && better(mine, last));
            if (todo == 0) return;   // uniform; every round below withdraws one offer
            const int from = __builtin_ctzll(todo);
            const Cand cand = {lane_value(mine.val, from), __builtin_amdgcn_readlane(mine.idx, from)};
            const int place = __popcll(__ballot(better(c, cand)));   // the better ones are the first lanes
            const float up_val = __builtin_bit_cast(float, dpp_move<kWaveShr1>(__builtin_bit_cast(int, c.val)));
            const int up_idx = dpp_move<kWaveShr1>(c.idx);
            c.val = lane < place ? c.val : lane == place ? cand.val : up_val;
            c.idx = lane < place ? c.idx : lane == place ? cand.idx : up_idx;
            offers = offers && lane != from;
        }
    }
};

// Log of the sum of exponentials and the top tokens of a row, one workgroup per row.
//   1. The row's granules are dealt to the lanes.  The k-th largest of a wavefront's lane maxima is a value that k tokens
//      reach, and so is the least of the four wavefronts' (k / 4)-th largest: the row's k best tokens reach the larger of them all, the bound.
//   2. Only granules whose maximum reaches the bound are read again, and only their tokens that reach it are kept: k to
//      about 2 k of them where values differ.
//   3. A thread per kept token counts the better ones: its place.
// Many equal logits (rows of zeros), logits in order, or more places than granules bring more tokens to the bound than the lists
// hold.  Of granules that just reach it a wavefront reads only its first k, and where the bound is the largest logit of all it keeps
// only its first k tokens.  Else the logits that were read raise the bound in the way of step 1, and a second reading keeps the tokens that reach
// the new one, of ties the first k.  Where that is still too many, the wavefronts keep their k best in a third reading and the first merges
// them.  us, whole call, without these steps (third reading at once) and with them: 1 x 128256 (K = 1024), top 1, rows of zeros 167.5 -> 43.6,
// 10 x 128256 (K = 4096), top 10, the same 289.9 -> 165.5, 4 x 65000 (K = 1024), top 64, rising logits 595 -> 44 (random ones 33 before and now).
// Nothing in the usual path runs k times in a row.  A round trip to memory for the statistics, one for the logits: latency bounds it.
// The two passes this replaces (the k best of every 512 logits, then a merge of those lists) read all logits again:
// top 10 of 10 x 128256 8.3 + 9.6 -> 7.8 us, top 1 of 60 x 128256 8.3 + 4.7 -> 4.8; whole calls 174.0 -> 165.6 and 337.7 -> 328.9 (K = 4096, 8192),
// top 10 of 5 x 5000 (K = 2048) 26.2 -> 17.9, top 32 of 64 x 128256 271 -> 203.
constexpr int kLmKept = kLmThreads;       // tokens the lists hold, and the third step ranks
constexpr int kLmMaxPerLane = 16;         // 262144 tokens in granules of 64: 4096 of them over 256 lanes
constexpr int kLmAhead = 16;              // logits in flight per lane
template <int PER>
__global__ __launch_bounds__(kLmThreads) void lm_head_merge_kernel(const float *__restrict__ logits, const LmStat *__restrict__ stats, int V,
                                                                   int granules, int granule, int top_k, int32_t *__restrict__ top_idx,
                                                                   float *__restrict__ top_logprob)
{
    constexpr int kWaves = kLmThreads / 64;
    __shared__ float wave_alone[kWaves], wave_shared[kWaves];
    __shared__ LmStat wave_stat[kWaves];
    __shared__ int wave_kept[kWaves];
    __shared__ Cand kept[kWaves][kLmKept];
    __shared__ int chosen[kWaves][PER * 64];
    fetch_arguments_together(logits, stats, V, granules, granule, top_k, top_idx, top_logprob);
    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *const row = logits + (size_t)m * V;
    // This lane's granules.  Up to 64 stay with the first wavefront, which then knows the k-th largest maximum of all -- if there are k.  Otherwise
    // and up to 256 they are dealt in turn, so that each wavefront gives its share of the bound and of the reading: us, whole call, top 64 of
    // 10 x 22794 (K = 128) 70 -> 17.5, of 5 x 3808 53 -> 14.6.  More fill all lanes in either order, and this one reads the statistics in whole lines.
    const int first = PER == 1 && (granules > 64 || top_k > granules) ? lane * kWaves + wave : tid;
    LmStat st[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) st[i] = stats[(size_t)m * granules + min(first + kLmThreads * i, granules - 1)];   // lanes past the end drop theirs
    float lane_mx = kNegInf;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (first + kLmThreads * i >= granules) st[i] = {kNegInf, 0.f};
        lane_mx = fmaxf(lane_mx, st[i].max);
    }
    const float wave_mx = wave_max(lane_mx);
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < PER; ++i) se += st[i].sum * __expf(st[i].max - sum_base(wave_mx));   // absent ones: 0 * exp(-inf) = 0
    se = wave_sum(se);
    // values that k, and k / 4, of this wavefront's lanes reach with theirs
    const auto store_reached = [&](float lane_max) {
        float alone = kNegInf, shared = kNegInf;
        if (top_k > 1) {   // uniform
            int larger = 0;
#pragma unroll
            for (int l = 0; l < 64; ++l) larger += lane_value(lane_max, l) > lane_max ? 1 : 0;
            alone = -wave_max(larger < top_k ? -lane_max : kNegInf);   // the least of the lanes that fewer than k surpass
            shared = -wave_max(larger < (top_k + kWaves - 1) / kWaves ? -lane_max : kNegInf);
        }
        if (lane == 0) {
            wave_alone[wave] = alone;
            wave_shared[wave] = shared;
        }
    };
    const auto reached = [&]() {
        float alone = kNegInf, shared = wave_shared[0];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            alone = fmaxf(alone, wave_alone[w]);
            shared = fminf(shared, wave_shared[w]);
        }
        return fmaxf(alone, shared);
    };
    store_reached(lane_mx);
    if (lane == 0) wave_stat[wave] = {wave_mx, se};
    __syncthreads();
    float mx = kNegInf;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mx = fmaxf(mx, wave_stat[w].max);
    float bound = top_k > 1 ? reached() : mx;
    se = 0.f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) se += wave_stat[w].sum * __expf(wave_stat[w].max - sum_base(mx));
    const float lse = mx + __logf(se);

    // this wavefront's granules that reach the bound, as pieces of 64 tokens; of those that just reach it the first k, which hold k tokens
    // that do
    const auto reaches = [&](float v) { return v >= bound && v > kNegInf; };
    int found = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint64_t which = __ballot(reaches(st[i].max));
        if (reaches(st[i].max)) chosen[wave][found + lanes_below(which)] = first + kLmThreads * i;
        found += __popcll(which);
    }
    if (found > top_k) {   // uniform: once more, without those that are too many
        int level = 0;
        found = 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const bool just = reaches(st[i].max) && st[i].max == bound;
            const uint64_t which_just = __ballot(just);
            const bool take = reaches(st[i].max) && (!just || level + lanes_below(which_just) < top_k);
            const uint64_t which = __ballot(take);
            if (take) chosen[wave][found + lanes_below(which)] = first + kLmThreads * i;
            found += __popcll(which);
            level += __popcll(which_just);
        }
    }
    const int shift = 31 - __builtin_clz((unsigned)granule) - 6;   // granules are 64, 128, 256 or 512 tokens
    const int pieces = found << shift;
    // goes through them: take(logit, token) once per piece, lane by lane
    const auto each_piece = [&](auto take) {
        for (int p0 = 0; p0 < pieces; p0 += kLmAhead) {
            float l[kLmAhead];
            int token[kLmAhead];
#pragma unroll
            for (int i = 0; i < kLmAhead; ++i) {   // a piece past the last repeats it and is not looked at
                const int p = min(p0 + i, pieces - 1);
                token[i] = chosen[wave][p >> shift] * granule + (p & ((1 << shift) - 1)) * 64 + lane;
                l[i] = row[min(token[i], V - 1)];
            }
#pragma unroll
            for (int i = 0; i < kLmAhead; ++i)
                if (p0 + i < pieces) take(token[i] < V ? l[i] : kNegInf, token[i]);   // uniform
        }
    };
    int total, w_mine, at;   // the tid-th kept token is entry `at` of list w_mine
    float seen = kNegInf;    // the largest logit that this lane has read
    const int limit = bound == mx ? top_k : kLmKept;   // all tokens at the bound are equal: the first k of a wavefront will do
    // keeps the tokens that reach the bound; with `cut_ties` only the first k of this wavefront's that just reach it
    const auto collect = [&](auto cut_ties) {
        int keeps = 0, level = 0;
        each_piece([&](float l, int token) {
            bool keep = reaches(l);
            if constexpr (decltype(cut_ties)::value) {
                const uint64_t just = __ballot(keep && l == bound);
                keep = keep && (l > bound || level + lanes_below(just) < top_k);
                level += __popcll(just);
            } else {
                seen = fmaxf(seen, l);
            }
            const uint64_t which = __ballot(keep);
            const int place = keeps + lanes_below(which);
            if (keep && place < limit) kept[wave][place] = {l, token};
            keeps += __popcll(which);
        });
        if (lane == 0) wave_kept[wave] = limit < kLmKept ? min(keeps, limit) : keeps;   // more than a list holds: not enough of a bound
        __syncthreads();
        total = 0, w_mine = 0, at = tid;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int n = wave_kept[w];
            total += n;
            if (w_mine == w && at >= n && w + 1 < kWaves) at -= n, ++w_mine;
        }
    };
    collect(std::false_type{});
    if (total > kLmKept) {   // uniform
        store_reached(seen);
        __syncthreads();   // everybody has read the counts
        bound = fmaxf(bound, reached());
        collect(std::true_type{});
    }
    const auto store = [&](int place, Cand c) {
        top_idx[m * top_k + place] = c.idx;
        top_logprob[m * top_k + place] = c.val - lse;
    };
    if (total <= kLmKept) {   // uniform
        if (tid < top_k && tid >= total) store(tid, {kNegInf, kNoToken});   // fewer tokens than that have a logit
        if (wave * 64 >= total) return;
        const Cand mine = tid < total ? kept[w_mine][at] : Cand{kNegInf, kNoToken};
        int place = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
#pragma unroll 8
            for (int j = 0; j < wave_kept[w]; ++j) place += better(kept[w][j], mine) ? 1 : 0;
        if (tid < total && place < top_k) store(place, mine);
        return;
    }
    Best top;
    each_piece([&](float l, int token) { top.offer({l, token}, reaches(l), top_k - 1); });
    __syncthreads();   // everybody has left the lists
    kept[wave][lane] = top.c;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < kWaves; ++w) top.offer(kept[w][lane], lane < top_k && kept[w][lane].idx != kNoToken, top_k - 1);
    if (lane < top_k) store(lane, top.c);
}

// Which logits kernel, how many wavefronts share a workgroup and how many vocabulary tiles each takes.
// Up to 16 rows every wavefront fetches its own x fragments from L2 and a fragment serves all its tiles, which matters once
// the hidden-state rows differ (K = 4096: M = 16 240 -> 194 us with two); a single row is a broadcast and runs best with one.
// More rows share x through LDS.  A workgroup then takes T = 4, 8, 16 or 32 tiles and a compute unit works on about one at a
// time, so the call takes about rounds x T: the T with the least of it, where a smaller T also shares x less
// (V = 128256, where 8, 16 and 32 tie at a multiple of 256 workgroups: 204 / 192 / 177 us at 24 rows, K = 4096).  With T by this
// rule against 32 throughout: V = 4000 104 -> 32 us, 32000 113 -> 62, 50000 120 -> 82 (60 rows, K = 4096).
// Short walks amortise the fill of the pipeline over too few steps: up to K = 1024 at most eight tiles (V = 128256, 60 rows:
// 84 us with 32, 71 with 8, 73 in the kernel above), and with fewer rows the kernel above, whose wavefronts need no barrier, stays
// ahead beyond one such round (V = 128256: K = 1024 55 against 63 us at 24 rows, 62 against 67 at 40; K = 2048 95 against 97 at
// 24).  It also does where 16 tiles fill the chip and K is a power of two, so that all tiles of a workgroup ask the same memory
// channels at any moment (V = 64000: K = 4096 91 against 101 us at 24 rows, K = 2048 57 against 68 at 40 and 68 against 70 at 60;
// but K = 3840 90 against 84 at 24 rows, and K = 4096 103 against 100 at 40).  (All: whole call, top 1, two weight copies in turn.)
struct LmPlan { bool shared; int nw, twl; bool kept = false; };   // kept: the kernel that keeps x in LDS; nw * twl tiles to a workgroup there too
// Small vocabularies go to the kernel whose workgroups keep x in LDS, four tiles each: up to one workgroup per compute unit with 5 to 16 rows
// (beyond, a second pass over the chip costs more than is saved: 24000 tokens, K = 4096, 16 rows 49.0 against 51.1 us, 32000 51.7 against 60.5); up to
// 160 of them with more rows, which the kernel with shared x tiles serves better by then (16000 tokens, K = 2048, 60 rows 24.3 against 25.9; 10000
// tokens 21.4 against 20.7); up to 64 with four rows or fewer, whose x is little to fetch either way (16000 tokens, K = 4096, one row 27.4 against 33.6; 4000
// tokens, K = 5120 21.6 against 20.5).  Its walk goes in phases, the fewest whose x tiles fit LDS, each with two or four steps for every wavefront at least;
// with four rows or fewer, four.  On the shortest walks below that (K = 1024) this kernel is no gain: 4000 tokens, one row 9.8 against 9.6 us, two 9.9 against 9.8,
// four 10.0 against 10.1.  (From K = 1408 on it would be, K = 1920 10.7 against 11.2, 10.9 against 11.6 and 10.9 against 12.2: the line could lie lower.)
struct LmKept { int hb, depth, phases, q, rem; size_t lds; };
static LmKept lm_kept(int M, int K)
{
    const int hb = M <= 8 ? 1 : 2 * ((M + 15) / 16), steps = K / kLmStepK, tile = hb * 2048, most = kLmKeptLds / tile;
    const int phases = (steps + most - 1) / most, q = steps / phases, rem = steps % phases;
    const int depth = q >= 4 * kLmKeptSets ? 4 : q >= 2 * kLmKeptSets ? 2 : 0;   // never 4 with more than 32 rows: q <= most
    const size_t x_bytes = (size_t)(q + (rem > 0)) * tile, sum_bytes = (size_t)kLmKeptWaves * ((hb + 1) / 2) * 1024;
    return {hb, depth, phases, q, rem, x_bytes > sum_bytes ? x_bytes : sum_bytes};
}
static LmPlan lm_plan(int M, int tiles, int K)
{
    const int knob = params().lm_tiles;
    if (knob > 0 && knob != 1 && knob != 2 && !(knob == 4 && M > 16)) return {false, 0, 0};   // not compiled
    if (knob == 0 && K <= kLmSharedMaxK && (tiles + 3) / 4 <= (M > 16 ? 160 : M > 4 ? 256 : 64)) {
        const LmKept walk = lm_kept(M, K);
        if (walk.depth > 0 && (M > 4 || walk.depth == 4)) return {false, 4, 1, true};
    }
    if (M <= 16) return {false, 4, knob > 0 ? knob : (M <= 4 ? 1 : 2)};
    if (K > kLmSharedMaxK) return {false, 4, 4};
    if (knob > 0) return {true, 8, knob};
    static const struct { int t, penalty; } kChoices[] = {{32, 100}, {16, 110}, {8, 117}, {4, 117}};   // penalty in percent
    const int most = K <= 1024 ? 8 : 32;
    int best_t = 0;
    long long best_cost = 0;
    for (const auto &ch : kChoices) {
        if (ch.t > most) continue;
        const long long rounds = ((tiles + ch.t - 1) / ch.t + 255) / 256, cost = rounds * ch.t * ch.penalty;
        if (best_t == 0 || cost < best_cost) best_t = ch.t, best_cost = cost;
    }
    const bool one_channel = (K & (K - 1)) == 0 && best_t == 16 && (M <= 32 || K <= 2048);
    const bool short_walk = tiles > 2048 && ((M <= 32 && K <= 2048) || (M <= 48 && K <= 1024));
    if (one_channel || short_walk) return {false, 4, 4};
    return best_t == 4 ? LmPlan{true, 4, 1} : LmPlan{true, 8, best_t / 8};
}

static int lm_chunks(int V) { return (V + kLmChunk - 1) / kLmChunk; }
constexpr int kLmMaxChunks = 512, kLmMaxCandidates = 8192;   // chunks, chunks * top_k: the sizes that are served

// Least accepted workspace.  It always holds the statistics of the chunks.
static size_t lm_least_bytes(int M, int V, int top_k)
{
    const size_t slots = (size_t)M * lm_chunks(V);
    return slots * 2 * sizeof(float) + slots * top_k * (sizeof(float) + sizeof(int)) + 256;
}

static int check_lm_head(int M, int V, int K, int top_k)
{
    if (M < 1 || V < 1 || K < 1 || top_k < 1 || top_k > V) return W4A16_EINVAL;
    if (K % kLmStepK != 0) return W4A16_EINVAL;
    if (M > W4A16_MAX_M || top_k > kLmMaxTopK) return W4A16_EUNSUP;
    if (lm_chunks(V) > kLmMaxChunks || (long long)lm_chunks(V) * top_k > kLmMaxCandidates) return W4A16_EUNSUP;
    return W4A16_OK;
}

}  // namespace w4

using namespace w4;

extern "C" {

size_t lm_head_packed_bytes(int V, int K)
{
    if (V < 1 || K < 1 || K % kLmStepK != 0) return 0;
    return (size_t)((V + 15) / 16) * 16 * K * sizeof(_Float16);
}

int lm_head_pack(const void *W, void *packed, int V, int K, void *stream)
{
    if (V < 1 || K < 1 || K % kLmStepK != 0) return W4A16_EINVAL;
    if (!W || !packed) return W4A16_ENULL;
    if (misaligned(W) || misaligned(packed)) return W4A16_EALIGN;
    const long long total = (long long)((V + 15) / 16) * (K / 32) * 64;
    hipLaunchKernelGGL(lm_head_pack_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       (const _Float16 *)W, (u32x4 *)packed, V, K, total);
    return launch_status();
}

size_t lm_head_workspace_bytes(int M, int V, int K, int top_k)
{
    if (check_lm_head(M, V, K, top_k) != W4A16_OK) return 0;
    const size_t least = lm_least_bytes(M, V, top_k), finest = (size_t)M * ((V + 63) / 64) * sizeof(LmStat);   // the smallest granules
    return finest > least ? finest : least;
}

int lm_head_plan_describe(int M, int V, int K, int *out)
{
    if (!out) return W4A16_ENULL;
    const int rc = check_lm_head(M, V, K, 1);
    if (rc != W4A16_OK) return rc;
    const LmPlan plan = lm_plan(M, (V + 15) / 16, K);
    if (plan.nw == 0) return W4A16_EUNSUP;
    out[0] = plan.shared || plan.kept;
    out[1] = plan.kept ? kLmKeptWaves : plan.nw;
    out[2] = plan.twl;
    return W4A16_OK;
}

int lm_head_topk(const void *x, const void *packed, int M, int V, int K, int top_k, float *logits, int32_t *top_idx,
                 float *top_logprob, void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_lm_head(M, V, K, top_k);
    if (rc != W4A16_OK) return rc;
    if (!x || !packed || !logits || !top_idx || !top_logprob) return W4A16_ENULL;
    if (misaligned(x) || misaligned(packed) || misaligned(logits) || misaligned(workspace)) return W4A16_EALIGN;
    if ((reinterpret_cast<uintptr_t>(top_idx) | reinterpret_cast<uintptr_t>(top_logprob)) & 3u) return W4A16_EALIGN;
    if (!workspace || workspace_bytes < lm_least_bytes(M, V, top_k)) return W4A16_EWORKSPACE;
    const int tiles = (V + 15) / 16;
    hipStream_t s = (hipStream_t)stream;
    const int mtl = (M + 15) / 16;
    const LmPlan plan = lm_plan(M, tiles, K);
    if (plan.nw == 0) return W4A16_EUNSUP;
    const dim3 grid((unsigned)((tiles + plan.nw * plan.twl - 1) / (plan.nw * plan.twl)));
    // the logits kernel leaves its statistics; a workspace below the stated size may have room for coarser ones only, which then take a pass
    const bool fine = workspace_bytes >= (size_t)M * grid.x * sizeof(LmStat);
    const int granule = fine ? plan.nw * plan.twl * 16 : kLmChunk, granules = fine ? (int)grid.x : lm_chunks(V);
    LmStat *const all_stats = reinterpret_cast<LmStat *>(workspace), *const stats = fine ? all_stats : nullptr;
    if (plan.shared) {
#define W4_LM_SHARED(MTL_, NW_, TWL_, D_)                                                                               \
    if (mtl == MTL_ && plan.nw == NW_ && plan.twl == TWL_)                                                              \
        hipLaunchKernelGGL((lm_head_logits_shared_kernel<MTL_, NW_, TWL_, D_>), grid, dim3(64 * NW_), 0, s,             \
                           (const _Float16 *)x, (const u32x4 *)packed, logits, stats, M, V, K, tiles)
        W4_LM_SHARED(2, 4, 1, 4); W4_LM_SHARED(2, 8, 1, 4); W4_LM_SHARED(2, 8, 2, 2); W4_LM_SHARED(2, 8, 4, 2);
        W4_LM_SHARED(3, 4, 1, 4); W4_LM_SHARED(3, 8, 1, 4); W4_LM_SHARED(3, 8, 2, 2); W4_LM_SHARED(3, 8, 4, 2);
        W4_LM_SHARED(4, 4, 1, 4); W4_LM_SHARED(4, 8, 1, 4); W4_LM_SHARED(4, 8, 2, 2); W4_LM_SHARED(4, 8, 4, 2);
#undef W4_LM_SHARED
    } else if (plan.kept) {
        const LmKept walk = lm_kept(M, K);
        static bool lds_ok[9][2] = {};
#define W4_LM_KEPT(HB_, D_)                                                                                                                \
    if (walk.hb == HB_ && walk.depth == D_) {                                                                                              \
        static_assert(kLmKeptLds / (HB_ * 2048) >= D_ * kLmKeptSets, "a phase holds D_ steps for every set");                              \
        const auto kernel = &lm_head_logits_kept_kernel<HB_, D_>;                                                                          \
        bool &ok = lds_ok[HB_][D_ == 4];                                                                                                   \
        if (!ok && walk.lds > 48 * 1024) {                                                                                                 \
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, kLmKeptLds) != hipSuccess) \
                return W4A16_EHIP;                                                                                                         \
            ok = true;                                                                                                                     \
        }                                                                                                                                  \
        hipLaunchKernelGGL(kernel, grid, dim3(64 * kLmKeptWaves), walk.lds, s, (const _Float16 *)x, (const u32x4 *)packed, logits, stats,  \
                           M, V, K, tiles, walk.phases, walk.q, walk.rem);                                                                 \
    }
        W4_LM_KEPT(1, 2) W4_LM_KEPT(2, 2) W4_LM_KEPT(4, 2) W4_LM_KEPT(6, 2) W4_LM_KEPT(8, 2)
        W4_LM_KEPT(1, 4) W4_LM_KEPT(2, 4) W4_LM_KEPT(4, 4)
#undef W4_LM_KEPT
    } else {
        const int depth = mtl > 1 ? 2 : kLmDepth;
        const bool even = (K / kLmStepK) % depth == 0;
#define W4_LM_LAUNCH(TWL_, MTL_, DEPTH_)                                                                                \
    do {                                                                                                                \
        if (even)                                                                                                       \
            hipLaunchKernelGGL((lm_head_logits_kernel<true, TWL_, MTL_, DEPTH_>), grid, dim3(256), 0, s,                \
                               (const _Float16 *)x, (const u32x4 *)packed, logits, stats, M, V, K, tiles);                     \
        else                                                                                                            \
            hipLaunchKernelGGL((lm_head_logits_kernel<false, TWL_, MTL_, DEPTH_>), grid, dim3(256), 0, s,               \
                               (const _Float16 *)x, (const u32x4 *)packed, logits, stats, M, V, K, tiles);                     \
    } while (0)
        if (mtl == 1 && plan.twl == 1) W4_LM_LAUNCH(1, 1, kLmDepth);
        else if (mtl == 1) W4_LM_LAUNCH(2, 1, kLmDepth);
        else if (mtl == 2) W4_LM_LAUNCH(4, 2, 2);
        else if (mtl == 3) W4_LM_LAUNCH(4, 3, 2);
        else W4_LM_LAUNCH(4, 4, 2);
#undef W4_LM_LAUNCH
    }
    if (!fine)
        hipLaunchKernelGGL(lm_head_stats_kernel, dim3((unsigned)((granules + kLmThreads / 64 - 1) / (kLmThreads / 64)), (unsigned)M), dim3(kLmThreads), 0, s,
                           (const float *)logits, all_stats, V, granules);
#define W4_LM_MERGE(PER_)                                                                                                \
    hipLaunchKernelGGL(lm_head_merge_kernel<PER_>, dim3((unsigned)M), dim3(kLmThreads), 0, s, (const float *)logits,           \
                       (const LmStat *)all_stats, V, granules, granule, top_k, top_idx, top_logprob)
    const int per_lane = (granules + kLmThreads - 1) / kLmThreads;
    if (per_lane <= 1) W4_LM_MERGE(1);
    else if (per_lane <= 4) W4_LM_MERGE(4);
    else W4_LM_MERGE(kLmMaxPerLane);
#undef W4_LM_MERGE
    return launch_status();
}

}  // extern "C"
