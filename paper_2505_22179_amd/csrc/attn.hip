// tree_verify_attn: attention of the tree-verification pass (paper section 2.1) on gfx950.
//
// Scores are computed transposed, S^T = K . Q^T, with 16x16x32 fp16 MFMA steps over the head
// dimension, so that a lane ends up with eight scores of ONE query row: exactly the operand
// fragment the P.V product needs, with no shuffle in between.  The tree mask is applied to the
// draft keys only, softmax runs online in fp32 (base-2 exponentials), and V enters its product
// transposed (the contraction there runs over keys while V is stored with the head dimension
// contiguous).  Key ranges of different workgroups are combined in range order, by the last
// workgroup of a tile to finish or by a second small kernel, so the result does not depend on
// scheduling.  Three kernels: tree_attn_shared_kernel (eight wavefronts, K and V tiles brought to LDS once
// per workgroup and shared) for row tiles of 33 .. 64 rows, tree_attn_wave_kernel (each wavefront brings its own tiles and
// walks without barriers) for shorter ones, and the older tree_attn_kernel (every wavefront fetches its own K fragments
// and V rows), kept selectable.
#include <type_traits>

#include "internal.h"
#include "devscope.h"

namespace w4 {

typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kHeadDim = 128;
constexpr int kKeyBlock = 32;
constexpr int kRowsPad = 64;
// LDS of a workgroup of 4 * RG wavefronts with RT row tiles each: one exchange slot per wavefront
// (8 * RT accumulator quads + 2 * RT state values per lane); the slots cover the 8 KB V tiles
constexpr int attn_lds_bytes(int rt, int rg) { return 4 * rg * (8 * rt * 4 + 2 * rt) * 64 * 4; }
constexpr int kMaxSplits = 16;   // key ranges per row tile of the plain plan
constexpr int kMaxRanges = 32;   // of any plan (the merge keeps one value per range in registers)
constexpr int kChipTiles = 256;  // tiles x ranges of the plans that are picked by predicted time: one workgroup per compute unit

// v_max3_f32 and v_max_f32 as they stand: fmaxf chains are compiled with a canonicalising v_max x, x per
// operand, which doubles the instruction count of a row maximum; no score here is a NaN.
// The compiler adds no wait states before inline assembly: results of matrix instructions pass through settled() first.
__device__ __forceinline__ float max_of_three(float a, float b, float c)
{
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

__device__ __forceinline__ float max_of_two(float a, float b)
{
    float d;
    asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
    return d;
}

// Wait states until results of matrix instructions that were just issued may be read: passes + 4, that is eight after a 16x16x32 step and twelve
// after a 32x32x16 one.  settled<N>() adds N of them and keeps reads of its operands behind it; the steps and other
// instructions in between make up the rest, on every path from the products to the first read.
template <int N>
__device__ __forceinline__ void settled(float4v &a, float4v &b)
{
    static_assert(N >= 0 && N <= 8, "one s_nop");
    if constexpr (N == 0) asm volatile("" : "+v"(a), "+v"(b));
    else asm volatile("s_nop %2" : "+v"(a), "+v"(b) : "n"(N - 1));
}
__device__ __forceinline__ void settled(float16v &a) { asm volatile("s_nop 7\n\ts_nop 3" : "+v"(a)); }

// Maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48 (the lanes that share a query row), returned to
// all four.  v_permlane16_swap exchanges the odd 16-lane rows of its first operand with the even rows of
// its second, v_permlane32_swap the upper half of the first with the lower half of the second; applied
// to two copies of a value each leaves the two partners of a pair side by side in the two registers.
// They run on the vector ALU: no LDS round trip as with a cross-lane shuffle.  (Written in assembly:
// the compiler's builtin folded the maximum of the two results into one of them.)
__device__ __forceinline__ float row_group_max(float v)
{
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane16_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    a = max_of_two(a, b);
    b = a;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return max_of_two(a, b);
}

// maximum over the lanes l and l ^ 32, returned to both
__device__ __forceinline__ float half_wave_max(float v)
{
    float a = v, b = v;
    asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
    return max_of_two(a, b);
}

constexpr float kLowest = -1.0e30f;   // "no key seen yet": finite, so differences of two of them are 0, not NaN

// The rows of a row tile.  The group * M (head, query row) pairs that share a KV head, head by head, are cut into
// tiles_per_kv tiles of tile_rows rows (the last may have fewer): M for one query head per tile, d * M for d heads, or any
// other number up to 64, where a tile ends inside a head.  Row rho of tile `unit` is pair first + rho of its KV head.
struct RowTile {
    int kvh, group, M, Hq;
    int first;    // pair of tile row 0
    int rows;     // valid rows
    int index;    // number of the tile in its KV head
    bool whole;   // one query head per tile: no division
    __device__ __forceinline__ RowTile(int kvh_, int index_, int M_, int Hq_, int group_, int tile_rows)
    {
        M = M_;
        Hq = Hq_;
        group = group_;
        kvh = kvh_;
        index = index_;
        first = index * tile_rows;
        rows = min(tile_rows, group * M - first);
        whole = tile_rows == M;
    }
    // query row and head of a tile row; rows beyond the last repeat it (and are never stored)
    __device__ __forceinline__ void locate(int rho, int &qrow, int &head) const
    {
        const int pair = first + min(rho, rows - 1);
        const int j = whole ? index : pair / M;
        qrow = pair - j * M;
        head = kvh * group + j;
    }
};

// The row tile and the key range of a workgroup.  Workgroups go to the eight XCDs in turn; numbered so that each XCD gets a run of
// consecutive numbers, and the tiles of one KV head and one range next to each other, an XCD reads few keys, and its L2 brings them
// in once for all their tiles.  Any grid, each pair once.  Before, a grid that eight does not divide kept the order of launch, and its XCDs all read all keys; and
// the ranges of a tile stood together, so that with fewer KV heads than XCDs each XCD read most keys of a head.  us: 28/4 heads, M = 28, prefix
// 11477 31.1 -> 18.7, M = 8, prefix 3404 14.4 -> 10.0; 24/3 heads, M = 36, prefix 21792 43.3 -> 25.6; 20/5 heads, M = 52, prefix 3695 17.7 -> 12.9.
struct Share {
    int kvh, tile, range;   // KV head, row tile in it, key range
    // by_tiles, by_ranges: divider() of tiles_per_kv and nsplit -- the divisions stand before the first address, where nothing hides them
    __device__ __forceinline__ Share(unsigned block, unsigned grid, int nsplit, int tiles_per_kv, uint32_t by_tiles, uint32_t by_ranges)
    {
        const unsigned xcd = block & 7u;
        const unsigned number = xcd * (grid >> 3) + min(xcd, grid & 7u) + (block >> 3);
        const unsigned rest = __umulhi(2 * number, by_tiles);
        tile = (int)(number - rest * (unsigned)tiles_per_kv);
        kvh = (int)__umulhi(2 * rest, by_ranges);
        range = (int)rest - kvh * nsplit;
    }
};
// n / d == umulhi(2 n, divider(d)) while n d < 2^31: the factor exceeds 2^31 / d by less than one, n times that stays below 2^31 / d
static uint32_t divider(int d) { return (uint32_t)(((1u << 31) + (unsigned)d - 1) / (unsigned)d); }

// Merge of the key ranges of one tile by the workgroup that finished last (fused mode): NS = compiled
// upper bound of the number of ranges, IT = items a thread handles at once (all their loads are issued
// together).  Loads are device-scope: other workgroups, on other XCDs, wrote the partials in this kernel.
template <int NS, int IT>
__device__ __forceinline__ void merge_ranges(PartialBuffer unit_o, PartialBuffer unit_ml, _Float16 *__restrict__ out,
                                             int tid, int threads, const RowTile &tile, int nsplit)
{
    const int items = tile.rows * (kHeadDim / 4);   // one item = four consecutive outputs of a tile row
    const float NEG_INF = -__builtin_inff();
    for (int base = tid; base < items; base += threads * IT) {
        float ms[IT][NS], ls[IT][NS];
        float4v os[IT][NS];
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int idx = base + it * threads;
            const int trow = idx / (kHeadDim / 4), d4 = idx % (kHeadDim / 4);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                ms[it][s] = NEG_INF;
                ls[it][s] = 0.f;
                os[it][s] = (float4v){0.f, 0.f, 0.f, 0.f};
                if (s < nsplit && idx < items) {
                    ms[it][s] = load_partial_f32(unit_ml, (s * kRowsPad + trow) * 2);
                    ls[it][s] = load_partial_f32(unit_ml, (s * kRowsPad + trow) * 2 + 1);
                    os[it][s] = load_partial(unit_o, (s * kRowsPad + trow) * (kHeadDim / 4) + d4);
                }
            }
        }
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int idx = base + it * threads;
            if (idx >= items) break;
            const int trow = idx / (kHeadDim / 4), d4 = idx % (kHeadDim / 4);
            float m_all = NEG_INF;
#pragma unroll
            for (int s = 0; s < NS; ++s) m_all = fmaxf(m_all, ms[it][s]);
            float den = 0.f;
            float4v num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                float wgt = (ms[it][s] == NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(ms[it][s] - m_all);
                den += wgt * ls[it][s];
                num += wgt * os[it][s];
            }
            const float inv = 1.f / den;
            int qrow, h;
            tile.locate(trow, qrow, h);
            typedef _Float16 half4v __attribute__((ext_vector_type(4)));
            half4v hv = {(_Float16)(num[0] * inv), (_Float16)(num[1] * inv), (_Float16)(num[2] * inv), (_Float16)(num[3] * inv)};
            *reinterpret_cast<half4v *>(out + ((size_t)qrow * tile.Hq + h) * kHeadDim + d4 * 4) = hv;
        }
    }
}

__device__ __forceinline__ void merge_tile(PartialBuffer unit_o, PartialBuffer unit_ml, _Float16 *__restrict__ out, int tid,
                                           int threads, const RowTile &tile, int nsplit)
{
    if (nsplit <= 4) merge_ranges<4, 4>(unit_o, unit_ml, out, tid, threads, tile, nsplit);
    else if (nsplit <= 8) merge_ranges<8, 2>(unit_o, unit_ml, out, tid, threads, tile, nsplit);
    else if (nsplit <= 16) merge_ranges<16, 1>(unit_o, unit_ml, out, tid, threads, tile, nsplit);
    else merge_ranges<kMaxRanges, 1>(unit_o, unit_ml, out, tid, threads, tile, nsplit);
}

// One workgroup = one 64-row tile (a query head, or the heads of a KV group) x one contiguous range
// of 32-key steps.  Its 4 * RG wavefronts are RG row groups of four: the four wavefronts of a row
// group split the KEYS -- wavefront kw takes steps kw, kw + 4, ... of the range -- and each carries,
// for the RT * 16 rows of its group, its own online-softmax state -- running maximum, running sum and an
// unnormalised output tile -- so K and V rows are fetched once per workgroup (no wavefront re-reads
// another's keys), the main loop has no workgroup barrier, and the four states meet once, at the
// end, through LDS.  RT = 4, RG = 1: one wavefront per SIMD holds all 64 rows.  RT = 2, RG = 2: two
// wavefronts per SIMD with 32 rows each (half the accumulator and Q registers, K/V fragments fetched
// twice from L2): one wavefront's dependent softmax chain hides behind the other's matrix work.
// RT = 2, RG = 1: tiles of at most 32 rows; two such workgroups fit a compute unit.
//
// Per step a lane's registers hold, for row tile rt (rows 16 rt + c) and lane (r, c):
//   S^T = K . Q^T     sa[rt][i], sb[rt][i]: keys 4r + i of the step's two 16-key tiles, row 16 rt + c
//                     -- eight scores of ONE query row, which after exp2 and fp16 rounding are, as they
//                     stand, the second operand P^T of the next product (contraction slot 8r + p:
//                     p < 4 the first tile's key 4r + p, p >= 4 the second tile's key 4r + p - 4)
//   O^T += V^T . P^T  o[dt][rt][i]: head-dim element 16 dt + 4r + i of row 16 rt + c: the row index
//                     is the lane's c again, so the rescale factor of a row is lane-local
// V^T (first operand: head-dim element 16 dt + c, the eight keys of contraction slots 8r ..) comes
// from a per-wavefront LDS tile vt[d][32 keys in slot order], written as 8-byte units of four keys
// and read as one 16-byte load per dt; 16-byte chunks are XOR-swizzled by bits of d against bank
// conflicts.  The same wavefront writes and reads the tile: LDS keeps its program order.
template <int RT, int RG>
__global__ __launch_bounds__(256 * RG) void tree_attn_kernel(
    const _Float16 *__restrict__ q, const _Float16 *__restrict__ k, const _Float16 *__restrict__ v,
    const uint8_t *__restrict__ mask, _Float16 *__restrict__ out, float *__restrict__ part_o,
    float *__restrict__ part_ml, uint32_t *__restrict__ tickets, int M, int P, int Hq, int Hkv,
    int group, float scale_log2e, int nsplit, int bq, int brem, int tile_rows, int tiles_per_kv, int fused)
{
    extern __shared__ float4v smem4[];
    // one batch of scalar loads instead of three dependent ones before the first K/V request goes out
    const unsigned grid = gridDim.x;
    fetch_arguments_together(q, k, v, mask, out, part_o, part_ml, tickets, M, P, Hq, Hkv, group, scale_log2e, nsplit, bq, brem, tile_rows,
                             tiles_per_kv, fused, grid);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave & 3, rg = wave >> 2;   // key wavefront inside the row group, row group
    const int r = lane >> 4, c = lane & 15;
    // Workgroups are dealt to the eight XCDs round-robin by index, and each XCD has its own L2.
    // Renumber so that the workgroups of one KV head (consecutive logical ids) share an XCD and
    // its K/V rows are fetched into one L2 instead of all eight.
    int lid = blockIdx.x;
    if ((grid & 7) == 0) lid = (blockIdx.x & 7) * (grid >> 3) + (blockIdx.x >> 3);
    // Tiles that hold the rows of several query heads of a KV group read K and V once for all of them.
    const int unit = lid / nsplit, sp = lid % nsplit;
    const RowTile tile(unit / tiles_per_kv, unit % tiles_per_kv, M, Hq, group, tile_rows);
    const int kvh = tile.kvh, R = tile.rows;
    const int T = P + M;
    // key steps of this split: bq = nblk / nsplit each, the first brem = nblk % nsplit one more (host-computed)
    const int b0 = sp * bq + (sp < brem ? sp : brem), b1 = b0 + bq + (sp < brem ? 1 : 0);
    const size_t kv_stride = (size_t)Hkv * kHeadDim;

    int row[RT], head[RT];   // query row and head of tile row 16 (rg RT + rt) + c; tile rows >= R repeat row R-1 and are never stored
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) tile.locate((rg * RT + rt) * 16 + c, row[rt], head[rt]);
    // Tree mask as one 64-bit word per query row (bit j = draft key j visible), built once by the
    // workgroups whose key range reaches the draft keys: a byte load per key inside the step loop
    // would put some thirty dependent memory round trips on the critical path of the last steps.
    __shared__ uint64_t row_bits[kRowsPad];
    uint64_t mbits[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) mbits[rt] = 0;
    const bool reaches_draft = b1 * kKeyBlock > P;   // uniform over the workgroup
    // Requested first and used after the Q, K and V requests: the oldest loads.  Every lane loads from a
    // clamped, valid address and discards what lies outside the mask afterwards: a load under a per-lane
    // condition would be compiled as a branch with its own wait, sixteen memory round trips in a row.
    uint8_t mask_byte[16];
    const int mcol = min(lane, M - 1);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int mrow = min((wave & 3) * 16 + i, M - 1);   // wavefronts 0..3 cover the 64 rows
        mask_byte[i] = mask[(size_t)mrow * M + mcol];
    }
    // Q^T fragments (second operand of S^T): lane (r, c) holds q[row, h, 32 j + 8 r .. +7]
    half8v qf[RT][4];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            qf[rt][j] = *reinterpret_cast<const half8v *>(q + ((size_t)row[rt] * Hq + head[rt]) * kHeadDim + 32 * j + 8 * r);

    float4v o[8][RT];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) o[dt][rt] = (float4v){0.f, 0.f, 0.f, 0.f};
    float m_run[RT], l_run[RT];   // l_run: this lane's share (its keys 4r + i) of the row's sum
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        m_run[rt] = kLowest;
        l_run[rt] = 0.f;
    }

    // this wavefront's transposed V tile: 128 rows (d) x 64 B (32 keys in contraction-slot order)
    uint8_t *vt = reinterpret_cast<uint8_t *>(smem4) + wave * (kHeadDim * 64);
    const _Float16 *kbase = k + (size_t)kvh * kHeadDim + 8 * r;
    // V staging: lane (g, ch) = (lane % 8, lane / 8) fetches keys 4g .. 4g+3 of the step, head-dim
    // chunks ch and ch + 8 (eight elements each); key group g sits in 8-byte unit 2 (g % 4) + g / 4
    const int vg = lane & 7, vch = lane >> 3;
    const _Float16 *vbase = v + (size_t)kvh * kHeadDim + vch * 8;
    auto load_k = [&](int step, half8v (&fa)[4], half8v (&fb)[4]) {
        const int key0 = step * kKeyBlock;
        const int ra = key0 + c, rb = key0 + 16 + c;
        const bool ragged = key0 + kKeyBlock > T;   // uniform: only the last step
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            fa[j] = *reinterpret_cast<const half8v *>(kbase + (size_t)(ragged ? min(ra, T - 1) : ra) * kv_stride + 32 * j);
            fb[j] = *reinterpret_cast<const half8v *>(kbase + (size_t)(ragged ? min(rb, T - 1) : rb) * kv_stride + 32 * j);
        }
    };
    auto load_v = [&](int step, u32x4 (&vr)[2][4]) {
        const int key0 = step * kKeyBlock;
        const int rv = key0 + 4 * vg;
        const bool ragged = key0 + kKeyBlock > T;
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                vr[it][kk] = *reinterpret_cast<const u32x4 *>(vbase + (size_t)(ragged ? min(rv + kk, T - 1) : rv + kk) * kv_stride + it * 64);
    };
    auto park_v = [&](const u32x4 (&vr)[2][4]) {
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int dd = 0; dd < 8; ++dd) {
                const uint32_t sel = (dd & 1) ? 0x07060302u : 0x05040100u;   // the odd or the even halves of two words
                u32x2 unit;
                unit[0] = __builtin_amdgcn_perm(vr[it][1][dd >> 1], vr[it][0][dd >> 1], sel);
                unit[1] = __builtin_amdgcn_perm(vr[it][3][dd >> 1], vr[it][2][dd >> 1], sel);
                const int d = (vch + 8 * it) * 8 + dd;
                const int chunk = (vg & 3) ^ ((d >> 1) & 3) ^ ((d >> 3) & 3);
                *reinterpret_cast<u32x2 *>(vt + d * 64 + chunk * 16 + (vg >> 2) * 8) = unit;
            }
    };
    // One 32-key step.  The K fragments and the V rows of the wavefront's next step are requested
    // into the very registers this step has just emptied (V after its rows are parked in LDS, K after
    // the score products), so one register set each gives a prefetch distance of most of a step.
    auto step_fn = [&](int step, bool more, half8v (&fa)[4], half8v (&fb)[4], u32x4 (&vr)[2][4]) {
        const int key0 = step * kKeyBlock, next = step + 4;
        park_v(vr);
        if (more) load_v(next, vr);
        __builtin_amdgcn_sched_barrier(0);
        float4v sa[RT], sb[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            sa[rt] = (float4v){0.f, 0.f, 0.f, 0.f};
            sb[rt] = (float4v){0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                sa[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[j], qf[rt][j], sa[rt], 0, 0, 0);
                sb[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[j], qf[rt][j], sb[rt], 0, 0, 0);
            }
        if (more) load_k(next, fa, fb);
        __builtin_amdgcn_sched_barrier(0);
        half8v pb[RT];
        const bool prefix_only = key0 + kKeyBlock <= P;   // uniform: committed keys, all visible
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            float s[8];
            if (prefix_only) {
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] = ((i < 4) ? sa[rt][i & 3] : sb[rt][i & 3]) * scale_log2e;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int key = key0 + 4 * r + (i & 3) + (i >> 2) * 16;
                    const int j = key - P;   // draft key index; bits at and beyond M are clear
                    const bool vis = j < 0 || (j < 64 && ((mbits[rt] >> j) & 1));
                    const float raw = (i < 4) ? sa[rt][i & 3] : sb[rt][i & 3];
                    s[i] = vis ? raw * scale_log2e : -__builtin_inff();
                }
            }
            float m_blk = s[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) m_blk = fmaxf(m_blk, s[i]);
            m_blk = row_group_max(m_blk);
            const float m_new = fmaxf(m_run[rt], m_blk);
            const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - m_new);
            float psum = 0.f;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float pv = __builtin_amdgcn_exp2f(s[i] - m_new);
                psum += pv;
                pb[rt][i] = (_Float16)pv;
            }
            l_run[rt] = l_run[rt] * alpha + psum;
            m_run[rt] = m_new;
            if (__any(alpha != 1.0f)) {   // after the first steps a row's maximum rarely moves
#pragma unroll
                for (int dt = 0; dt < 8; ++dt) o[dt][rt] *= alpha;
            }
        }
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            const int d = dt * 16 + c;
            const int chunk = r ^ ((d >> 1) & 3) ^ ((d >> 3) & 3);
            const half8v va = *reinterpret_cast<const half8v *>(vt + d * 64 + chunk * 16);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, pb[rt], o[dt][rt], 0, 0, 0);
        }
    };

    half8v ka[4], kb[4];
    u32x4 vr[2][4];
    const int first = b0 + kw;
    if (first < b1) {
        load_k(first, ka, kb);
        load_v(first, vr);
    }
    if (reaches_draft) {
        uint64_t mine = 0;   // lane i keeps the word of row 16 wave + i: one LDS write per wavefront instead of sixteen
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint64_t bits = __ballot(mask_byte[i] != 0 && wave * 16 + i < M && lane < M);
            mine = lane == i ? bits : mine;
        }
        if (lane < 16 && wave < 4) row_bits[wave * 16 + lane] = mine;
        __syncthreads();
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) mbits[rt] = row_bits[row[rt]];
    }
    for (int step = first; step < b1; step += 4)
        step_fn(step, step + 4 < b1, ka, kb, vr);

    // a row's sum over this wavefront's keys: add the four lanes (r = 0..3) that share the row
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        l_run[rt] += __shfl_xor(l_run[rt], 16, 64);
        l_run[rt] += __shfl_xor(l_run[rt], 32, 64);
    }
    // The wavefronts' states meet in LDS: each parks its whole state (8 * RT accumulator quads and
    // 2 * RT state values per lane, lane-contiguous), and after one barrier wavefront (rg, kw) combines, in
    // wavefront order, the head-dim tiles 2 kw and 2 kw + 1 of the four key wavefronts of its row group.
    constexpr int kQuads = 8 * RT;
    float4v *xq = smem4;                                                             // [slots][8 RT quads][64 lanes]
    float *xs = reinterpret_cast<float *>(smem4 + 4 * RG * kQuads * 64);             // [slots][2 RT values][64 lanes]
    __syncthreads();   // every wavefront has left its V tile: the exchange reuses that LDS
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) xq[(wave * kQuads + dt * RT + rt) * 64 + lane] = o[dt][rt];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        xs[(wave * 2 * RT + rt) * 64 + lane] = m_run[rt];
        xs[(wave * 2 * RT + RT + rt) * 64 + lane] = l_run[rt];
    }
    __syncthreads();
    const bool last = nsplit == 1;
    float *po = part_o + (size_t)lid * kRowsPad * kHeadDim;
    float *pml = part_ml + (size_t)lid * kRowsPad * 2;
    // fused mode: the partials of a tile's key ranges are published with device-scope stores and merged by
    // the last workgroup of the tile to finish (below)
    const PartialBuffer unit_o = partial_buffer(part_o + (size_t)unit * nsplit * kRowsPad * kHeadDim);
    const PartialBuffer unit_ml = partial_buffer(part_ml + (size_t)unit * nsplit * kRowsPad * 2);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        float ms[4], wgt[4], m_all = kLowest, l_all = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            ms[w2] = xs[((rg * 4 + w2) * 2 * RT + rt) * 64 + lane];
            m_all = fmaxf(m_all, ms[w2]);
        }
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            wgt[w2] = __builtin_amdgcn_exp2f(ms[w2] - m_all);
            l_all += wgt[w2] * xs[((rg * 4 + w2) * 2 * RT + RT + rt) * 64 + lane];
        }
        const int orow = (rg * RT + rt) * 16 + c;
        const float inv = last ? 1.f / l_all : 1.f;
#pragma unroll
        for (int dd = 0; dd < 2; ++dd) {
            const int dt = 2 * kw + dd;
            float4v val = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w2 = 0; w2 < 4; ++w2) val += wgt[w2] * xq[((rg * 4 + w2) * kQuads + dt * RT + rt) * 64 + lane];
            val *= inv;
            // tile row orow, head-dim elements 16 dt + 4r .. + 3: four consecutive outputs
            if (orow < R) {
                if (last) {
                    typedef _Float16 half4v __attribute__((ext_vector_type(4)));
                    half4v hv = {(_Float16)val[0], (_Float16)val[1], (_Float16)val[2], (_Float16)val[3]};
                    *reinterpret_cast<half4v *>(out + ((size_t)row[rt] * Hq + head[rt]) * kHeadDim + dt * 16 + 4 * r) = hv;
                } else if (fused) {
                    store_partial(unit_o, (sp * kRowsPad + orow) * (kHeadDim / 4) + dt * 4 + r, val);
                } else {
                    *reinterpret_cast<float4v *>(po + orow * kHeadDim + dt * 16 + 4 * r) = val;
                }
            }
        }
        if (!last && kw == 0 && r == 0 && orow < R) {
            // partial state of this key range
            if (fused) {
                store_partial_f32(unit_ml, (sp * kRowsPad + orow) * 2, m_all);
                store_partial_f32(unit_ml, (sp * kRowsPad + orow) * 2 + 1, l_all);
            } else {   // a second kernel merges the ranges (the kernel boundary makes them visible, at no fence cost)
                pml[orow * 2] = m_all;
                pml[orow * 2 + 1] = l_all;
            }
        }
    }
    if (last || !fused) return;   // uniform over the grid
    // The workgroups of a tile take a ticket each once their partials have reached device scope; the one
    // that draws the last ticket merges the tile's key ranges, in range order, with the arithmetic of
    // tree_attn_merge_kernel, and leaves the ticket at zero for the next call.
    __shared__ uint32_t ticket_sh;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) ticket_sh = __hip_atomic_fetch_add(&tickets[unit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket_sh != (uint32_t)(nsplit - 1)) return;
    if (tid == 0) __hip_atomic_store(&tickets[unit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    merge_tile(unit_o, unit_ml, out, tid, 256 * RG, tile, nsplit);
}

// ---- Row tiles of 33..64 rows: K and V tiles shared through LDS -------------------------------------
// The kernel above lets every wavefront fetch its own K fragments and V rows from global memory.  With
// a full tile that costs twice: a K fragment load touches sixteen key rows with 64 bytes each, the
// costliest pattern for the address path of a compute unit (about four times the time of a load of
// whole cache lines), and 64 rows of accumulators and Q fragments fill the register file of a SIMD
// with one wavefront, so nothing overlaps that wavefront's softmax arithmetic, its matrix products
// and its memory waits.  Here a workgroup has eight wavefronts, two per SIMD: wavefront (kw, rh)
// holds tile rows 32 rh .. 32 rh + 31 and takes key step 4 t + kw of the workgroup's range in round t.
// All K and V tiles of a round (four steps of 32 keys, 8 KB each for K and for V) are brought in one
// round ahead by direct global -> LDS loads of whole key rows (one instruction: four rows of 256 B),
// the K tile of a step by wavefront (kw, 0) and the V tile by (kw, 1), double-buffered, one workgroup
// barrier per round.  Both wavefronts of a pair read the same tiles:
//   K fragments   one 16-byte LDS read per fragment; the 16-byte chunks of a key row are stored at
//                 chunk ^ (key % 8), the permutation being applied to the SOURCE address of the
//                 transfer (its destination is fixed: lane l of a transfer fills bytes 16 l ..)
//   V^T fragments the transposing LDS read (ds_read_b64_tr_b16): in each block of 16 lanes, lane s
//                 points at four consecutive head-dim elements 4 (s % 4) .. of key row s / 4, and
//                 lane c receives element c of the four rows -- four keys at one head-dim index,
//                 which is the operand layout, with no pass through registers.  Chunks of a V row
//                 are stored at chunk ^ (2 key % 16).
// Q reaches its fragments the same way (once, through the second round buffer).  The softmax is that
// of the kernel above with the scale folded into the exponent's multiply-add; the states of the four
// key wavefronts of a row half meet in LDS at the end, in a row-major layout (rows padded to 528 B)
// from which thread t then reads, merges and stores whole 512-byte output rows.
constexpr int kSharedWaves = 8;
constexpr int kTileBytes = kKeyBlock * kHeadDim * 2;         // one K or V tile: 32 keys x 256 B
constexpr int kStepBytes = 2 * kTileBytes;                   // K tile, then V tile
constexpr int kRoundBytes = 4 * kStepBytes;                  // the four key steps of a round
constexpr int kExRow = kHeadDim * 4 + 16;                    // exchange row: 128 fp32 + 16 B of padding
constexpr int kExWave = 32 * kExRow;                         // per wavefront: its 32 rows
constexpr int kExState = kSharedWaves * kExWave;             // then [8 wavefronts][32 rows] (max, sum)
constexpr int kSharedLds = kExState + kSharedWaves * 32 * 8 > 2 * kRoundBytes ? kExState + kSharedWaves * 32 * 8 : 2 * kRoundBytes;

typedef __attribute__((address_space(3))) void lds_void;
typedef const __attribute__((address_space(1))) void global_void;
typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v lds_short4v;

__device__ __forceinline__ uint32_t lds_address(const void *p)
{
    return (uint32_t)(size_t)(lds_void *)p;
}
// The transposing read of the rows at lds_addr and 16 key rows (4 KB) further on.  Written in assembly: through
// the builtin the compiler waits, before every such read, for ALL outstanding global -> LDS transfers -- the
// next round's, requested a moment earlier precisely so that they overlap this round's arithmetic.  The
// compiler therefore does not know of these reads; wait_lds_reads says when their results may be used.
template <int OFFSET>
__device__ __forceinline__ void read_transposed_pair(short4v &lo, short4v &hi, uint32_t lds_addr)
{
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                 : "=&v"(lo), "=&v"(hi)
                 : "v"(lds_addr), "n"(OFFSET), "n"(OFFSET + 16 * 256));
}
// returns once at most N LDS operations of this wavefront (the N most recent) are still under way; lo and hi are the
// oldest pair still awaited, so that no use of it, not even a copy, can be moved above the wait
template <int N>
__device__ __forceinline__ void wait_lds_reads(short4v &lo, short4v &hi)
{
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(lo), "+v"(hi) : "n"(N));
}
// lane l's 16 bytes at src land at lds_base + 16 l (lds_base wavefront-uniform); counted by vmcnt
__device__ __forceinline__ void row_to_lds(const uint8_t *src, uint8_t *lds_base)
{
    __builtin_amdgcn_global_load_lds((global_void *)src, (lds_void *)lds_base, 16, 0, 0);
}

// (The arguments fill two lines of the scalar cache, here and in the next kernel.  A third, for gridDim, costs every call 0.06 us.)
__global__ __launch_bounds__(64 * kSharedWaves) void tree_attn_shared_kernel(
    uint32_t by_tiles, uint32_t by_ranges, const _Float16 *__restrict__ q, const _Float16 *__restrict__ k, const _Float16 *__restrict__ v,
    const uint8_t *__restrict__ mask, _Float16 *__restrict__ out, float *__restrict__ part_o,
    float *__restrict__ part_ml, uint32_t *__restrict__ tickets, int M, int P, int Hq, int Hkv,
    int group, float scale_log2e, int nsplit, int bq, int brem, int tile_rows, int tiles_per_kv, int fused)
{
    extern __shared__ float4v smem4[];
    uint8_t *lds = reinterpret_cast<uint8_t *>(smem4);
    fetch_arguments_together(by_tiles, by_ranges, q, k, v, mask, out, part_o, part_ml, tickets, M, P, Hq, Hkv, group, scale_log2e, nsplit, bq, brem, tile_rows,
                             tiles_per_kv, fused);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = wave >> 1, rh = wave & 1;   // key wavefront, row half
    const int r = lane >> 4, c = lane & 15;
    const Share share(blockIdx.x, (unsigned)(Hkv * tiles_per_kv * nsplit), nsplit, tiles_per_kv, by_tiles, by_ranges);
    const int kvh = share.kvh, unit = kvh * tiles_per_kv + share.tile, sp = share.range;
    const RowTile tile(kvh, share.tile, M, Hq, group, tile_rows);
    const int R = tile.rows;
    const int T = P + M;
    const int b0 = sp * bq + (sp < brem ? sp : brem), b1 = b0 + bq + (sp < brem ? 1 : 0);
    const int rounds = (b1 - b0 + 3) >> 2;
    const size_t kv_row_bytes = (size_t)Hkv * kHeadDim * 2;

    // tile row -> its query row and the element offset of its (query row, head) in q and out
    auto locate = [&](int rho, int &qrow) {
        int head;
        tile.locate(rho, qrow, head);
        return (uint32_t)(qrow * Hq + head) * kHeadDim;
    };
    // tree mask of the draft keys, one 64-bit word per query row, in the workgroups that reach them:
    // wavefront w asks for the bytes of rows 8 w .. 8 w + 7 first (lane = column) and turns them into words
    // after the transfers below have been requested
    __shared__ uint64_t row_bits[kRowsPad];
    const bool reaches_draft = b1 * kKeyBlock > P;   // uniform over the workgroup
    uint32_t mask_byte[8] = {};
    if (reaches_draft) {
        const int mcol = min(lane, M - 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) mask_byte[i] = mask[(size_t)min(wave * 8 + i, M - 1) * M + mcol];
    }

    // transfers: lane l of transfer i fills bytes 16 (l % 16) .. of tile row 4 i + l / 16
    const int trow = lane >> 4, tchunk = lane & 15;
    // LDS: per key wavefront pair 32 KB = two buffers of (K tile, V tile); Q sits in pair 0's second buffer until
    // that pair requests the tiles of its second round
    uint8_t *const pair_lds = lds + kw * (2 * kStepBytes);
    uint8_t *const qtile = lds + kStepBytes;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int rho = 4 * (2 * wave + u) + trow;
        int qrow;
        const uint32_t elem = locate(rho, qrow);
        row_to_lds(reinterpret_cast<const uint8_t *>(q) + (size_t)elem * 2 + ((tchunk ^ (rho & 7)) << 4), qtile + (2 * wave + u) * 1024);
    }
    // K (rh = 0) or V (rh = 1) rows of this wavefront's key steps.  Tile row 4 i + trow goes to chunk positions
    // permuted by key % 8 (K) or 2 key % 16 (V), which depends on i through its parity only: two lane offsets,
    // added to a wavefront-uniform address that moves with the step and with i.
    const uint8_t *const kv_src = reinterpret_cast<const uint8_t *>(rh ? v : k) + (size_t)kvh * kHeadDim * 2;
    uint32_t lane_src[2];
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int key = 4 * par + trow;
        lane_src[par] = (uint32_t)trow * (uint32_t)kv_row_bytes + (uint32_t)((tchunk ^ (rh ? (2 * key) & 15 : key & 7)) << 4);
    }
    auto request_round = [&](int t, int buf) {
        const int step = b0 + 4 * t + kw;
        if (step >= b1) return;   // uniform over the wavefront
        const int key0 = step * kKeyBlock;
        uint8_t *dst = pair_lds + buf * kStepBytes + rh * kTileBytes;
        if (key0 + kKeyBlock <= T) {
            const uint8_t *from = kv_src + (size_t)key0 * kv_row_bytes;
#pragma unroll
            for (int i = 0; i < 8; ++i) row_to_lds(from + (size_t)(4 * i) * kv_row_bytes + lane_src[i & 1], dst + i * 1024);
        } else {   // the last step of all: rows beyond the last key repeat it (they are masked out below)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int key = 4 * i + trow;
                const int swz = rh ? (2 * key) & 15 : key & 7;
                row_to_lds(kv_src + (size_t)min(key0 + key, T - 1) * kv_row_bytes + ((tchunk ^ swz) << 4), dst + i * 1024);
            }
        }
    };
    request_round(0, 0);

    if (reaches_draft) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            asm volatile("" : "+v"(mask_byte[i]));   // keeps the comparison, and with it the wait for the byte, from being done before the transfers
            const uint64_t bits = __ballot(mask_byte[i] != 0 && wave * 8 + i < M && lane < M);
            if (lane == i) row_bits[wave * 8 + i] = bits;
        }
    }
    // Q fragments (second operand of S^T): lane (r, c) holds elements 32 j + 8 r .. + 7 of tile row 32 rh + 16 rt + c
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    half8v qf[2][4];
    uint64_t mbits[2] = {0, 0};
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
        const int rho = 32 * rh + 16 * rt + c;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            qf[rt][j] = *reinterpret_cast<const half8v *>(qtile + rho * 256 + (((4 * j + r) ^ (rho & 7)) << 4));
        int qrow;
        locate(rho, qrow);
        if (reaches_draft) mbits[rt] = row_bits[qrow];
    }

    float4v o[8][2];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) o[dt][rt] = (float4v){0.f, 0.f, 0.f, 0.f};
    float m_run[2] = {kLowest, kLowest}, l_run[2] = {0.f, 0.f};   // l_run: this lane's share (its keys) of the row's sum

    // fragment addresses inside the pair's first buffer (the second lies kStepBytes further on: an immediate offset)
    const uint8_t *kfrag[4];   // K: key c (and 16 + c: + 4 KB), chunk (4 j + r) ^ (c % 8)
#pragma unroll
    for (int j = 0; j < 4; ++j) kfrag[j] = pair_lds + ((c * 256 + ((r ^ (c & 7)) << 4)) ^ (j << 6));
    // V: lane c of block r points at key row 4 r + c / 4 (and 16 + that: + 4 KB), elements 16 dt + 4 (c % 4) ..
    const int vkey = 4 * r + (c >> 2);
    const int voff = vkey * 256 + (((((c >> 1) & 1)) ^ ((2 * vkey) & 15)) << 4) + (c & 1) * 8;
    uint32_t vfrag[8];
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) vfrag[dt] = lds_address(pair_lds + kTileBytes) + (voff ^ (dt << 5));

    // one round, on buffer BUF of the pair (the loop below alternates them, so that BUF is a compile-time offset)
    auto round = [&](auto buf_tag, int t) {
        constexpr int BUF = decltype(buf_tag)::value;
        // this wavefront's transfers of round t have landed; after the barrier everybody's have, and nobody
        // still reads the other buffer
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __syncthreads();
        if (t + 1 < rounds) request_round(t + 1, BUF ^ 1);
        const int step = b0 + 4 * t + kw;
        const bool active = step < b1;   // uniform over the wavefront; the barriers are outside these branches
        const int key0 = step * kKeyBlock;
        half8v pb[2];
        if (active) {
            float4v sa[2], sb[2];
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                sa[rt] = (float4v){0.f, 0.f, 0.f, 0.f};
                sb[rt] = (float4v){0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const half8v fa = *reinterpret_cast<const half8v *>(kfrag[j] + BUF * kStepBytes);
                const half8v fb = *reinterpret_cast<const half8v *>(kfrag[j] + BUF * kStepBytes + 16 * 256);
#pragma unroll
                for (int rt = 0; rt < 2; ++rt) {
                    sa[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa, qf[rt][j], sa[rt], 0, 0, 0);
                    sb[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb, qf[rt][j], sb[rt], 0, 0, 0);
                }
            }
            const bool prefix_only = key0 + kKeyBlock <= P;   // uniform: committed keys, all visible
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) {
                if (rt == 0) settled<6>(sa[0], sb[0]);   // two more steps were issued after theirs
                else settled<0>(sa[1], sb[1]);           // the first row tile's maximum lies in between
                float s[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] = (i < 4) ? sa[rt][i & 3] : sb[rt][i & 3];
                if (!prefix_only) {
                    // visibility of the step's 32 keys as one word: the step's first key is draft key `first`
                    // (-31 .. 63; negative: the step begins with committed keys, all visible); mask bits at and
                    // beyond M are clear, so keys past the last one are hidden
                    const int first = key0 - P;
                    const uint64_t window = first >= 0 ? mbits[rt] >> first : (mbits[rt] << -first) | ((1ull << -first) - 1);
                    const uint32_t mine = (uint32_t)window >> (4 * r);   // bit i: key 4 r + i; bit 16 + i: key 16 + 4 r + i
#pragma unroll
                    for (int i = 0; i < 8; ++i) s[i] = ((mine >> ((i & 3) + 16 * (i >> 2))) & 1u) ? s[i] : -__builtin_inff();
                }
                // the scale is positive (checked by the host): the largest raw score is the largest scaled one
                const float m_blk = row_group_max(max_of_three(max_of_three(s[0], s[1], s[2]), max_of_three(s[3], s[4], s[5]), max_of_two(s[6], s[7])));
                const float m_new = max_of_two(m_run[rt], m_blk * scale_log2e);
                const float alpha = __builtin_amdgcn_exp2f(m_run[rt] - m_new);
                float pv[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    pv[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], scale_log2e, -m_new));
                    pb[rt][i] = (_Float16)pv[i];
                }
                const float psum = ((pv[0] + pv[1]) + (pv[2] + pv[3])) + ((pv[4] + pv[5]) + (pv[6] + pv[7]));
                l_run[rt] = l_run[rt] * alpha + psum;
                m_run[rt] = m_new;
                if (__any(alpha != 1.0f)) {   // after the first steps a row's maximum rarely moves
#pragma unroll
                    for (int dt = 0; dt < 8; ++dt) o[dt][rt] *= alpha;
                }
            }
        }
        if (!active) return;
        // V^T fragments, two head-dim tiles ahead of the products that use them: contraction slots 8 r .. 8 r + 3
        // are keys 4 r .. of the step's first 16, slots 8 r + 4 .. those of its second 16
        short4v lo[8], hi[8];
        read_transposed_pair<BUF * kStepBytes>(lo[0], hi[0], vfrag[0]);
        read_transposed_pair<BUF * kStepBytes>(lo[1], hi[1], vfrag[1]);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            if (dt + 2 < 8) read_transposed_pair<BUF * kStepBytes>(lo[dt + 2], hi[dt + 2], vfrag[dt + 2]);
            if (dt + 2 < 8)
                wait_lds_reads<4>(lo[dt], hi[dt]);
            else if (dt + 1 < 8)
                wait_lds_reads<2>(lo[dt], hi[dt]);
            else
                wait_lds_reads<0>(lo[dt], hi[dt]);
            typedef short short8v __attribute__((ext_vector_type(8)));
            const short8v both = __builtin_shufflevector(lo[dt], hi[dt], 0, 1, 2, 3, 4, 5, 6, 7);
            const half8v va = __builtin_bit_cast(half8v, both);
#pragma unroll
            for (int rt = 0; rt < 2; ++rt) o[dt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(va, pb[rt], o[dt][rt], 0, 0, 0);
        }
    };
    for (int t = 0; t < rounds; t += 2) {
        round(std::integral_constant<int, 0>{}, t);
        if (t + 1 < rounds) round(std::integral_constant<int, 1>{}, t + 1);
    }

    // a row's sum over this wavefront's keys: add the four lanes (r = 0..3) that share the row
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
        l_run[rt] += __shfl_xor(l_run[rt], 16, 64);
        l_run[rt] += __shfl_xor(l_run[rt], 32, 64);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __syncthreads();   // every wavefront has left the K and V tiles: the exchange reuses that LDS
    uint8_t *const mine = lds + wave * kExWave;
    float *const state = reinterpret_cast<float *>(lds + kExState);   // [wavefront][row of its half][max, sum]
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
#pragma unroll
        for (int dt = 0; dt < 8; ++dt)
            *reinterpret_cast<float4v *>(mine + (16 * rt + c) * kExRow + (4 * dt + r) * 16) = o[dt][rt];
        if (r == 0) {
            state[(wave * 32 + 16 * rt + c) * 2] = m_run[rt];
            state[(wave * 32 + 16 * rt + c) * 2 + 1] = l_run[rt];
        }
    }
    __syncthreads();
    // thread t merges, in wavefront order, the four key wavefronts' values of four consecutive outputs of a row:
    // 32 threads per row, whole rows per store
    const bool last = nsplit == 1;
    const PartialBuffer unit_o = partial_buffer(part_o + (size_t)unit * nsplit * kRowsPad * kHeadDim);
    const PartialBuffer unit_ml = partial_buffer(part_ml + (size_t)unit * nsplit * kRowsPad * 2);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
        const int item = tid + it * (64 * kSharedWaves);
        const int rho = item >> 5, quad = item & 31;   // tile row, its outputs 4 quad .. 4 quad + 3
        const int half_ = rho >> 5, hrow = rho & 31;
        float ms[4], wgt[4], m_all = kLowest, l_all = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            ms[w2] = state[((2 * w2 + half_) * 32 + hrow) * 2];
            m_all = fmaxf(m_all, ms[w2]);
        }
        float4v val = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w2 = 0; w2 < 4; ++w2) {
            wgt[w2] = __builtin_amdgcn_exp2f(ms[w2] - m_all);
            l_all += wgt[w2] * state[((2 * w2 + half_) * 32 + hrow) * 2 + 1];
            val += wgt[w2] * *reinterpret_cast<const float4v *>(lds + (2 * w2 + half_) * kExWave + hrow * kExRow + quad * 16);
        }
        if (rho >= R) continue;
        if (last) {
            val *= 1.f / l_all;
            typedef _Float16 half4v __attribute__((ext_vector_type(4)));
            half4v hv = {(_Float16)val[0], (_Float16)val[1], (_Float16)val[2], (_Float16)val[3]};
            int qrow;
            *reinterpret_cast<half4v *>(out + locate(rho, qrow) + quad * 4) = hv;
        } else {
            // written through to memory in either mode: left in the L2 as ordinary stores, the partials of the
            // two-kernel mode would all be written back at the end of the kernel, after the last workgroup
            store_partial(unit_o, (sp * kRowsPad + rho) * (kHeadDim / 4) + quad, val);
            if (quad == 0) {
                store_partial_f32(unit_ml, (sp * kRowsPad + rho) * 2, m_all);
                store_partial_f32(unit_ml, (sp * kRowsPad + rho) * 2 + 1, l_all);
            }
        }
    }
    if (last || !fused) return;   // uniform over the grid
    // last-arriver merge of the tile's key ranges, as in tree_attn_kernel
    __shared__ uint32_t ticket_sh;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) ticket_sh = __hip_atomic_fetch_add(&tickets[unit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket_sh != (uint32_t)(nsplit - 1)) return;
    if (tid == 0) __hip_atomic_store(&tickets[unit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    merge_tile(unit_o, unit_ml, out, tid, 64 * kSharedWaves, tile, nsplit);
}

// ---- Row tiles of at most 32 rows: wavefronts with K and V tiles of their own --------------------------
// With so few rows half of the wavefronts above would carry padding.  Here each of the eight wavefronts carries all 32 rows of
// the tile and takes key steps of its own, wave, wave + 8, ... of the range.  It shares no K or V tile, so it brings them itself
// (direct global -> LDS transfers into 16 KB of its own: the next step's K as soon as this step's scores are done, its V after
// the products) and meets the others only at the end: no barrier in the walk, and one wavefront's softmax runs beside another's products.
// 32x32x16 steps leave a lane with sixteen scores of ONE query row (column lane % 32; keys 8 a + 4 h + b, h = lane / 32), again the
// operand of O^T += V^T . P^T as they stand, and two lanes share a row.  Chunks of K, V and Q rows are permuted as above.
// What bounds it: at short prefixes the chain launch, first tiles, exchange, merge (5.5 us with one step); at long ones
// the transfers, 16 KB per step and 32 rows.  Against the kernel above, same split, us: prefix 2048, 64/8 heads, M = 1 9.1 -> 8.3, M = 8 11.2 -> 9.8;
// 32/8 heads, M = 30 11.8 -> 10.7; prefix 16000, 64/8 heads, M = 1 19.2 -> 17.5.  A form with 64 rows per wavefront (250 registers) lost
// to the kernel above (15.7 against 16.6 us at M = 60, prefix 2048; even at prefix 8000): the exchange doubles.
constexpr int kWaveBytes = 2 * kTileBytes;
constexpr int kWaveQ = kSharedWaves * kWaveBytes;                              // Q tile behind the K and V tiles
constexpr int kWaveState = kSharedWaves * kExWave;                             // after the walk: [row][wavefront] (max, sum) behind the exchange rows,
constexpr int kWaveRows = 32;
constexpr int kWaveWeights = kWaveState + kWaveRows * kSharedWaves * 8;        // [row][wavefront] (weight, weighted sum)
constexpr int kWaveEnd = kWaveWeights + kWaveRows * kSharedWaves * 8;
constexpr int kWaveLds = kWaveQ + kWaveRows * kHeadDim * 2 > kWaveEnd ? kWaveQ + kWaveRows * kHeadDim * 2 : kWaveEnd;
typedef float float2v __attribute__((ext_vector_type(2)));

// the transposing read of four key rows at lds_addr + OFFSET and the four that lie eight rows further on
template <int OFFSET>
__device__ __forceinline__ void read_transposed_rows(short4v &lo, short4v &hi, uint32_t lds_addr)
{
    asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                 : "=&v"(lo), "=&v"(hi)
                 : "v"(lds_addr), "n"(OFFSET), "n"(OFFSET + 8 * 256));
}

__global__ __launch_bounds__(64 * kSharedWaves) void tree_attn_wave_kernel(
    uint32_t by_tiles, uint32_t by_ranges, const _Float16 *__restrict__ q, const _Float16 *__restrict__ k, const _Float16 *__restrict__ v,
    const uint8_t *__restrict__ mask, _Float16 *__restrict__ out, float *__restrict__ part_o,
    float *__restrict__ part_ml, uint32_t *__restrict__ tickets, int M, int P, int Hq, int Hkv,
    int group, float scale_log2e, int nsplit, int bq, int brem, int tile_rows, int tiles_per_kv, int fused)
{
    extern __shared__ float4v smem4[];
    uint8_t *lds = reinterpret_cast<uint8_t *>(smem4);
    fetch_arguments_together(by_tiles, by_ranges, q, k, v, mask, out, part_o, part_ml, tickets, M, P, Hq, Hkv, group, scale_log2e, nsplit, bq, brem, tile_rows,
                             tiles_per_kv, fused);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, c = lane & 31;
    const Share share(blockIdx.x, (unsigned)(Hkv * tiles_per_kv * nsplit), nsplit, tiles_per_kv, by_tiles, by_ranges);
    const int kvh = share.kvh, unit = kvh * tiles_per_kv + share.tile, sp = share.range;
    const RowTile tile(kvh, share.tile, M, Hq, group, tile_rows);
    const int R = tile.rows;
    const int T = P + M;
    const int b0 = sp * bq + (sp < brem ? sp : brem), b1 = b0 + bq + (sp < brem ? 1 : 0);
    const size_t kv_row_bytes = (size_t)Hkv * kHeadDim * 2;
    auto locate = [&](int rho, int &qrow) {   // tile row -> its query row and the element offset of its (query row, head) in q and out
        int head;
        tile.locate(rho, qrow, head);
        return (uint32_t)(qrow * Hq + head) * kHeadDim;
    };
    // tree mask of the draft keys as in tree_attn_shared_kernel: bytes requested first, words made of them later
    __shared__ uint64_t row_bits[kRowsPad];
    const bool reaches_draft = b1 * kKeyBlock > P;   // uniform over the workgroup
    uint32_t mask_byte[8] = {};
    if (reaches_draft) {
        const int mcol = min(lane, M - 1);
#pragma unroll
        for (int i = 0; i < 8; ++i) mask_byte[i] = mask[(size_t)min(wave * 8 + i, M - 1) * M + mcol];
    }
    // transfers: lane l of transfer i fills bytes 16 (l % 16) .. of tile row 4 i + l / 16
    const int trow = lane >> 4, tchunk = lane & 15;
    uint8_t *const ktile = lds + wave * kWaveBytes, *const vtile = ktile + kTileBytes, *const qtile = lds + kWaveQ;
    {
        const int rho = 4 * wave + trow;
        int qrow;
        const uint32_t elem = locate(rho, qrow);
        row_to_lds(reinterpret_cast<const uint8_t *>(q) + (size_t)elem * 2 + ((tchunk ^ (rho & 7)) << 4), qtile + wave * 1024);
    }
    const uint8_t *const k_src = reinterpret_cast<const uint8_t *>(k) + (size_t)kvh * kHeadDim * 2;
    const uint8_t *const v_src = reinterpret_cast<const uint8_t *>(v) + (size_t)kvh * kHeadDim * 2;
    uint32_t lane_k[2], lane_v[2];   // the chunk permutation depends on the transfer's parity only
#pragma unroll
    for (int par = 0; par < 2; ++par) {
        const int key = 4 * par + trow;
        lane_k[par] = (uint32_t)trow * (uint32_t)kv_row_bytes + (uint32_t)((tchunk ^ (key & 7)) << 4);
        lane_v[par] = (uint32_t)trow * (uint32_t)kv_row_bytes + (uint32_t)((tchunk ^ ((2 * key) & 15)) << 4);
    }
    auto request = [&](int step, const uint8_t *src, const uint32_t (&lane_src)[2], int twice, uint8_t *dst) {
        const int key0 = step * kKeyBlock;
        if (key0 + kKeyBlock <= T) {   // uniform
            const uint8_t *from = src + (size_t)key0 * kv_row_bytes;
#pragma unroll
            for (int i = 0; i < 8; ++i) row_to_lds(from + (size_t)(4 * i) * kv_row_bytes + lane_src[i & 1], dst + i * 1024);
        } else {   // the last step of all: rows beyond the last key repeat it (they are masked out below)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int key = 4 * i + trow, swz = twice ? (2 * key) & 15 : key & 7;
                row_to_lds(src + (size_t)min(key0 + key, T - 1) * kv_row_bytes + ((tchunk ^ swz) << 4), dst + i * 1024);
            }
        }
    };
    int step = b0 + wave;
    __builtin_amdgcn_sched_barrier(0);   // Q before K before V: the waits below count on it
    if (step < b1) {   // uniform over the wavefront
        request(step, k_src, lane_k, 0, ktile);
        __builtin_amdgcn_sched_barrier(0);
        request(step, v_src, lane_v, 1, vtile);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (reaches_draft) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            asm volatile("" : "+v"(mask_byte[i]));   // keeps the comparison, and with it the wait for the byte, from being done before the transfers
            const uint64_t bits = __ballot(mask_byte[i] != 0 && wave * 8 + i < M && lane < M);
            if (lane == i) row_bits[wave * 8 + i] = bits;
        }
    }
    // everybody's part of the Q tile has landed (it is older than the sixteen transfers of K and V), and the mask words.  As compiled, the first step
    // waits for its V tile all the same: the compiler cannot count across these waits, so it waits for every transfer where the mask
    // bytes are used, and in all workgroups once more ahead of the loop, where the registers of those bytes are taken for the sums.
    if (step < b1) asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");

    const uint32_t frag = (uint32_t)(c * 256 + ((h ^ (c & 7)) << 4));   // fragment j of K or Q: chunk (2 j + h) ^ (row % 8)
    half8v qf[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) qf[j] = *reinterpret_cast<const half8v *>(qtile + (frag ^ (j << 5)));
    uint64_t mbits = 0;
    if (reaches_draft) {
        int qrow;
        locate(c, qrow);
        mbits = row_bits[qrow];
    }
    // V: lane s of 16-lane block b points at key row 4 (b / 2) + s / 4 (and 8 further on), elements 32 dt + 16 (b % 2) + 4 (s % 4) ..
    const int vkey = 4 * h + ((lane & 15) >> 2);
    const uint32_t vbase = lds_address(vtile), vfrag = vkey * 256 + (((2 * ((lane >> 4) & 1) + ((lane >> 1) & 1)) ^ (2 * vkey)) << 4) + 8 * (lane & 1);
    float16v o[4];
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
    float m_run = kLowest, l_run = 0.f;   // l_run: this lane's share (its keys) of the row's sum

    while (step < b1) {   // uniform over the wavefront; no barrier inside
        const int next = step + kSharedWaves, key0 = step * kKeyBlock;
        const bool more = next < b1;
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");   // K of this step; its V is newer
        float16v sc;
#pragma unroll
        for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            sc = __builtin_amdgcn_mfma_f32_32x32x16_f16(*reinterpret_cast<const half8v *>(ktile + (frag ^ (j << 5))), qf[j], sc, 0, 0, 0);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the K tile has been read
        if (more) request(next, k_src, lane_k, 0, ktile);
        settled(sc);
        half8v pb[2];
        const bool prefix_only = key0 + kKeyBlock <= P;   // uniform: committed keys, all visible
        float s[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = sc[i];   // key 8 (i / 4) + 4 h + i % 4 of the step
        if (!prefix_only) {   // the visibility window of tree_attn_shared_kernel
            const int first = key0 - P;
            const uint64_t window = first >= 0 ? mbits >> first : (mbits << -first) | ((1ull << -first) - 1);
            const uint32_t mine = (uint32_t)window >> (4 * h);
#pragma unroll
            for (int i = 0; i < 16; ++i) s[i] = ((mine >> (8 * (i >> 2) + (i & 3))) & 1u) ? s[i] : -__builtin_inff();
        }
        // the scale is positive (checked by the host): the largest raw score is the largest scaled one
        const float m_a = max_of_three(max_of_three(s[0], s[1], s[2]), max_of_three(s[3], s[4], s[5]), max_of_three(s[6], s[7], s[8]));
        const float m_b = max_of_three(max_of_three(s[9], s[10], s[11]), max_of_three(s[12], s[13], s[14]), s[15]);
        const float m_new = max_of_two(m_run, half_wave_max(max_of_two(m_a, m_b)) * scale_log2e);
        const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
        float psum[4];
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            float p[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i + e], scale_log2e, -m_new));
                pb[i >> 3][(i & 7) + e] = (_Float16)p[e];
            }
            psum[i >> 2] = (p[0] + p[1]) + (p[2] + p[3]);
        }
        l_run = l_run * alpha + ((psum[0] + psum[1]) + (psum[2] + psum[3]));
        m_run = m_new;
        if (__any(alpha != 1.0f)) {
#pragma unroll
            for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
        }
        if (more) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");   // V of this step; the next K is newer
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        // V^T fragments (dt, u), two ahead of the products that use them: slots 8 h .. 8 h + 3 are keys 16 u + 4 h .., slots
        // 8 h + 4 .. those eight further on -- the keys whose probabilities this lane's column holds
        short4v lo[8], hi[8];
        auto read_v = [&](auto f) {
            constexpr int F = decltype(f)::value;
            read_transposed_rows<(F & 1) * 16 * 256>(lo[F], hi[F], vbase + (vfrag ^ ((F >> 1) << 6)));
        };
        auto product = [&](auto f) {
            constexpr int F = decltype(f)::value;
            if constexpr (F + 2 < 8) read_v(std::integral_constant<int, F + 2>{});
            wait_lds_reads<F + 2 < 8 ? 4 : F + 1 < 8 ? 2 : 0>(lo[F], hi[F]);
            typedef short short8v __attribute__((ext_vector_type(8)));
            const short8v both = __builtin_shufflevector(lo[F], hi[F], 0, 1, 2, 3, 4, 5, 6, 7);
            const half8v va = __builtin_bit_cast(half8v, both);
            o[F >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(va, pb[F & 1], o[F >> 1], 0, 0, 0);
        };
        read_v(std::integral_constant<int, 0>{});
        read_v(std::integral_constant<int, 1>{});
        product(std::integral_constant<int, 0>{});
        product(std::integral_constant<int, 1>{});
        product(std::integral_constant<int, 2>{});
        product(std::integral_constant<int, 3>{});
        product(std::integral_constant<int, 4>{});
        product(std::integral_constant<int, 5>{});
        product(std::integral_constant<int, 6>{});
        product(std::integral_constant<int, 7>{});
        if (more) request(next, v_src, lane_v, 1, vtile);
        step = next;
    }

    // The states of the eight wavefronts meet in LDS; the weights are worked out once per (row, wavefront)
    l_run += __shfl_xor(l_run, 32, 64);
    __syncthreads();   // every wavefront has left the K, V and Q tiles
    uint8_t *const mine = lds + wave * kExWave;
    float2v *const state = reinterpret_cast<float2v *>(lds + kWaveState), *const weights = reinterpret_cast<float2v *>(lds + kWaveWeights);
    if (h == 0) state[c * kSharedWaves + wave] = (float2v){m_run, l_run};
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
        for (int a = 0; a < 4; ++a)
            *reinterpret_cast<float4v *>(mine + c * kExRow + (8 * dt + 2 * a + h) * 16) =
                (float4v){o[dt][4 * a], o[dt][4 * a + 1], o[dt][4 * a + 2], o[dt][4 * a + 3]};
    __syncthreads();
    auto row_max = [&](int row) {
        float m_all = kLowest;
#pragma unroll
        for (int w = 0; w < kSharedWaves; ++w) m_all = fmaxf(m_all, state[row * kSharedWaves + w][0]);
        return m_all;
    };
    if (tid < kWaveRows * kSharedWaves) {
        const float2v me = state[tid];
        const float wgt = __builtin_amdgcn_exp2f(me[0] - row_max(tid / kSharedWaves));
        weights[tid] = (float2v){wgt, wgt * me[1]};
    }
    __syncthreads();
    const bool last = nsplit == 1;
    const PartialBuffer unit_o = partial_buffer(part_o + (size_t)unit * nsplit * kRowsPad * kHeadDim);
    const PartialBuffer unit_ml = partial_buffer(part_ml + (size_t)unit * nsplit * kRowsPad * 2);
#pragma unroll
    for (int it = 0; it < 2; ++it) {   // thread t: four consecutive outputs of a row, 32 threads per row
        const int item = tid + it * (64 * kSharedWaves);
        const int rho = item >> 5, quad = item & 31;
        float4v val = {0.f, 0.f, 0.f, 0.f};
        float l_all = 0.f;
#pragma unroll
        for (int w = 0; w < kSharedWaves; ++w) {
            const float2v wl = weights[rho * kSharedWaves + w];
            l_all += wl[1];
            val += wl[0] * *reinterpret_cast<const float4v *>(lds + w * kExWave + rho * kExRow + quad * 16);
        }
        if (rho >= R) continue;
        if (last) {
            val *= 1.f / l_all;
            typedef _Float16 half4v __attribute__((ext_vector_type(4)));
            half4v hv = {(_Float16)val[0], (_Float16)val[1], (_Float16)val[2], (_Float16)val[3]};
            int qrow;
            *reinterpret_cast<half4v *>(out + locate(rho, qrow) + quad * 4) = hv;
        } else {   // written through to memory in either mode (see tree_attn_shared_kernel)
            store_partial(unit_o, (sp * kRowsPad + rho) * (kHeadDim / 4) + quad, val);
            if (quad == 0) {
                store_partial_f32(unit_ml, (sp * kRowsPad + rho) * 2, row_max(rho));
                store_partial_f32(unit_ml, (sp * kRowsPad + rho) * 2 + 1, l_all);
            }
        }
    }
    if (last || !fused) return;   // uniform over the grid
    __shared__ uint32_t ticket_sh;   // last-arriver merge of the tile's key ranges, as in tree_attn_kernel
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) ticket_sh = __hip_atomic_fetch_add(&tickets[unit], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (ticket_sh != (uint32_t)(nsplit - 1)) return;
    if (tid == 0) __hip_atomic_store(&tickets[unit], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    merge_tile(unit_o, unit_ml, out, tid, 64 * kSharedWaves, tile, nsplit);
}

// merge of the key ranges: one thread per four consecutive output elements, ranges in order;
// NS = compiled upper bound of the number of ranges (all loads of a thread are issued at once)
template <int NS>
__global__ __launch_bounds__(256) void tree_attn_merge_kernel(const float *__restrict__ part_o,
                                                              const float *__restrict__ part_ml,
                                                              _Float16 *__restrict__ out, int M, int Hq, int group, int nsplit,
                                                              int tile_rows, int tiles_per_kv)
{
    fetch_arguments_together(part_o, part_ml, out, M, Hq, group, nsplit, tile_rows, tiles_per_kv);
    const int idx = blockIdx.x * 256 + threadIdx.x;   // over M * Hq * 32 quads
    if (idx >= M * Hq * (kHeadDim / 4)) return;
    const int d4 = idx % (kHeadDim / 4), h = (idx / (kHeadDim / 4)) % Hq, qrow = idx / (kHeadDim / 4) / Hq;
    const float NEG_INF = -__builtin_inff();
    // where the first kernel left this (row, head): tile `unit`, tile row `row` (see RowTile)
    const int kvh = h / group, head = h - kvh * group;
    int index = head, row = qrow;
    if (tile_rows != M) {   // uniform
        const int pair = head * M + qrow;
        index = pair / tile_rows;
        row = pair - index * tile_rows;
    }
    const int unit = kvh * tiles_per_kv + index;
    const float *hml = part_ml + (size_t)unit * nsplit * kRowsPad * 2;
    const float4v *ho = reinterpret_cast<const float4v *>(part_o + (size_t)unit * nsplit * kRowsPad * kHeadDim);
    float ms[NS], ls[NS];
    float4v os[NS];
    const auto load = [&](int s, int range) {
        const size_t at = (size_t)range * kRowsPad + row;
        ms[s] = hml[at * 2];
        ls[s] = hml[at * 2 + 1];
        os[s] = ho[at * (kHeadDim / 4) + d4];
    };
    const auto drop = [&](int s) {
        ms[s] = NEG_INF;
        ls[s] = 0.f;
        os[s] = (float4v){0.f, 0.f, 0.f, 0.f};
    };
    if constexpr (NS <= 8) {
        // Ranges beyond the last read it again and are dropped.  Under a condition (below) the compiler made the loads of the four- and
        // eight-range forms wait for one another: whole calls with eight ranges, 64/8 heads, M = 24, prefix 2048 14.0 us against 12.0 now;
        // with more ranges the loads do go out together, and those that are not needed would cost 0.2 to 1.4 us.
#pragma unroll
        for (int s = 0; s < NS; ++s) load(s, min(s, nsplit - 1));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (s >= nsplit) drop(s);   // uniform
    } else {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            drop(s);
            if (s < nsplit) load(s, s);
        }
    }
    float m_all = NEG_INF;
#pragma unroll
    for (int s = 0; s < NS; ++s) m_all = fmaxf(m_all, ms[s]);
    float den = 0.f;
    float4v num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        float wgt = (ms[s] == NEG_INF) ? 0.f : __builtin_amdgcn_exp2f(ms[s] - m_all);   // ranges without a visible key: l = 0
        den += wgt * ls[s];
        num += wgt * os[s];
    }
    const float inv = 1.f / den;
    typedef _Float16 half4v __attribute__((ext_vector_type(4)));
    half4v hv = {(_Float16)(num[0] * inv), (_Float16)(num[1] * inv), (_Float16)(num[2] * inv), (_Float16)(num[3] * inv)};
    *reinterpret_cast<half4v *>(out + ((size_t)qrow * Hq + h) * kHeadDim + d4 * 4) = hv;
}

// Greedy acceptance of a verified draft tree, then compaction of the accepted K/V rows.
// Wavefront 0 walks the tree with lane i = node i: at node cur it broadcasts target[cur], every lane
// tests "my parent is cur and my token is that", and the lowest set bit of the ballot is the next
// node.  cur grows strictly, so the walk ends after at most M rounds whatever the input holds.
// Then all 256 threads move the accepted rows: thread t owns 16-byte column chunk t of every row and
// copies row path[j] to row j for j = 1, 2, ... in this order; path[j] >= j and the path is
// increasing, so a row is never overwritten before it has been read, and threads never share bytes.
__global__ __launch_bounds__(256) void tree_accept_kernel(const int32_t *__restrict__ parent,
                                                          const int32_t *__restrict__ token,
                                                          const int32_t *__restrict__ target, int M,
                                                          int32_t *__restrict__ path, int32_t *__restrict__ result,
                                                          u32x4 *k, u32x4 *v, int P, int row_chunks)
{
    __shared__ int32_t path_sh[kRowsPad];
    __shared__ int32_t n_sh;
    fetch_arguments_together(parent, token, target, M, path, result, k, v, P, row_chunks);
    const int tid = threadIdx.x;
    if (tid < 64) {
        const int lane = tid;
        const bool node = lane < M;
        const int32_t my_parent = node ? parent[lane] : -2;
        const int32_t my_token = node ? token[lane] : 0;
        const int32_t my_target = node ? target[lane] : 0;
        int cur = 0, n = 1;
        int32_t mine = lane == 0 ? 0 : -1;   // path entry of position `lane`
        for (;;) {
            const int32_t want = __shfl(my_target, cur, 64);
            const uint64_t hits = __ballot(node && lane > cur && my_parent == cur && my_token == want);
            if (hits == 0) break;
            cur = __builtin_ctzll(hits);
            if (lane == n) mine = cur;
            ++n;
        }
        const int32_t next_token = __shfl(my_target, cur, 64);   // the target model's own token after the last accepted node
        path_sh[lane] = mine;
        if (node) path[lane] = mine;
        if (lane == 0) {
            n_sh = n;
            result[0] = n;
            result[1] = next_token;
        }
    }
    __syncthreads();
    if (k == nullptr) return;
    const int n = n_sh;
    for (int item = tid; item < 2 * row_chunks; item += 256) {
        u32x4 *base = (item < row_chunks ? k : v) + (size_t)P * row_chunks + (item < row_chunks ? item : item - row_chunks);
        for (int j = 1; j < n; ++j) {
            const int src = path_sh[j];
            if (src != j) base[(size_t)j * row_chunks] = base[(size_t)src * row_chunks];
        }
    }
}

static int key_steps(int M, int P) { return (P + M + kKeyBlock - 1) / kKeyBlock; }

// How a call is cut up: row tiles (RowTile), key ranges per tile, who merges the ranges.
struct AttnPlan { int tile_rows, tiles_per_kv, ranges, fused; };
static size_t partial_bytes_of(int units, int ranges)
{
    return (size_t)units * ranges * kRowsPad * (kHeadDim + 2) * sizeof(float);
}

// Query heads per row tile of the plain plan.  The heads of a KV group can share a tile, which reads K
// and V once for all of them; fewer tiles, on the other hand, mean more key ranges per tile to fill the chip,
// and every range costs a partial result that has to be merged.  Measured over M = 1 .. 32 with 64/8 and 32/8
// heads (prefix 2048), the best point is about 32 tiles (eight key ranges each, merged by the last workgroup):
// the smallest pack that leaves at most 32 tiles is taken -- two heads of a group of eight with 64 heads (10.3
// to 12.9 us for M = 1 .. 16, against 12.7 to 13.2 unpacked), none with 32 heads (10.0 to 12.6 us for
// M = 1 .. 32, against 10.7 to 18.6 with two per tile).  Calls of so few rows that a whole group fits eight
// tile rows pack the group (plain decoding: 9.9 against 10.3 us).
static int heads_per_tile(int M, int Hq, int Hkv, int knob)
{
    const int group = Hq / Hkv;
    if (knob == 1 || group < 2) return 1;
    if (knob >= 10) {   // 10 + d: exactly d heads per tile, where that is possible
        const int d = knob - 10;
        return (d >= 2 && group % d == 0 && M * d <= kRowsPad) ? d : 1;
    }
    if (knob == 2) return M * group <= kRowsPad ? group : 1;
    if (M * group <= 8) return group;
    int best = 1;
    for (int d = 1; d <= group; ++d) {
        if (group % d != 0 || M * d > kRowsPad) continue;
        best = d;
        if (Hq / d <= 32) break;
    }
    return best;
}

// the whole group cut evenly into as few tiles as 64 rows allow; a tile may end inside a head
static void even_tiles(int pairs, int most, int &tile_rows, int &tiles_per_kv)
{
    const int n = (pairs + most - 1) / most;
    tile_rows = (pairs + n - 1) / n;
    tiles_per_kv = (pairs + tile_rows - 1) / tile_rows;
}

// Partial results (tiles x ranges) that the stated workspace holds: those of the plain plan with up to one tile per query head, and those
// of any plan_by_size() -- at most kChipTiles in all.  Grows with M and P, so one workspace serves smaller calls.  Tiles of at most 32 rows may
// be twice as many as query heads: the plain plan then takes no more ranges than fit.
static size_t stated_partials(int M, int P, int Hq)
{
    const size_t steps = (size_t)key_steps(M, P), heads = (size_t)Hq;
    const size_t plain = heads * (steps < kMaxSplits ? steps : kMaxSplits);
    const size_t by_size = heads * (steps < kMaxRanges ? steps : kMaxRanges);
    const size_t capped = by_size < kChipTiles ? by_size : kChipTiles;
    return plain > capped ? plain : capped;
}

// The plain plan, and what the knobs make of it.  The key ranges of a tile are merged by the last of its workgroups to
// finish, or by a second kernel.  Fused saves a launch and the wait for it, but one workgroup then reads all the partials
// of its tile (rows x ranges x 512 B), which pays while they are few.  Measured break-even points, prefix 2048: about 160
// row-ranges with up to four ranges (64 heads, M = 33 .. 64: 14.7 fused against 14.9 us at 132, 16.3 against
// 15.5 at 256); with five to eight ranges 512 for tiles of one head (32 heads, M = 64: 15.6 against 16.7 us)
// and 256 for packed ones (64 heads in pairs: 12.9 against 13.1 us at M = 16, 14.4 against 13.6 at M = 24);
// 256 with more ranges (M = 4 of 32 heads 10.7 against 11.0 us at 256, M = 8 of 64 heads 14.0 against 11.0
// at 512).
static AttnPlan plain_plan(int M, int P, int Hq, int Hkv, int pack, int splits, int most_ranges)
{
    const int group = Hq / Hkv, steps = key_steps(M, P);
    AttnPlan p;
    if (pack == 3 || pack == 4) {
        even_tiles(group * M, pack == 3 ? kRowsPad : kRowsPad / 2, p.tile_rows, p.tiles_per_kv);
    } else {
        const int d = heads_per_tile(M, Hq, Hkv, pack);
        p.tile_rows = d * M;
        p.tiles_per_kv = group / d;
    }
    const int units = Hkv * p.tiles_per_kv;
    int want = splits > 0 ? splits : (256 + units - 1) / units;   // about one workgroup per compute unit
    want = want > steps ? steps : want;
    if (pack == 4) {
        const int fit = (int)(stated_partials(M, P, Hq) / (size_t)units);   // one at least: more than Hq tiles have more than 32 rows and so two key steps
        most_ranges = most_ranges < fit ? most_ranges : fit;
    }
    p.ranges = want > most_ranges ? most_ranges : want < 1 ? 1 : want;
    const int row_ranges = p.tile_rows * p.ranges;
    p.fused = p.ranges > 1 && row_ranges <= (p.ranges <= 4 ? 160 : (p.ranges <= 8 && p.tile_rows == M) ? 512 : 256);
    return p;
}

// Time of a plan in microseconds, up to errors of some six percent: least-squares fits to 5700 measured plans of 165 calls (64/8,
// 40/8, 32/8, 16/2, 12/2 and 8/8 heads, M = 1 .. 64, prefixes of 16 .. 20000, every tiling, 1 .. 32 ranges, both merges), one for each
// of the two kernels.  A workgroup's walk costs per round of its key wavefronts and per step (its transfers), more when the chip is full; a fused
// merge costs by the last workgroup's rows and ranges, the second kernel its launch.
static float plan_time(const AttnPlan &p, int M, int P, int Hkv)
{
    const int units = Hkv * p.tiles_per_kv, groups = units * p.ranges, passes = (groups + 255) / 256;
    const int steps = (key_steps(M, P) + p.ranges - 1) / p.ranges;
    const float fill = (float)(groups < 256 ? groups : 256) / 256.f, rows = (float)p.tile_rows, ranges = (float)p.ranges;
    const bool beyond_l2 = (float)(P + M) * (Hkv > 8 ? (float)Hkv / 8.f : 1.f) > 5860.f;   // 3 MB of K and V per XCD (fewer than eight KV heads leave an XCD less)
    const float far = beyond_l2 ? fill * (float)steps : 0.f;
    if (p.tile_rows <= kWaveRows) {
        const float rounds = (float)((steps + 7) / 8);
        const float t = 5.225f + 0.028f * rows + (float)passes * (0.1672f * rounds * fill + 0.1562f * (float)steps + (steps > 8 ? 0.435f : 0.f) + 0.0487f * far);
        if (p.ranges > 1) return t + (p.fused ? 1.297f + 0.0557f * ranges + 0.0058f * rows * ranges : 2.715f + 0.00002f * (float)groups * rows + 0.042f * ranges);
        // the fit's error for one range of a few rounds: 40/8 heads, M = 2, nine steps 7.5 us, in three ranges 7.3.  With it the picks of nine head counts and prefixes of
        // 200 .. 760 are within 5 % of the best, but for 128/16 heads at 16 rows (two ranges 8.7, one 7.8)
        return steps > 8 ? t + 0.4f : t;
    }
    const float rounds = (float)((steps + 3) / 4);
    const float t = 5.73f + 0.0184f * rows + (float)passes * (0.4556f * (rounds - 1.f) + 0.0965f * rounds * fill + 0.2233f * (float)steps + 0.0183f * far);
    if (p.ranges == 1) return t;
    return t + (p.fused ? 1.55f + 0.00713f * rows * ranges : 2.27f + 0.0001122f * (float)groups * rows + 0.0229f * ranges + (p.ranges > 16 ? 0.268f : 0.f));
}

// The plain plan, or the one of these that promises the least time: d heads per tile, or even tiles of at most 64 or 32 rows, with one, two, four
// or eight ranges or as many as fill the chip (or a half or three quarters of it).  At long prefixes that is full tiles, which read K and V least often and
// waste no rows, and up to 32 ranges; at short ones a single range and no merge; and where the plain plan's rounding up
// makes more workgroups than compute units (40/8 heads: 280), as many as there are.  Tiles of up to 32 rows run in the kernel whose wavefronts share
// nothing and cover eight key steps at a time, so they need half the ranges: us, before that kernel -> now: prefix 2048, M = 24 of 64/8 heads 13.7 -> 11.3,
// M = 60 of 32/8 heads 14.9 -> 11.4, M = 1 8.5 -> 7.7; prefix 500, M = 18 of 64/8 heads 11.5 -> 8.4; prefix 16001, M = 40 of 32/8 heads 27.1 -> 25.0; 1025 random
// calls of sixteen head counts 0.87 to 0.89 of the time before, one of them 9 % more, no other 5 %.  (Nothing speaks for the plain plan as such: with a twentieth's
// allowance on long walks 39 of these calls took 2 to 3 % more.)  The picks lie 2 to 3 % behind the best measured plan in the mean.
static AttnPlan plan_by_size(const AttnPlan &plain, int M, int P, int Hq, int Hkv)
{
    const int group = Hq / Hkv, steps = key_steps(M, P);
    const int stated = (int)stated_partials(M, P, Hq);
    AttnPlan best = plain;
    float least = plan_time(plain, M, P, Hkv);
    // A group of at most eight rows stays in one tile.  Eight head counts, prefixes 60 .. 20000, against the best split of the group: ahead from prefix 1000 on with
    // eight KV heads (32/8, prefix 2048: 8.0 us against 8.4), elsewhere within 0.2 us; with two KV heads 0.2 to 1 us behind at prefixes of 300 to 12000
    for (int d = M * group <= 8 ? group : -1; d <= group; ++d) {
        AttnPlan p = {d * M, 0, 1, 0};
        if (d <= 0) {
            even_tiles(group * M, d == 0 ? kRowsPad : kWaveRows, p.tile_rows, p.tiles_per_kv);
        } else {
            if (group % d != 0 || M * d > kRowsPad) continue;
            p.tiles_per_kv = group / d;
        }
        const int units = Hkv * p.tiles_per_kv;
        int most = steps < kMaxRanges ? steps : kMaxRanges;
        most = most > kChipTiles / units ? kChipTiles / units : most;
        const int choices[7] = {1, 2, 4, 8, most / 2, most * 3 / 4, most};
        for (int i = 0; i < 7; ++i) {
            p.ranges = choices[i];
            if (p.ranges < 1 || p.ranges > most || (p.ranges > 1 && units * p.ranges > stated)) continue;
            if (i > 3 && (p.ranges <= 2 || p.ranges == 4 || p.ranges == 8)) continue;   // already looked at
            for (p.fused = 0; p.fused < (p.ranges > 1 ? 2 : 1); ++p.fused) {
                const float t = plan_time(p, M, P, Hkv);
                if (t < least) least = t, best = p;
            }
        }
    }
    return best;
}

// bytes of partial results a plan writes; one range writes none
static size_t plan_bytes(const AttnPlan &p, int Hkv)
{
    return p.ranges > 1 ? partial_bytes_of(Hkv * p.tiles_per_kv, p.ranges) : 0;
}

// The plan of a call whose workspace has `room` bytes for partial results.  It follows from the sizes of the call alone, so
// that the bits of the result do not depend on how large a workspace the caller keeps.  Less than the stated size is
// accepted as long as it holds the plain plan, which runs where the preferred one does not fit; ranges == 0: not even that.
static AttnPlan attn_plan(int M, int P, int Hq, int Hkv, size_t room)
{
    const Params &pr = params();
    AttnPlan plain = plain_plan(M, P, Hq, Hkv, pr.attn_pack, pr.attn_splits, kMaxSplits);
    if (plan_bytes(plain, Hkv) > room) {
        plain.ranges = 0;
        return plain;
    }
    AttnPlan best = plain;
    if (pr.attn_splits > kMaxSplits) {   // asked for: as many of them as the stated workspace holds
        const size_t fit = stated_partials(M, P, Hq) / (size_t)(Hkv * plain.tiles_per_kv);
        best = plain_plan(M, P, Hq, Hkv, pr.attn_pack, pr.attn_splits, fit < kMaxRanges ? (int)fit : kMaxRanges);
    } else if (pr.attn_pack == 0 && pr.attn_splits == 0) {
        best = plan_by_size(plain, M, P, Hq, Hkv);
    }
    if (plan_bytes(best, Hkv) > room) best = plain;
    if (pr.attn_fused_merge != 0) best.fused = best.ranges > 1 && pr.attn_fused_merge == 2;
    if (Hkv * best.tiles_per_kv > kMaxTickets) best.fused = 0;   // a ticket per tile
    return best;
}

template <int RT, int RG, typename... Args>
static int launch_attn_variant(int grid, hipStream_t stream, Args... args)
{
    static bool lds_ok = false;   // LDS above 48 KB needs an opt-in, once per variant
    constexpr int lds = attn_lds_bytes(RT, RG);
    if (!lds_ok) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_kernel<RT, RG>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return W4A16_EHIP;
        lds_ok = true;
    }
    hipLaunchKernelGGL((tree_attn_kernel<RT, RG>), dim3((unsigned)grid), dim3(256 * RG), lds, stream, args...);
    return W4A16_OK;
}

template <typename... Args>
static int launch_attn_shared(int grid, hipStream_t stream, Args... args)
{
    static bool lds_ok = false;
    if (!lds_ok) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_shared_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kSharedLds) != hipSuccess)
            return W4A16_EHIP;
        lds_ok = true;
    }
    hipLaunchKernelGGL(tree_attn_shared_kernel, dim3((unsigned)grid), dim3(64 * kSharedWaves), kSharedLds, stream, args...);
    return W4A16_OK;
}

template <typename... Args>
static int launch_attn_wave(int grid, hipStream_t stream, Args... args)
{
    static bool lds_ok = false;
    if (!lds_ok) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(&tree_attn_wave_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kWaveLds) != hipSuccess)
            return W4A16_EHIP;
        lds_ok = true;
    }
    hipLaunchKernelGGL(tree_attn_wave_kernel, dim3((unsigned)grid), dim3(64 * kSharedWaves), kWaveLds, stream, args...);
    return W4A16_OK;
}

template <typename... Args>
static int launch_attn(int rt, int rgroups, int grid, hipStream_t stream, uint32_t by_tiles, uint32_t by_ranges, Args... args)
{
    if (rt == 0) return rgroups == 2 ? launch_attn_shared(grid, stream, by_tiles, by_ranges, args...) : launch_attn_wave(grid, stream, by_tiles, by_ranges, args...);
    if (rt == 4) return launch_attn_variant<4, 1>(grid, stream, args...);
    if (rgroups == 2) return launch_attn_variant<2, 2>(grid, stream, args...);
    return launch_attn_variant<2, 1>(grid, stream, args...);
}

static int check_attn(int M, int P, int Hq, int Hkv, int D)
{
    if (M < 1 || P < 0 || Hq < 1 || Hkv < 1 || D < 1) return W4A16_EINVAL;
    if (Hq % Hkv != 0) return W4A16_EINVAL;
    if (D != kHeadDim || M > W4A16_MAX_M || Hq > kMaxTickets || Hq / Hkv > 8) return W4A16_EUNSUP;
    return W4A16_OK;
}

}  // namespace w4

using namespace w4;

extern "C" {

size_t tree_verify_attn_workspace_bytes(int M, int P, int Hq, int Hkv, int D)
{
    if (check_attn(M, P, Hq, Hkv, D) != W4A16_OK) return 0;
    return kTicketBytes + stated_partials(M, P, Hq) * partial_bytes_of(1, 1);
}

int tree_verify_attn(const void *q, const void *k, const void *v, const uint8_t *mask, void *out,
                     int M, int P, int Hq, int Hkv, int D, float scale,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    int rc = check_attn(M, P, Hq, Hkv, D);
    if (rc != W4A16_OK) return rc;
    if (!(scale > 0.f) || scale > 3.0e38f) return W4A16_EINVAL;   // the kernels take row maxima before scaling
    if (!q || !k || !v || !mask || !out) return W4A16_ENULL;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || workspace_misaligned(workspace)) return W4A16_EALIGN;
    const AttnPlan pl = attn_plan(M, P, Hq, Hkv, workspace && workspace_bytes > kTicketBytes ? workspace_bytes - kTicketBytes : 0);
    if (pl.ranges == 0) return W4A16_EWORKSPACE;
    const int units = Hkv * pl.tiles_per_kv, ns = pl.ranges, rows = pl.tile_rows;
    float *part_o = reinterpret_cast<float *>(reinterpret_cast<uint8_t *>(workspace) + kTicketBytes);
    float *part_ml = part_o + (size_t)units * ns * kRowsPad * kHeadDim;
    const float scale_log2e = scale * 1.4426950408889634f;
    const int nblk = key_steps(M, P);
    // Tiles of more than 32 rows run in the kernel that shares K and V tiles through LDS, others in the one whose wavefronts have
    // their own (rt = 0 below).  The older kernel stays selectable for comparison: one wavefront per SIMD carrying all 64 rows (4), or 32
    // rows per wavefront, in two row groups for taller tiles (2).
    const int knob = params().attn_row_tiles;
    const int rt = knob == 4 ? 4 : knob == 2 ? 2 : 0, rgroups = rows > kWaveRows ? 2 : 1;
    rc = launch_attn(rt, rgroups, units * ns, (hipStream_t)stream, divider(pl.tiles_per_kv), divider(ns), (const _Float16 *)q, (const _Float16 *)k,
                     (const _Float16 *)v, mask, (_Float16 *)out, part_o, part_ml, reinterpret_cast<uint32_t *>(workspace),
                     M, P, Hq, Hkv, Hq / Hkv, scale_log2e, ns, nblk / ns, nblk % ns, rows, pl.tiles_per_kv, pl.fused);
    if (rc != W4A16_OK) return rc;
    if (ns > 1 && !pl.fused) {
        const int quads = M * Hq * (kHeadDim / 4);
        const dim3 grid((unsigned)((quads + 255) / 256));
#define W4_ATTN_MERGE(NS_)                                                                                              \
        hipLaunchKernelGGL(tree_attn_merge_kernel<NS_>, grid, dim3(256), 0, (hipStream_t)stream, (const float *)part_o,  \
                           (const float *)part_ml, (_Float16 *)out, M, Hq, Hq / Hkv, ns, rows, pl.tiles_per_kv)
        if (ns <= 4) W4_ATTN_MERGE(4);
        else if (ns <= 8) W4_ATTN_MERGE(8);
        else if (ns <= 16) W4_ATTN_MERGE(16);
        else W4_ATTN_MERGE(kMaxRanges);
#undef W4_ATTN_MERGE
    }
    return launch_status();
}

int tree_verify_attn_plan_describe(int M, int P, int Hq, int Hkv, int D, size_t workspace_bytes, int *out)
{
    if (!out) return W4A16_ENULL;
    int rc = check_attn(M, P, Hq, Hkv, D);
    if (rc != W4A16_OK) return rc;
    const AttnPlan pl = attn_plan(M, P, Hq, Hkv, workspace_bytes > kTicketBytes ? workspace_bytes - kTicketBytes : 0);
    if (pl.ranges == 0) return W4A16_EWORKSPACE;
    const AttnPlan plain = plain_plan(M, P, Hq, Hkv, params().attn_pack, params().attn_splits, kMaxSplits);
    out[0] = pl.tile_rows;
    out[1] = pl.tiles_per_kv;
    out[2] = pl.ranges;
    out[3] = pl.fused;
    out[4] = pl.tile_rows == plain.tile_rows && pl.tiles_per_kv == plain.tiles_per_kv && pl.ranges == plain.ranges;
    return W4A16_OK;
}

int tree_accept(const int32_t *parent, const int32_t *token, const int32_t *target, int M, int32_t *path,
                int32_t *result, void *k, void *v, int P, int Hkv, int D, void *stream)
{
    if (M < 1 || P < 0) return W4A16_EINVAL;
    if (M > W4A16_MAX_M) return W4A16_EUNSUP;
    if (!parent || !token || !target || !path || !result) return W4A16_ENULL;
    if ((k == nullptr) != (v == nullptr)) return W4A16_ENULL;
    int row_chunks = 0;
    if (k) {
        if (Hkv < 1 || D < 1) return W4A16_EINVAL;
        if (((size_t)Hkv * D * 2) % 16 != 0) return W4A16_EUNSUP;
        if (misaligned(k) || misaligned(v)) return W4A16_EALIGN;
        row_chunks = (int)((size_t)Hkv * D * 2 / 16);
    }
    if ((reinterpret_cast<uintptr_t>(parent) | reinterpret_cast<uintptr_t>(token) | reinterpret_cast<uintptr_t>(target) |
         reinterpret_cast<uintptr_t>(path) | reinterpret_cast<uintptr_t>(result)) & 3u)
        return W4A16_EALIGN;
    hipLaunchKernelGGL(tree_accept_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, parent, token, target, M, path,
                       result, (u32x4 *)k, (u32x4 *)v, P, row_chunks);
    return launch_status();
}

}  // extern "C"
