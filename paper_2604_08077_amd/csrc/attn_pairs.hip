// Sparse attention (Eq. 3 + own-cube rule, Sec. 3.2), key-stationary: the work follows the selected
// (query row, key cube) pairs instead of the rows.
//
// The two row-stationary kernels (attn_walk.hip, attn_compact.hip) stream every key cube past every block of
// rows, so with rows that select independently they cost what dense attention costs however little is selected.
// Here the selection is first transposed into one work list per (KV head, key cube): the rows that selected the
// cube.  A workgroup keeps ONE key cube's K and V^T tiles in LDS and its wavefronts run a chunk of that list
// through the tiles, 32 rows at a time, with no workgroup barrier after the load.  What a row gets from one cube
// is a partial result -- unnormalised O, running maximum m, sum l -- written to a record in caller-provided
// scratch memory.  A record holds m, l and s = max |O| in fp32 and O / s in fp16: the merged output is a weighted
// mean of the records' O / l, so a record's rounding error enters it with at most 2^-11 of that record's largest
// element, an eighth of the rounding of the bf16 output itself, at half the memory traffic of fp32 records.  The causal part of every row's own cube is one more record, written by workgroups of
// their own in the same launch, over the rows of each cube.  A last kernel merges each row's records (they are contiguous: a row's
// records are numbered in cube order after an exclusive scan of the per-row counts, the own cube last) into the
// output.
//
// Cost: MFMA work in proportion to the selected pairs, plus 2 * D + 16 bytes written and read per pair and 8
// bytes of work list.  The entry (attn_walk.hip: launch_attn) decides on the device, from the exact pair count and
// per KV head (heads can differ widely in how much they select), whether this path or a row-stationary kernel
// takes the head's rows.
#include <algorithm>

#include "attn_tile.h"

namespace adaspark {

constexpr int PAIRS_MAX_TPC = 4;          // a key cube of up to 256 tokens stays in LDS
constexpr int PAIRS_MAX_SEGMENTS = 8192;  // (KV head, cube) work lists: two LDS histograms of that many counters
constexpr int PAIRS_CHUNK = 3584;         // work-list entries per workgroup (staged in LDS: 28 KB); 14 steps per wavefront
constexpr int PAIRS_TILE = 1024;          // rows per workgroup, a thread each, in the passes over the selection

template <int D>
struct Pairs {
    static constexpr int WAVES = 8;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int NS = FWD_NS;
    static constexpr int ROWS = 16 * NS;  // rows a wavefront takes per step
    static constexpr int PF = 4;
    static constexpr int CHUNK = KEY_TILE * D * 2;
    static constexpr int PIECES = CHUNK / 1024;  // 1 KB direct-to-LDS copies per tile
    // K and V^T tiles alternate in LDS (K0 V0 K1 V1 ...): both tiles of a step's operand loads then lie within 64 KB
    // of one base register, the reach of the LDS instructions' immediate offset
    static constexpr int OFF_K = 0;
    static constexpr int OFF_V = CHUNK;
    static constexpr int TILE_STRIDE = 2 * CHUNK;
    static constexpr int OFF_ROWS = 2 * PAIRS_MAX_TPC * CHUNK;  // (row id, record) of the workgroup's rows
    static constexpr int OFF_FILL = OFF_ROWS + PAIRS_CHUNK * 8;  // fill_masks
    static constexpr int BYTES = OFF_FILL + FILL_MASK_BYTES;
    static_assert(BYTES <= 160 * 1024, "LDS of one CU");
    static_assert(PAIRS_CHUNK % (2 * WAVES * ROWS) == 0, "an even number of steps per wavefront");
};

bool pairs_supported(const Geom &g)
{
    return g.TPC <= PAIRS_MAX_TPC && g.Hkv * g.N <= PAIRS_MAX_SEGMENTS && g.Hkv <= PAIRS_MAX_KV_HEADS;
}

// Scratch memory of the pair path, carved from `bytes` bytes at `base` (256-byte aligned):
//   flags      i32 [4 + Hkv]  the kernel-choice flags (geom.h)
//   share      i32 [Hkv]      estimated share of selected candidate cubes per KV head, permille (behind the flags)
//   qs         fp16 [R][D]    Q times the softmax scale in base 2 (rows of the heads this path takes): the operand of
//                             the score MFMAs, see softmax_tile_folded
//   cnt        i32 [R]        selected cubes per row
//   pair_ptr   i64 [R + 1]    a row's records, in cube order, the own cube last: exclusive scan of cnt + 1 over the rows of
//                             the heads this path takes
//   tile_need  u32 [tiles][Hkv]  records that the rows of a tile (PAIRS_TILE rows) and KV head would need
//   tile_off   i64 [tiles]    exclusive scan of the tiles' records
//   seg_count  u32 [Hkv * N]  rows that selected cube j, per KV head
//   seg_start  u32 [Hkv * N + 1]
//   seg_cursor u32 [Hkv * N]
//   seg_chunk  u32 [Hkv * N + 1]  exclusive scan of the lists' chunk counts (a chunk: PAIRS_CHUNK entries)
//   entries    u32 [cap][2]   the work lists: (row id, record index), list (kv, j) at seg_start[kv * N + j]
//   ml         f32 [cap][4]   of every record: running maximum m (base-2, scaled), sum l, s = max |O|, unused
//   rec        f16 [cap][D]   O / s, unnormalised partial outputs scaled to [-1, 1]; element (e, q4, v) of the
//                             MFMA output layout (head-dim 16 e + 4 q4 + v) sits at ((e / 2) * 4 + q4) * 8 + (e % 2) * 4 + v
struct PairsScratch {
    int *flags;
    uint16_t *qs;
    int32_t *cnt;
    int64_t *pair_ptr;
    uint32_t *tile_need;
    long long *tile_off;
    uint32_t *seg_count, *seg_start, *seg_cursor, *seg_chunk;
    uint32_t *entries;
    float *ml;
    uint16_t *rec;
    long long cap;  // records that fit; <= 0: not even the tables do
};

static size_t up256(size_t x) { return (x + 255) / 256 * 256; }

static size_t pairs_tiles(const Geom &g) { return ((size_t)g.S * g.Hq + PAIRS_TILE - 1) / PAIRS_TILE; }

static size_t pairs_table_bytes(const Geom &g)
{
    const size_t R = (size_t)g.S * g.Hq, segs = (size_t)g.Hkv * g.N;
    return FLAG_BLOCK_BYTES + 512 + up256(R * (size_t)g.D * 2) + up256(R * 4) + up256((R + 1) * 8) + up256(pairs_tiles(g) * g.Hkv * 4) +
           up256(pairs_tiles(g) * 8) + 4 * up256((segs + 1) * 4);
}

static size_t pairs_record_bytes(const Geom &g, size_t records)
{
    return up256(records * 8) + up256(records * 16) + up256(records * (size_t)g.D * 2);
}

size_t pairs_scratch_bytes(const Geom &g, long long max_selected)
{
    const size_t records = (size_t)max_selected + (size_t)g.S * g.Hq;
    return pairs_table_bytes(g) + pairs_record_bytes(g, records);
}

static PairsScratch pairs_layout(const Geom &g, void *base, size_t bytes)
{
    PairsScratch s{};
    const size_t R = (size_t)g.S * g.Hq, segs = (size_t)g.Hkv * g.N;
    const size_t tables = pairs_table_bytes(g);
    if (base == nullptr || bytes < tables + pairs_record_bytes(g, 1)) {
        s.cap = 0;
        return s;
    }
    static_assert((FLAG_KV + PAIRS_MAX_KV_HEADS) * 4 <= FLAG_BLOCK_BYTES && PAIRS_MAX_KV_HEADS * 4 <= 512,
                  "flag block, head shares");
    char *p = reinterpret_cast<char *>(base);
    s.flags = reinterpret_cast<int *>(p);
    p += FLAG_BLOCK_BYTES + 512;
    s.qs = reinterpret_cast<uint16_t *>(p);
    p += up256(R * (size_t)g.D * 2);
    s.cnt = reinterpret_cast<int32_t *>(p);
    p += up256(R * 4);
    s.pair_ptr = reinterpret_cast<int64_t *>(p);
    p += up256((R + 1) * 8);
    s.tile_need = reinterpret_cast<uint32_t *>(p);
    p += up256(pairs_tiles(g) * g.Hkv * 4);
    s.tile_off = reinterpret_cast<long long *>(p);
    p += up256(pairs_tiles(g) * 8);
    s.seg_count = reinterpret_cast<uint32_t *>(p);
    p += up256((segs + 1) * 4);
    s.seg_start = reinterpret_cast<uint32_t *>(p);
    p += up256((segs + 1) * 4);
    s.seg_cursor = reinterpret_cast<uint32_t *>(p);
    p += up256((segs + 1) * 4);
    s.seg_chunk = reinterpret_cast<uint32_t *>(p);
    p += up256((segs + 1) * 4);
    const size_t left = bytes - tables;
    size_t cap = left / (24 + (size_t)g.D * 2);
    while (cap > 0 && pairs_record_bytes(g, cap) > left) --cap;  // every array starts on a 256-byte boundary
    if (cap > 0xfffffff0ull) cap = 0xfffffff0ull;                // record indices are 32-bit
    s.entries = reinterpret_cast<uint32_t *>(p);
    p += up256(cap * 8);
    s.ml = reinterpret_cast<float *>(p);
    p += up256(cap * 16);
    s.rec = reinterpret_cast<uint16_t *>(p);
    s.cap = (long long)cap;
    return s;
}

// Bits of a row's mask word w that count: cubes before the row's own cube i (a well-formed mask has no others;
// stray ones are ignored here as the row-stationary kernels ignore them).
__device__ __forceinline__ uint32_t valid_bits(uint32_t word, int w, int i)
{
    const int hi = i - 32 * w;
    if (hi <= 0) return 0u;
    return hi >= 32 ? word : (word & ((1u << hi) - 1u));
}

// The counting kernels are skipped when the sampled estimate of the selected share (flag[1], permille) says that
// this path will not be chosen anyway: well above the threshold, and not forced.
// The break-even share was measured against a masked walk that computes every candidate cube; it computes only the
// share flag[FLAG_UNION] of them (cubes no row of a workgroup selected are left out), and the break-even moves with it.
__device__ __forceinline__ int pairs_threshold(const int *flag, int pairs_below_permille)
{
    // (a tenth of the candidates on top: the walk's fixed costs do not shrink with the union)
    return (int)((long long)pairs_below_permille * min(1000, flag[FLAG_UNION] + 100) / 1000);
}

__device__ __forceinline__ bool pairs_gate_closed(const int *flag, int force, int pairs_below_permille)
{
    const int below = pairs_threshold(flag, pairs_below_permille);
    return !force && flag[FLAG_ESTIMATE] > below + below / 4;
}

// Whether the rows of KV head kv may become this path's: its estimated share is not well above the threshold.
__device__ __forceinline__ bool pairs_head_open(const int *flag, int kv, int force, int pairs_below_permille)
{
    const int below = pairs_threshold(flag, pairs_below_permille);
    return force || flag[FLAG_SHARE + kv] <= below + below / 4;
}

// The preparation is three passes, all of them over in a few microseconds where the path is not taken:
//   pair_count_kernel   over the rows: selected cubes per row; records per (tile of rows, KV head); rows per (KV head, cube)
//   pairs_plan_kernel   one workgroup: the heads this path takes; scans of the tiles' records, the lists' lengths and chunks
//   pair_fill_kernel    over the rows: pair_ptr, the work lists, the scaled copy of Q
// A row of a head that cannot be taken costs the first pass its counts only.  65,536 tokens of 28/4 heads, Top-p 0.5: 44 + 12 + 490 us (a
// third of it the copy of Q); seven kernels with 256 rows a workgroup and 64-bit row numbers took 720.
// (Ranges of 1,024 rows: a workgroup adds its counts to every list with one atomic, and its entries of a list lie together.)
__device__ __forceinline__ void row_of(const Geom &g, uint32_t r, int &kv, int &i)
{
    const uint32_t n = r / (uint32_t)g.Hq;
    kv = (int)((r - n * (uint32_t)g.Hq) / (uint32_t)g.G);
    i = cube_of_token(g, (int)n);
}

template <typename F>
__device__ __forceinline__ void for_selected(const uint32_t *mr, int i, F &&f)
{
    for (int w = 0; 32 * w < i; ++w) {
        uint32_t bits = valid_bits(mr[w], w, i);
        while (bits) {
            const int b = __ffs(bits) - 1;
            bits &= bits - 1;
            f(32 * w + b);
        }
    }
}

__global__ __launch_bounds__(PAIRS_TILE) void pair_count_kernel(Geom g, uint32_t R, const uint32_t *__restrict__ sel_mask,
                                                                int32_t *__restrict__ cnt, uint32_t *__restrict__ seg_count,
                                                                uint32_t *__restrict__ tile_need, const int *__restrict__ flag,
                                                                int force, int pairs_below_permille)
{
    if (pairs_gate_closed(flag, force, pairs_below_permille)) return;
    extern __shared__ uint32_t hist[];  // [segs]
    __shared__ uint32_t need[PAIRS_MAX_KV_HEADS];
    const int segs = g.Hkv * g.N;
    for (int x = threadIdx.x; x < segs; x += PAIRS_TILE) hist[x] = 0u;
    if (threadIdx.x < PAIRS_MAX_KV_HEADS) need[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t r = blockIdx.x * PAIRS_TILE + threadIdx.x;
    if (r < R) {
        int kv, i, c = 0;
        row_of(g, r, kv, i);
        const uint32_t *mr = sel_mask + (size_t)r * g.words;
        if (pairs_head_open(flag, kv, force, pairs_below_permille))
            for_selected(mr, i, [&](int j) {
                atomicAdd(&hist[kv * g.N + j], 1u);
                ++c;
            });
        cnt[r] = c;
        atomicAdd(&need[kv], (uint32_t)c + 1u);
    }
    __syncthreads();
    for (int x = threadIdx.x; x < segs; x += PAIRS_TILE)
        if (hist[x]) atomicAdd(&seg_count[x], hist[x]);
    if (threadIdx.x < g.Hkv) tile_need[(size_t)blockIdx.x * g.Hkv + threadIdx.x] = need[threadIdx.x];
}

// Exclusive scan of one value per thread over the workgroup; all threads get the total.
__device__ __forceinline__ unsigned long long block_scan(unsigned long long x, unsigned long long *lds,
                                                         unsigned long long &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long incl = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long up = __shfl_up(incl, d, 64);
        if (lane >= d) incl += up;
    }
    __syncthreads();  // (lds: of the scan before)
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    unsigned long long before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < PAIRS_TILE / 64; ++w) {
        const unsigned long long t = lds[w];
        if (w < wave) before += t;
        total += t;
    }
    return before + incl - x;
}

// The key-stationary kernel takes a KV head's rows (flags[FLAG_KV + kv] = 3) if its share of selected candidate cubes is
// below the threshold (or force); if the records of the heads so chosen do not fit, or (together) one is not chosen, none is taken.
__global__ __launch_bounds__(PAIRS_TILE) void pairs_plan_kernel(Geom g, long long cap, unsigned long long candidates_per_head,
                                                                int tiles, const uint32_t *__restrict__ tile_need,
                                                                const uint32_t *__restrict__ seg_count,
                                                                long long *__restrict__ tile_off,
                                                                uint32_t *__restrict__ seg_start,
                                                                uint32_t *__restrict__ seg_chunk, int *__restrict__ flags,
                                                                int force, int together, int pairs_below_permille)
{
    if (pairs_gate_closed(flags, force, pairs_below_permille)) return;
    __shared__ unsigned long long need[PAIRS_MAX_KV_HEADS], scan[PAIRS_TILE / 64];
    __shared__ int take[PAIRS_MAX_KV_HEADS], active;
    const int t = threadIdx.x;
    if (t < PAIRS_MAX_KV_HEADS) need[t] = 0ull;
    __syncthreads();
    const int entries = tiles * g.Hkv;  // (tile, head): consecutive threads, consecutive entries
    unsigned long long mine = 0;
    const int step = PAIRS_TILE / g.Hkv * g.Hkv;  // a thread stays with one head
    if (t < step)
        for (int x = t; x < entries; x += step) mine += tile_need[x];
    if (t < step && mine) atomicAdd(&need[t % g.Hkv], mine);
    __syncthreads();
    if (t == 0) {
        unsigned long long total = 0;
        bool all = true;
        const unsigned long long rows = (unsigned long long)g.S * g.G;
        for (int kv = 0; kv < g.Hkv; ++kv) {
            take[kv] = force || (pairs_head_open(flags, kv, force, pairs_below_permille) &&
                                 (need[kv] - rows) * 1000ull <
                                     candidates_per_head * (unsigned long long)pairs_threshold(flags, pairs_below_permille));
            if (take[kv]) total += need[kv];
            else all = false;
        }
        active = total > 0ull && total <= (unsigned long long)cap && (all || !together);
        flags[FLAG_ACTIVE] = active;
    }
    __syncthreads();
    if (t < g.Hkv) flags[FLAG_KV + t] = active && take[t] ? 3 : 0;
    if (!active) return;
    unsigned long long carry = 0, total;
    for (int x0 = 0; x0 < tiles; x0 += PAIRS_TILE) {
        const int x = x0 + t;
        unsigned long long v = 0;
        if (x < tiles)
            for (int kv = 0; kv < g.Hkv; ++kv)
                if (take[kv]) v += tile_need[(size_t)x * g.Hkv + kv];
        const unsigned long long at = block_scan(v, scan, total);
        if (x < tiles) tile_off[x] = (long long)(carry + at);
        carry += total;
    }
    // lists: entries in the low half, chunks in the high one (fewer than 2^32 entries: record indices are 32-bit)
    carry = 0;
    const int segs = g.Hkv * g.N;
    for (int x0 = 0; x0 < segs; x0 += PAIRS_TILE) {
        const int x = x0 + t;
        const unsigned long long n = x < segs && take[x / g.N] ? seg_count[x] : 0u;
        const unsigned long long at = carry + block_scan(n | (n + PAIRS_CHUNK - 1) / PAIRS_CHUNK << 32, scan, total);
        if (x < segs) {
            seg_start[x] = (uint32_t)at;
            seg_chunk[x] = (uint32_t)(at >> 32);
        }
        carry += total;
    }
    if (t == 0) {
        seg_start[segs] = (uint32_t)carry;
        seg_chunk[segs] = (uint32_t)(carry >> 32);
    }
}

// Every (row, cube) pair of the heads taken is written into list (kv, j) as (row id, record index): the block's count of a
// list reserves a range of it with one global atomic.  qs = fp16(Q * log2(e)/sqrt(D)) for the rows of these heads (the score
// operand: attn_tile.h).
__global__ __launch_bounds__(PAIRS_TILE) void pair_fill_kernel(Geom g, uint32_t R, float c2, const uint16_t *__restrict__ Q,
                                                               const uint32_t *__restrict__ sel_mask,
                                                               const int32_t *__restrict__ cnt,
                                                               const long long *__restrict__ tile_off,
                                                               const int *__restrict__ mode_flag,
                                                               const uint32_t *__restrict__ seg_start,
                                                               uint32_t *__restrict__ seg_cursor,
                                                               int64_t *__restrict__ pair_ptr, uint32_t *__restrict__ entries,
                                                               uint16_t *__restrict__ qs)
{
    if (!mode_flag[FLAG_ACTIVE]) return;
    extern __shared__ uint32_t hist[];  // [segs] counts, then the ranges' first positions; [segs] positions handed out
    __shared__ unsigned long long scan[PAIRS_TILE / 64];
    const int segs = g.Hkv * g.N;
    uint32_t *taken = hist + segs;
    for (int x = threadIdx.x; x < 2 * segs; x += PAIRS_TILE) hist[x] = 0u;
    __syncthreads();
    const uint32_t r = blockIdx.x * PAIRS_TILE + threadIdx.x;
    int i = 0, kv = 0;
    bool mine = false;  // rows of heads left to a row-stationary kernel take no part
    const uint32_t *mr = sel_mask + (size_t)r * g.words;
    if (r < R) {
        row_of(g, r, kv, i);
        mine = mode_flag[FLAG_KV + kv] == 3;
        if (mine) for_selected(mr, i, [&](int j) { atomicAdd(&hist[kv * g.N + j], 1u); });
    }
    unsigned long long total;
    const unsigned long long slot0 =
        (unsigned long long)tile_off[blockIdx.x] + block_scan(mine ? (unsigned long long)cnt[r] + 1ull : 0ull, scan, total);
    if (r < R) pair_ptr[r] = (int64_t)slot0;
    if (r == R - 1) pair_ptr[R] = (int64_t)(slot0 + (mine ? cnt[r] + 1 : 0));
    // (the barriers of the scan: the counts are complete)
    for (int x = threadIdx.x; x < segs; x += PAIRS_TILE)
        if (hist[x]) hist[x] = seg_start[x] + atomicAdd(&seg_cursor[x], hist[x]);
    __syncthreads();
    if (mine) {
        uint32_t slot = (uint32_t)slot0;  // records of a row are numbered in cube order
        for_selected(mr, i, [&](int j) {
            const int x = kv * g.N + j;
            const uint32_t pos = hist[x] + atomicAdd(&taken[x], 1u);
            *reinterpret_cast<uint2 *>(entries + 2 * (size_t)pos) = make_uint2(r, slot);
            ++slot;
        });
    }
    const uint32_t per_row = (uint32_t)g.D / 8, first = blockIdx.x * PAIRS_TILE;
    for (uint32_t x = threadIdx.x; x < PAIRS_TILE * per_row; x += PAIRS_TILE) {
        const uint32_t row = first + x / per_row;
        if (row >= R || mode_flag[FLAG_KV + (int)(row % (uint32_t)g.Hq) / g.G] != 3) continue;
        const size_t at = (size_t)first * g.D + (size_t)x * 8;
        *reinterpret_cast<bf16x8 *>(qs + at) = score_operand(*reinterpret_cast<const bf16x8 *>(Q + at), c2);
    }
}

// OWN = false: workgroup b runs chunk b of all lists' chunks: entries [c * PAIRS_CHUNK, ...) of the work list (kv, j)
//              with seg_chunk[kv * N + j] <= b < seg_chunk[kv * N + j + 1], c = b - seg_chunk[kv * N + j].
// OWN = true:  workgroup b = (kv, j, c) runs rows [c * PAIRS_CHUNK, ...) of cube j itself against it, causally (key rank
//              <= query rank); own_chunks workgroups per cube.
template <int D, bool OWN>
__device__ __forceinline__ void attn_pairs_work(
    uint32_t block, const Geom &g, int own_chunks, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kp,
    const uint16_t *__restrict__ Vt, const int32_t *__restrict__ csize, const int64_t *__restrict__ pair_ptr, const uint32_t *__restrict__ seg_count,
    const uint32_t *__restrict__ seg_start, const uint32_t *__restrict__ seg_chunk,
    const uint32_t *__restrict__ entries, const int *__restrict__ mode_flag, uint16_t *__restrict__ rec,
    float *__restrict__ ml)
{
    using C = Pairs<D>;
    constexpr int NS = C::NS, WAVES = C::WAVES, PF = C::PF;
    constexpr int KSTEPS = D / 32, DT = D / 16;
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;

    uint2 *rows = reinterpret_cast<uint2 *>(smem + C::OFF_ROWS);
    int seg = (int)(block / (uint32_t)own_chunks), c = (int)(block % (uint32_t)own_chunks);
    if (!OWN) {
        // the list this chunk belongs to: the last seg with seg_chunk[seg] <= block (scalar binary search)
        const int segs = g.Hkv * g.N;
        const uint32_t b = block;
        if (b >= seg_chunk[segs]) return;
        int lo = 0, hi = segs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (seg_chunk[mid] <= b) lo = mid;
            else hi = mid - 1;
        }
        seg = lo;
        c = (int)(b - seg_chunk[seg]);
    }
    const int j = seg % g.N, kv = seg / g.N;
    if (OWN && mode_flag[FLAG_KV + kv] != 3) return;  // (the lists of such a head are empty)
    const int jsize = __builtin_amdgcn_readfirstlane(g.ragged ? csize[j] : g.Cmax);
    const CubeBox jbox = cube_box(g, j);  // (OWN) the rows
    // this workgroup's rows: positions [first, first + nrows) of the work list, or all rows of cube j
    uint32_t first = 0;
    int nrows;
    if (OWN) {
        first = (uint32_t)c * PAIRS_CHUNK;
        nrows = min(g.G * jsize - (int)first, PAIRS_CHUNK);
        if (nrows <= 0) return;
    } else {
        const uint32_t count = seg_count[seg];
        first = seg_start[seg] + (uint32_t)c * PAIRS_CHUNK;
        nrows = (int)min(count - (uint32_t)c * PAIRS_CHUNK, (uint32_t)PAIRS_CHUNK);
    }
    nrows = __builtin_amdgcn_readfirstlane(nrows);
    const int nsteps = (nrows + C::ROWS - 1) / C::ROWS;
    const int nt = (jsize + KEY_TILE - 1) / KEY_TILE;  // 1 .. PAIRS_MAX_TPC

    // ---- the key cube's tiles: global -> LDS, all wavefronts
    {
        const size_t cube_off = ((size_t)kv * g.N + j) * g.TPC * C::CHUNK;
        const unsigned char *kbase = reinterpret_cast<const unsigned char *>(Kp) + cube_off;
        const unsigned char *vbase = reinterpret_cast<const unsigned char *>(Vt) + cube_off;
        const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
        const int per = nt * C::PIECES;  // 1 KB pieces of K, and of V^T
        for (int p = wave; p < 2 * per; p += WAVES) {
            const bool isv = p >= per;
            const int q = isv ? p - per : p;  // = tile * PIECES + piece: the tiles of a cube are contiguous in memory
            // wave-uniform by construction; said again so that they are kept in scalar registers
            const uint32_t dst = __builtin_amdgcn_readfirstlane(
                lds0 + (uint32_t)((isv ? C::OFF_V : C::OFF_K) + (q / C::PIECES) * C::TILE_STRIDE + (q % C::PIECES) * 1024));
            const unsigned char *src = reinterpret_cast<const unsigned char *>(isv ? vbase : kbase) + (size_t)q * 1024;
            dma_1k_s(dst, uniform_ptr(src), (uint32_t)(lane * 16));
        }
    }

    fill_masks_init(smem + C::OFF_FILL, tid);
    // ---- the workgroup's rows as (row id, record) in LDS: a piece of the work list, or (OWN) rows of cube j in
    // (rank, head) order with the own cube's record, which is the row's last
    for (int x = tid; x < nrows; x += C::THREADS) {
        if (OWN) {
            const int idx = (int)first + x;
            const uint32_t rid = (uint32_t)(token_of(g, jbox, idx / g.G) * g.Hq + kv * g.G + idx % g.G);
            rows[x] = make_uint2(rid, (uint32_t)(pair_ptr[rid + 1] - 1));
        } else {
            rows[x] = *reinterpret_cast<const uint2 *>(entries + 2 * (size_t)(first + x));
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tiles (direct-to-LDS loads) and the rows
    __syncthreads();

    // ---- the Q operands run a step ahead of the MFMAs
    struct RowIds {
        uint32_t rid[NS], slot[NS];
        int lim[NS];  // last key (rank in cube j) the row attends
    };
    auto ids_of = [&](int step, RowIds &r) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int idx = min(step * C::ROWS + 16 * s + n16, nrows - 1);  // padding rows repeat the last one
            const uint2 e = rows[idx];
            r.rid[s] = e.x;
            r.slot[s] = e.y;
            r.lim[s] = OWN ? ((int)first + idx) / g.G : jsize - 1;
        }
    };
    auto q_of = [&](const RowIds &r, bf16x8 (&q)[NS][KSTEPS]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const uint16_t *qrow = Q + (size_t)r.rid[s] * D + 8 * q4;
#pragma unroll
            for (int k = 0; k < KSTEPS; ++k) q[s][k] = *reinterpret_cast<const bf16x8 *>(qrow + 32 * k);
        }
    };
    // A step: 32 rows (ids: their row ids and records, q: their Q operands) through the cube's tiles; then the
    // buffers are refilled for step `refill`, two of this wavefront's steps ahead, and the records are written.
    // The loop below alternates between two sets of buffers, so that what is loaded here is read only after the
    // other set's step: no register copies, and the wait for these loads (which, the counter being in order, is
    // also a wait for the older stores) finds everything long done.
    auto run_step = [&](RowIds &ids, bf16x8 (&qf)[NS][KSTEPS], int step, int refill) __attribute__((always_inline)) {
        // (the scores start from minus the reference point of the exponentials: softmax_tile_folded)
        float m_run[NS];
        bool fresh[NS];
        f32x4 l_run[NS], sinit[NS];
        f32x4 oacc[NS][DT];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            m_run[s] = 0.f;
            fresh[s] = true;
            l_run[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < DT; ++e) oacc[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        f32x4 sacc[NS][4];
        bf16x8 pf[NS][2];
        bf16x8 ring[PF];
        // (OWN) rows come in rank order: no row of the step attends keys past the rank of its last row
        int nts = nt;
        if (OWN) nts = min(nt, ((int)first + min(step * C::ROWS + C::ROWS, nrows) - 1) / g.G / KEY_TILE + 1);
        auto k_tile = [&](int t) -> const unsigned char * { return smem + C::OFF_K + t * C::TILE_STRIDE; };
        auto v_tile = [&](int t) -> const unsigned char * { return smem + C::OFF_V + t * C::TILE_STRIDE; };
        auto softmax_step = [&](int t) __attribute__((always_inline)) {
            const int key0 = KEY_TILE * t;
            const int fill = jsize - key0;
            // (after a step's first tile every row has its reference point: fresh is false for all)
            if (OWN || !softmax_tile_fast<NS>(sacc, pf, t > 0, smem + C::OFF_FILL, fill, q4))
                softmax_tile_folded<D, NS>(sacc, pf, oacc, m_run, l_run, fresh, ids.lim, key0, OWN || fill < KEY_TILE, q4);
#pragma unroll
            for (int s = 0; s < NS; ++s) sinit[s] = f32x4{-m_run[s], -m_run[s], -m_run[s], -m_run[s]};
        };
#pragma unroll
        for (int s = 0; s < NS; ++s) sinit[s] = f32x4{0.f, 0.f, 0.f, 0.f};
        phase_prefetch<D, PF, false, true>(nullptr, k_tile(0), n16, q4, ring);
        mfma_phase_from<D, NS, PF, false, true>(nullptr, k_tile(0), n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);
        softmax_step(0);
        for (int t = 1; t < nts; ++t) {
            phase_prefetch<D, PF, true, true>(v_tile(t - 1), k_tile(t), n16, q4, ring);
            mfma_phase_from<D, NS, PF, true, true>(v_tile(t - 1), k_tile(t), n16, q4, ring, pf, oacc, l_run, qf, sinit,
                                                   sacc);
            softmax_step(t);
        }
        phase_prefetch<D, PF, true, false>(v_tile(nts - 1), nullptr, n16, q4, ring);
        mfma_phase_from<D, NS, PF, true, false>(v_tile(nts - 1), nullptr, n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);

        uint32_t slot[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) slot[s] = ids.slot[s];
        ids_of(refill, ids);
        q_of(ids, qf);
        // The records: m, l, s = max |O| and O / s in fp16 (round toward zero).  A lane holds 4 consecutive head-dim
        // elements per block of 16; two blocks make one 16-byte store.  Straight-line code, so that the stores are
        // counted exactly and the wait for the operands loaded above does not become a wait for them: a padding
        // row repeats the step's last row and writes the same record with the same values again.
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            float amax = 0.f;
#pragma unroll
            for (int e = 0; e < DT; ++e)
#pragma unroll
                for (int v = 0; v < 4; ++v) amax = vmax(amax, fabsf(oacc[s][e][v]));
            amax = vmax(quad_max(amax), 1e-30f);
            const float inv = 1.0f / amax;
            uint16_t *orec = rec + (size_t)slot[s] * D + 8 * q4;
#pragma unroll
            for (int e = 0; e < DT; e += 2) {
                typedef __fp16 h2 __attribute__((ext_vector_type(2)));
                union { h2 h[4]; u32x4 u; } pk;
                pk.h[0] = __builtin_amdgcn_cvt_pkrtz(oacc[s][e][0] * inv, oacc[s][e][1] * inv);
                pk.h[1] = __builtin_amdgcn_cvt_pkrtz(oacc[s][e][2] * inv, oacc[s][e][3] * inv);
                pk.h[2] = __builtin_amdgcn_cvt_pkrtz(oacc[s][e + 1][0] * inv, oacc[s][e + 1][1] * inv);
                pk.h[3] = __builtin_amdgcn_cvt_pkrtz(oacc[s][e + 1][2] * inv, oacc[s][e + 1][3] * inv);
                // written once, read once by the merge kernel: streaming stores
                __builtin_nontemporal_store(pk.u, reinterpret_cast<u32x4 *>(orec + 16 * e));
            }
            // the four lanes of a row write one of the four scalars each
            ml[(size_t)slot[s] * 4 + q4] = q4 == 0 ? m_run[s] : q4 == 1 ? l_run[s][0] : q4 == 2 ? amax : 0.f;
        }
    };

    // This wavefront's steps are wave, wave + WAVES, ...; even ones use buffer set A, odd ones set B.  Past the end
    // a step index is clamped to the last step: that step is then done again -- by this wavefront, and possibly by
    // other wavefronts of the workgroup at the same time -- and every such repetition writes the same records.
    // The duplicates are benign because they are bit-identical: a step's result depends only on its rows' Q, the
    // cube's tiles and a fixed instruction sequence (no atomics, no data-dependent order), so concurrent writers
    // store the same bytes to the same addresses.  Everything in the loop stays unconditional (a guarded store
    // would make the compiler merge its wait counts with the operand loads').  The tests that force this kernel
    // run geometries whose step counts are not multiples of the wavefront count, so the repeated step is covered.
    if (wave >= nsteps) return;
    const int last = nsteps - 1;
    RowIds ids_a{}, ids_b{};
    bf16x8 q_a[NS][KSTEPS], q_b[NS][KSTEPS];
    ids_of(wave, ids_a);
    q_of(ids_a, q_a);
    ids_of(min(wave + WAVES, last), ids_b);
    q_of(ids_b, q_b);
    // vmcnt(0), as a builtin so that the compiler's own wait-count bookkeeping knows nothing is pending at the
    // loop's entry (through inline assembly it would not, and would wait at the loop's top, on every trip, for the
    // record stores of the trip before)
    __builtin_amdgcn_s_waitcnt(0x0F70);
    for (int step = wave; step < nsteps; step += 2 * WAVES) {
        run_step(ids_a, q_a, step, min(step + 2 * WAVES, last));
        run_step(ids_b, q_b, min(step + WAVES, last), min(step + 3 * WAVES, last));
    }
}

// The own cubes' workgroups first, then the lists' (as many as could be; those past the last chunk return at once).
template <int D>
__global__ __launch_bounds__(FWD_MAX_THREADS) void attn_pairs_kernel(
    Geom g, int own_chunks, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kp, const uint16_t *__restrict__ Vt,
    const int32_t *__restrict__ csize, const int64_t *__restrict__ pair_ptr, const uint32_t *__restrict__ seg_count,
    const uint32_t *__restrict__ seg_start, const uint32_t *__restrict__ seg_chunk, const uint32_t *__restrict__ entries,
    const int *__restrict__ mode_flag, uint16_t *__restrict__ rec, float *__restrict__ ml)
{
    if (!mode_flag[FLAG_ACTIVE]) return;
    const uint32_t own = (uint32_t)(g.Hkv * g.N) * (uint32_t)own_chunks;
    if (blockIdx.x < own)
        attn_pairs_work<D, true>(blockIdx.x, g, own_chunks, Q, Kp, Vt, csize, pair_ptr, seg_count, seg_start, seg_chunk, entries,
                                 mode_flag, rec, ml);
    else
        attn_pairs_work<D, false>(blockIdx.x - own, g, 1, Q, Kp, Vt, csize, pair_ptr, seg_count, seg_start, seg_chunk, entries,
                                  mode_flag, rec, ml);
}

// D / 8 lanes per row: O = sum_k 2^(m_k - M) s_k h_k / sum_k 2^(m_k - M) l_k over the row's records (h = O / s in
// fp16), in one pass with a running maximum.  A lane owns the eight fp16 values at byte 16 * lane of a record: two blocks of
// four adjacent head-dim elements.  Bound by memory (a record once, 272 bytes at head-dim 128): 65,536 tokens of
// 28/4 heads, Top-p 0.5, 40.7 M records, 2.46 ms = 4.7 TB/s; four values and a 64-bit division per lane and row, 2.80.  30,000 tokens, half
// the heads with two records a row, 0.21 ms and 0.45.
template <int D>
__global__ __launch_bounds__(256) void pairs_merge_kernel(uint32_t S, const int64_t *__restrict__ pair_ptr,
                                                          const uint16_t *__restrict__ rec, const float *__restrict__ ml,
                                                          const int *__restrict__ mode_flag, int Hq, int G,
                                                          uint16_t *__restrict__ O, float *__restrict__ lse)
{
    constexpr int LPR = D / 8;  // lanes per row
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    const int a = blockIdx.y, l = threadIdx.x % LPR;
    if (!mode_flag[FLAG_ACTIVE] || mode_flag[FLAG_KV + a / G] != 3) return;  // (another kernel writes that head's rows)
    // grid-stride over the tokens: the grid is bounded, so that a launch that has nothing to do costs little
    for (uint32_t n = blockIdx.x * (256 / LPR) + threadIdx.x / LPR; n < S; n += gridDim.x * (256 / LPR)) {
        const size_t row = (size_t)n * Hq + a;
        const long long p0 = pair_ptr[row];
        const int count = (int)(pair_ptr[row + 1] - p0);
        const float *mlr = ml + (size_t)p0 * 4;
        const uint16_t *recr = rec + (size_t)p0 * D + 8 * l;
        float M = -INFINITY, L = 0.f;
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        constexpr int U = 4;  // records in flight per lane
        for (int k0 = 0; k0 < count; k0 += U) {
            f32x4 x[U];
            h8 h[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = min(k0 + u, count - 1);  // past the end: the last record again, with weight 0 below
                x[u] = *reinterpret_cast<const f32x4 *>(mlr + (size_t)k * 4);  // m, l, s
                h[u] = *reinterpret_cast<const h8 *>(recr + (size_t)k * D);
            }
            float mx = M;
#pragma unroll
            for (int u = 0; u < U; ++u) mx = fmaxf(mx, x[u][0]);
            const float scale = __builtin_amdgcn_exp2f(M - mx);  // 0 on the first trip (M = -inf)
            M = mx;
            L *= scale;
#pragma unroll
            for (int v = 0; v < 8; ++v) acc[v] *= scale;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float w = (k0 + u < count) ? __builtin_amdgcn_exp2f(x[u][0] - M) : 0.f;
                L = fmaf(w, x[u][1], L);
                const float ws = w * x[u][2];
#pragma unroll
                for (int v = 0; v < 8; ++v) acc[v] = fmaf(ws, (float)h[u][v], acc[v]);
            }
        }
        const float inv = 1.0f / L;
        // values 8 l .. 8 l + 7 of a record are elements 16 e + 4 q4 + 0..3 of e = 2 * (l / 4) and e + 1, q4 = l % 4
        uint16_t *o = O + row * D + 32 * (l / 4) + 4 * (l % 4);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const uint32_t w0 = (uint32_t)float_to_bf16_bits(acc[4 * e] * inv) | ((uint32_t)float_to_bf16_bits(acc[4 * e + 1] * inv) << 16);
            const uint32_t w1 = (uint32_t)float_to_bf16_bits(acc[4 * e + 2] * inv) | ((uint32_t)float_to_bf16_bits(acc[4 * e + 3] * inv) << 16);
            *reinterpret_cast<uint2 *>(o + 16 * e) = make_uint2(w0, w1);
        }
        if (lse != nullptr && l == 0) lse[row] = (M + log2f(L)) * 0.69314718055994530942f;
    }
}

// Number of candidate (row, cube) pairs: every row of cube i has i preceding cubes.  In closed form: the entry points ask a few times
// a call, and over 2,048 cubes one by one it took 15 us each time.
unsigned long long candidate_pairs(const Geom &g)
{
    typedef unsigned long long u64;
    // sum over the blocks b of `len` things cut by `by` of b * (things of block b)
    auto weighted = [](int len, int by) -> u64 {
        const u64 n = ((u64)len + by - 1) / by;
        return n == 0 ? 0 : (n - 1) * (n - 2) / 2 * by + (n - 1) * (len - (n - 1) * by);
    };
    const u64 T = g.T, H = g.H, W = g.W;
    u64 c = weighted(g.Sp, g.Cmax) + (u64)g.Np * g.Sv;                       // the text before the video, and the video behind it
    c += weighted(g.T, g.ct) * H * W * g.nHb * g.nWb + T * weighted(g.H, g.ch) * W * g.nWb + T * H * weighted(g.W, g.cw);
    c += weighted(g.St, g.Cmax) + (u64)(g.Np + g.Nv) * g.St;
    return c * (unsigned long long)g.Hq;
}

template <int D>
static hipError_t launch_pairs_d(const Geom &g, const void *packed, const PairsScratch &sc,
                                 const int *flag, uint16_t *O, float *lse, hipStream_t st)
{
    using C = Pairs<D>;
    const uint16_t *Kp = reinterpret_cast<const uint16_t *>(packed);
    const size_t half_elems = (size_t)g.Hkv * g.N * g.TPC * KEY_TILE * D;
    const uint16_t *Vt = Kp + half_elems;
    const int32_t *csize = reinterpret_cast<const int32_t *>(Vt + half_elems);
    static LdsOptIn opted;  // one per kernel instantiation
    const hipError_t e = opted.ensure(reinterpret_cast<const void *>(&attn_pairs_kernel<D>), C::BYTES);
    if (e != hipSuccess) return e;
    // Chunks of all lists together: at most one partly filled chunk per list, and no more entries than records fit
    // (or than there are candidate pairs).  Workgroups past the actual number of chunks return at once.
    const long long segs = (long long)g.Hkv * g.N;
    const long long most = (long long)std::min<unsigned long long>((unsigned long long)sc.cap, candidate_pairs(g));
    const long long chunks = most / PAIRS_CHUNK + segs;
    const int own_chunks = (g.G * g.Cmax + PAIRS_CHUNK - 1) / PAIRS_CHUNK;
    hipLaunchKernelGGL((attn_pairs_kernel<D>), dim3((unsigned)(segs * own_chunks + chunks)), dim3(C::THREADS), C::BYTES, st, g,
                       own_chunks, sc.qs, Kp, Vt, csize, sc.pair_ptr, sc.seg_count, sc.seg_start, sc.seg_chunk, sc.entries, flag,
                       sc.rec, sc.ml);
    constexpr int rows_per_block = 256 / (D / 8);
    const unsigned merge_blocks = (unsigned)std::min<long long>((g.S + rows_per_block - 1) / rows_per_block,
                                                                std::max(1, 256 * 64 / g.Hq));
    hipLaunchKernelGGL((pairs_merge_kernel<D>), dim3(merge_blocks, g.Hq), dim3(256), 0, st, (uint32_t)g.S, sc.pair_ptr, sc.rec,
                       sc.ml, flag, g.Hq, g.G, O, lse);
    return hipGetLastError();
}

int *pairs_flags(const Geom &g, void *scratch, size_t scratch_bytes)
{
    if (!pairs_supported(g)) return nullptr;
    const PairsScratch sc = pairs_layout(g, scratch, scratch_bytes);
    return sc.cap > 0 ? sc.flags : nullptr;
}

long long pairs_capacity(const Geom &g, void *scratch, size_t scratch_bytes)
{
    return pairs_layout(g, scratch, scratch_bytes).cap;
}

uint32_t *pairs_counters(const Geom &g, void *scratch, size_t scratch_bytes, int &words)
{
    const PairsScratch sc = pairs_layout(g, scratch, scratch_bytes);
    words = sc.cap > 0 ? (int)(sc.seg_chunk - sc.seg_count) : 0;
    return sc.seg_count;
}

// Counts the pairs per KV head, hands heads to this path (flags), numbers their records, and enqueues this path's
// kernels (they return at once for heads, or altogether, when nothing was handed over).
hipError_t launch_attn_pairs(const Geom &g, const uint16_t *Q, const void *packed, const uint32_t *sel_mask, void *scratch,
                             size_t scratch_bytes, int force, int together, int pairs_below_permille, uint16_t *O,
                             float *lse, hipStream_t st)
{
    const PairsScratch sc = pairs_layout(g, scratch, scratch_bytes);
    if (!pairs_supported(g) || sc.cap <= 0) return hipErrorInvalidValue;
    int *flag = sc.flags;
    const uint32_t R = (uint32_t)((long long)g.S * g.Hq);  // (below 2^31: the entry points check)
    const int segs = g.Hkv * g.N, tiles = (int)pairs_tiles(g);
    static LdsOptIn opted;  // (with the most lists the counters take 64 KB)
    hipError_t e = opted.ensure(reinterpret_cast<const void *>(&pair_fill_kernel), PAIRS_MAX_SEGMENTS * 8);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(pair_count_kernel, dim3(tiles), dim3(PAIRS_TILE), (size_t)segs * 4, st, g, R, sel_mask, sc.cnt,
                       sc.seg_count, sc.tile_need, flag, force, pairs_below_permille);
    hipLaunchKernelGGL(pairs_plan_kernel, dim3(1), dim3(PAIRS_TILE), 0, st, g, sc.cap,
                       candidate_pairs(g) / (unsigned long long)g.Hkv, tiles, sc.tile_need, sc.seg_count, sc.tile_off,
                       sc.seg_start, sc.seg_chunk, flag, force, together, pairs_below_permille);
    hipLaunchKernelGGL(pair_fill_kernel, dim3(tiles), dim3(PAIRS_TILE), (size_t)segs * 8, st, g, R,
                       1.44269504088896340736f / sqrtf((float)g.D), Q, sel_mask, sc.cnt, sc.tile_off, flag, sc.seg_start,
                       sc.seg_cursor, sc.pair_ptr, sc.entries, sc.qs);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return g.D == 64 ? launch_pairs_d<64>(g, packed, sc, flag, O, lse, st)
                     : launch_pairs_d<128>(g, packed, sc, flag, O, lse, st);
}

}  // namespace adaspark
