// Dense causal attention, and sparse attention (Eq. 3 + own-cube rule, Sec. 3.2) with the selection applied as a
// mask: every row walks every preceding cube.  Also the entry that chooses between this kernel and the
// others (attn_split.hip, attn_compact.hip, attn_pairs.hip).
//
// Fixed-row walk with two wavefront sets in counter-phase.
//
// On a SIMD an MFMA keeps the matrix pipe busy for ~16 cycles, and vector instructions of another wavefront can
// issue underneath it; a wavefront alone cannot use that room, because its softmax needs its finished scores.  So
// a workgroup holds eight wavefronts, two per SIMD, and the two of a SIMD take the two halves of a tile's work in
// opposite order.  Per tile t every wavefront runs one MFMA phase -- P.V of tile t-1, then S = Q.K^T of tile t --
// and one softmax; set X (wavefronts 0-3) runs the MFMA phase first and the softmax of tile t after it, set Y (4-7)
// first runs the softmax of tile t-1 (one tile late) and then the MFMA phase:
//
//   slot t:   X: [P.V(t-1), S(t)]  softmax(t)
//             Y: softmax(t-1)      [P.V(t-1), S(t)]
//
// so that one wavefront's softmax runs under the other's MFMAs, with one workgroup barrier per tile.
//
// K and V^T tiles go through three LDS stages each (tile t in stage t % 3).  Slot t reads K(t) and V(t-1); after
// the barrier that opens it nobody reads K(t-1) or V(t-2) any more, and the direct-to-LDS loads of K(t+2) and
// V(t+1) go into their stages; they are waited for two barriers later (the loads started one tile ago may stay in
// flight).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "attn_tile.h"

namespace adaspark {

template <int D>
struct Walk {
    static constexpr int WAVES = 8;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int NS = FWD_NS;
    static constexpr int MMAX = 16 * NS * WAVES;  // 256 rows per workgroup
    static constexpr int NST = 3;  // LDS stages of K and of V^T
    static constexpr int PF = 4;   // operand loads in flight ahead of the MFMAs
    static constexpr int CHUNK = KEY_TILE * D * 2;
    static constexpr int DMA = CHUNK / 1024 / WAVES;
    static constexpr int SMALL = (((MMAX + 1) * 4 + 15) / 16) * 16;
    static constexpr int OFF_K = 0;
    static constexpr int OFF_V = OFF_K + NST * CHUNK;
    static constexpr int OFF_ROWID = OFF_V + NST * CHUNK;
    static constexpr int OFF_RANK = OFF_ROWID + SMALL;
    static constexpr int OFF_OWN = OFF_RANK + SMALL;
    static constexpr int OFF_MISC = OFF_OWN + SMALL;
    static constexpr int OFF_FILL = OFF_MISC + 16;  // fill_masks
    // the cubes of the walk (sparse entry: those that some row of the workgroup attends; union of the rows' mask words), in
    // order, each with its size
    static constexpr int LIST_MAX = ADASPARK_MAX_CUBES;
    static constexpr int OFF_UNION = OFF_FILL + FILL_MASK_BYTES;
    static constexpr int OFF_LIST = OFF_UNION + LIST_MAX / 8;
    static constexpr int BYTES = OFF_LIST + LIST_MAX * 8;
    static_assert(DMA >= 1, "a tile is at least 1 KB per wavefront");
    static_assert(BYTES <= 160 * 1024, "LDS of one CU");
};


// Barrier that opens a slot: all direct-to-LDS loads but the newest KEEP of this wavefront have landed.  Nothing
// waits for LDS reads here: the operand reads of a slot are consumed by its MFMAs before the wavefront gets here.
template <int KEEP>
__device__ __forceinline__ void dma_barrier()
{
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(KEEP) : "memory");
}

// Blocks of 256 rows that follow each other on one XCD: as many as a whole cube fills.
__host__ __device__ inline int walk_group(const Geom &g) { return max(1, g.G * g.Cmax / Walk<64>::MMAX); }

// SMALL: no cube has more than 32 tokens, and every tile is worked as its first half; the other half held no keys, and its score
// products, exponentials and output products were a third of a step.  (This kernel, us, whole tiles and half: cubes of 32, 4,032 tokens
// of 6/2 heads of 128 222, 157; 8,064 of 28/4 840, 586; 8/2 of 64 367, 266.)
template <int D, bool MASKED, bool SMALL = false>
__global__ __launch_bounds__(FWD_MAX_THREADS) void attn_walk_kernel(
    Geom g, const uint16_t *__restrict__ Q, const uint16_t *__restrict__ Kp, const uint16_t *__restrict__ Vt,
    const int32_t *__restrict__ csize, const uint32_t *__restrict__ sel_mask, const int *__restrict__ mode_flag,
    int my_mode, int kv_modes, uint16_t *__restrict__ O, float *__restrict__ lse)
{
    if (mode_flag != nullptr && mode_flag[FLAG_MODE] != my_mode) return;
    using C = Walk<D>;
    constexpr int NS = C::NS, MMAX = C::MMAX, THREADS = C::THREADS, WAVES = C::WAVES, NST = C::NST;
    constexpr int KSTEPS = D / 32, DT = D / 16;
    constexpr int PF = C::PF;
    constexpr int KG = SMALL ? 2 : 4;                             // groups of 16 keys of a tile that are worked
    constexpr int DMA_K = SMALL && C::DMA == 2 ? 1 : C::DMA;      // loads of a K tile (SMALL: of its first half), per wavefront
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    int *rowid = reinterpret_cast<int *>(smem + C::OFF_ROWID);
    int *rrank = reinterpret_cast<int *>(smem + C::OFF_RANK);
    int *rown = reinterpret_cast<int *>(smem + C::OFF_OWN);  // the row's own cube
    int *misc = reinterpret_cast<int *>(smem + C::OFF_MISC);

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n16 = lane & 15, q4 = lane >> 4;
    const bool set_y = __builtin_amdgcn_readfirstlane(wave >> 2) != 0;

    // workgroup -> (KV head, block of 256 rows).  A KV head's rows are numbered cube by cube (row = cube's first row +
    // head-in-group * tokens + rank, so a block's rows are neighbouring tokens of one query head or two, the rows most
    // likely to select the same cubes) and cut into blocks from the last row on, across the cubes' borders: on a grid
    // that the cubes do not divide, or with cubes of few rows, a workgroup per cube would leave a part of its 256 rows
    // empty and still walk every cube before.  (A forward pass, us, with blocks across cubes and short steps for tiles with
    // padding keys, and with neither: 30,000 tokens of 32/8 heads of 128 in cubes of 112 to 256 tokens 4,906, 5,784; 76,302
    // tokens of 8/2 heads of 64 in cubes of 4 to 256 tokens 14,630, 43,400; 51,763 of 14/2 of 128 in cubes of 12 to 256: 10,030, 12,800.)
    // The blocks of as many rows as a whole cube has follow each other on the same XCD: they stream the same tiles.
    const int nrows = g.S * g.G, nblk = (nrows - 1) / MMAX + 1, per_group = walk_group(g);
    const int groups = (nblk + per_group - 1) / per_group;  // of one KV head
    const int xcd = blockIdx.x & 7, seq = blockIdx.x >> 3;
    // The KV heads whose rows are this kernel's: all, or those that the key-stationary kernel did not get.
    int heads = g.Hkv;
    unsigned long long mine = ~0ull;  // (of up to PAIRS_MAX_KV_HEADS, where some are not)
    if (kv_modes && mode_flag[FLAG_ACTIVE]) {
        mine = __ballot((int)(threadIdx.x & 63) < g.Hkv && mode_flag[FLAG_KV + min((int)(threadIdx.x & 63), g.Hkv - 1)] != 3);
        heads = __popcll(mine);
        if (heads == 0) return;
    }
    // Late rows, the long walks, first, and a round of eight groups (one per XCD) behind the other.  A head normally stays on the same
    // XCDs (group % 8 = xcd: its K/V tiles are the ones that XCD's L2 holds).  With fewer than eight heads a round holds several groups
    // of a head, one behind the other; every second round deals them out in the opposite order, or the XCDs that
    // always got the later group would finish last (a forward pass over 16,384 tokens, 28/4 heads of 128: 1.650 ms, without this
    // 1.667; over 8,736 in 36 cubes 0.591, 0.596; runs of one side differ by 0.2 %.  30,000 tokens of 32/8 heads, four of them this
    // kernel's: 3.16 ms with the heads rotated over the XCDs instead, which ended between 2.89 and 3.16.)  Where neither is a
    // multiple of the other, the XCDs themselves take turns at head-dim 128.  (This kernel, us, with turns and without: 16,384 tokens of 12/3 heads 653,
    // 667; 30,720 of 20/5 3,536, 3,565; 20,480 of 28/7 2,251, 2,275; 12,288 of 21/3 655, 651.  24,576 of 28/4, three of them its, the same; five and three
    // of 32/8 0.3 and 0.6 % slower with turns.  Head-dim 64: 20,480 of 12/12 769, 754; 16,384 of 10/5 460, 452.)
    const int round = seq / per_group;
    int grp = round * 8 + xcd;
    if (D == 128 && 8 % heads != 0 && heads % 8 != 0 && (round & 1)) grp = round * 8 + 7 - xcd;
    if (grp >= groups * heads) return;
    int kv = grp % heads;
    int pos = grp / heads;
    const int share = 8 % heads == 0 ? 8 / heads : 1, turn = pos / share;
    if (8 % heads == 0 && (turn & 1) && (turn + 1) * share <= groups) pos = (2 * turn + 1) * share - 1 - pos;
    if (heads < g.Hkv) {  // the kv-th of the heads that remain
        const int lane = threadIdx.x & 63;
        const bool it = ((mine >> lane) & 1ull) && __popcll(mine & ((1ull << lane) - 1ull)) == kv;
        kv = __ffsll(__ballot(it)) - 1;
    }
    kv = __builtin_amdgcn_readfirstlane(kv);
    const int blk = pos * per_group + seq % per_group;
    if (blk >= nblk) return;
    const int row1 = nrows - blk * MMAX, row0 = max(0, row1 - MMAX);
    const int Mrows = row1 - row0;

    for (int r = tid; r < Mrows; r += THREADS) {
        const RowAt at = row_at(g, kv, row0 + r);
        rowid[r] = at.id;
        rrank[r] = at.rank;
        rown[r] = at.cube;
        if (r == 0) {  // scratch row behind the padding columns of a partial slab
            rowid[MMAX] = at.id;
            rrank[MMAX] = 0;
            rown[MMAX] = at.cube;
        }
        if (r == Mrows - 1) misc[2] = block_max_rank(at, Mrows), misc[3] = at.size;
    }
    fill_masks_init(smem + C::OFF_FILL, tid);
    // Sparse entry: a cube that no row of the workgroup selected is left out of the walk altogether.  Rows that
    // select independently of each other leave no such cube; rows of neighbouring tokens with similar queries do.
    int2 *clist = reinterpret_cast<int2 *>(smem + C::OFF_LIST);
    uint32_t *uni = reinterpret_cast<uint32_t *>(smem + C::OFF_UNION);
    if (MASKED)
        for (int w = tid; w < g.words; w += THREADS) uni[w] = 0u;
    __syncthreads();
    // The last cube with rows here, and the first.  The walk ends, in cube i, behind the largest rank of the block's rows there
    // (non-causal mode: the whole own cubes, and it goes on over the cubes after them).
    const int i = __builtin_amdgcn_readfirstlane(rown[Mrows - 1]), i_first = __builtin_amdgcn_readfirstlane(rown[0]);
    const int own_keys = __builtin_amdgcn_readfirstlane(g.causal ? misc[2] + 1 : misc[3]);
    const int own_tiles = (own_keys + KEY_TILE - 1) / KEY_TILE;
    const int ncubes = g.causal ? i + 1 : g.N;
    const int wlim = (ncubes + 31) >> 5;  // mask words that hold cubes of the walk
    if (MASKED) {
        for (int x = tid; x < Mrows * wlim; x += THREADS) {
            const int r = x / wlim, w = x - r * wlim;
            const uint32_t m = sel_mask[(size_t)rowid[r] * g.words + w];
            if (m) atomicOr(&uni[w], m);
        }
        __syncthreads();
    }
    if (wave == 0) {  // in cube order; the rows' own cubes are always there
        int n = 0, tiles = 0;
        for (int c0 = 0; c0 < ncubes; c0 += 64) {
            const int c = c0 + lane;
            const bool in = c < ncubes && (!MASKED || (c >= i_first && c <= i) || ((uni[c >> 5] >> (c & 31)) & 1u));
            const unsigned long long b = __ballot(in);
            if (in) {
                const int size = g.ragged ? csize[c] : g.Cmax;
                clist[n + __popcll(b & ((1ull << lane) - 1ull))] = make_int2(c, size);
                tiles += c == i ? own_tiles : (size + KEY_TILE - 1) / KEY_TILE;
            }
            n += __popcll(b);
        }
        for (int off = 32; off > 0; off >>= 1) tiles += __shfl_xor(tiles, off, 64);
        if (lane == 0) {
            misc[0] = tiles;
            misc[1] = n;
        }
    }
    __syncthreads();
    const int ntiles = __builtin_amdgcn_readfirstlane(misc[0]);
    const int nlist = __builtin_amdgcn_readfirstlane(misc[1]);
    auto cube_tiles = [&](int j, int size) -> int { return j == i ? own_tiles : (size + KEY_TILE - 1) / KEY_TILE; };
    // The list entry after position k, fetched when position k is entered and used a whole cube later: the LDS
    // read is long over by then (read and used at the same cube boundary, its latency showed in every stream).
    auto peek_after = [&](int k) -> int2 { return clist[min(k + 1, nlist - 1)]; };  // past the end: any valid cube

    // the tile whose softmax comes next
    int cc_j = __builtin_amdgcn_readfirstlane(clist[0].x), cc_size = __builtin_amdgcn_readfirstlane(clist[0].y);
    int cc_t = 0, cc_nt = cube_tiles(cc_j, cc_size), cc_k = 0;
    int2 cc_next = peek_after(0);
    // The K and V^T tiles are fetched in the same order, V^T one tile behind K: one stream walks the list of cubes
    // (cubes are padded to TPC tiles in memory; a ragged cube's padding tiles are skipped) and yields the byte
    // offset of its current tile from the KV head's first tile, which is the same in the K and the V^T half of the
    // packed copy; the V^T load of a slot takes the offset the K load of the slot before it used.  (Two independent
    // streams cost twice the scalar registers and instructions, and this kernel has none to spare: what does not
    // fit is kept in lanes of a vector register and read back with vector instructions.)
    struct Stream {
        uint32_t off;  // of the current tile
        int k, t, nt;  // position in the list of cubes, tile in the cube, tiles of the cube
        int2 next;     // the list's entry at position k + 1 (per lane, as read)
    };
    const unsigned char *khead = reinterpret_cast<const unsigned char *>(Kp + (size_t)kv * g.N * g.TPC * (KEY_TILE * D));
    const unsigned char *vhead = reinterpret_cast<const unsigned char *>(Vt + (size_t)kv * g.N * g.TPC * (KEY_TILE * D));
    auto stream_begin = [&]() -> Stream {
        Stream q;
        q.k = 0;
        q.off = (uint32_t)cc_j * (uint32_t)(g.TPC * C::CHUNK);
        q.t = 0;
        q.nt = cc_nt;
        q.next = peek_after(0);
        return q;
    };
    auto stream_next = [&](Stream &q) __attribute__((always_inline)) {
        if (q.t + 1 < q.nt) {
            ++q.t;
            q.off += C::CHUNK;
        } else {
            q.k = min(q.k + 1, nlist - 1);  // past the end nothing is issued; the index only has to stay valid
            const int j = __builtin_amdgcn_readfirstlane(q.next.x), size = __builtin_amdgcn_readfirstlane(q.next.y);
            q.next = peek_after(q.k);
            q.off = (uint32_t)j * (uint32_t)(g.TPC * C::CHUNK);
            q.t = 0;
            q.nt = cube_tiles(j, size);
        }
    };
    const uint32_t lds_piece =
        __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + (uint32_t)(wave * C::DMA * 1024));
    const uint32_t src_piece = (uint32_t)(wave * C::DMA * 1024 + lane * 16);
    auto issue = [&](const unsigned char *head, uint32_t off, int off_bytes) __attribute__((always_inline)) {
        const void *tile = uniform_ptr(head + off);
#pragma unroll
        for (int u = 0; u < C::DMA; ++u)
            dma_1k_s(lds_piece + (uint32_t)(off_bytes + u * 1024), tile, src_piece + (uint32_t)(u * 1024));
    };
    auto issue_k = [&](uint32_t off, int off_bytes) __attribute__((always_inline)) {
        if constexpr (DMA_K == C::DMA) {
            issue(khead, off, off_bytes);
        } else {
            const uint32_t piece = (uint32_t)(wave * DMA_K * 1024);  // of the tile's first half
            dma_1k_s(__builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + piece) + (uint32_t)off_bytes,
                     uniform_ptr(khead + off), piece + (uint32_t)(lane * 16));
        }
    };
    auto next_stage = [](int st) -> int { return st + 1 == NST ? 0 : st + 1; };

    // rows of this wavefront: slab k of the block belongs to wavefront k % WAVES as its slot k / WAVES
    int lr[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int idx = 16 * (wave + WAVES * s) + n16;
        lr[s] = idx < Mrows ? idx : MMAX;
    }
    // the wavefront's rows: lowest rank, first and last own cube (without rows: those of the padding columns)
    int rank_lo = 0x7fffffff, own_lo = 0x7fffffff, own_hi = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (s == 0 || lr[s] != MMAX) {
            rank_lo = min(rank_lo, rrank[lr[s]]);
            own_lo = min(own_lo, rown[lr[s]]);
            own_hi = max(own_hi, rown[lr[s]]);
        }
    for (int off = 32; off > 0; off >>= 1) {
        rank_lo = min(rank_lo, __shfl_xor(rank_lo, off, 64));
        own_lo = min(own_lo, __shfl_xor(own_lo, off, 64));
        own_hi = max(own_hi, __shfl_xor(own_hi, off, 64));
    }
    own_lo = __builtin_amdgcn_readfirstlane(own_lo);
    own_hi = __builtin_amdgcn_readfirstlane(own_hi);
    rank_lo = __builtin_amdgcn_readfirstlane(own_lo == own_hi ? rank_lo : 0);

    // prologue: K(0), K(1), V(0)
    Stream sk = stream_begin();
    uint32_t klast = sk.off;  // offset of the K tile issued last
    issue_k(sk.off, C::OFF_K);  // (ntiles >= 1: the own cube has a tile)
    issue(vhead, sk.off, C::OFF_V);
    stream_next(sk);
    if (ntiles > 1) {
        klast = sk.off;
        issue_k(sk.off, C::OFF_K + C::CHUNK);
        stream_next(sk);
    }

    const float c2 = 1.44269504088896340736f / sqrtf((float)D);  // softmax scale in base 2, folded into Q
    bf16x8 qf[NS][KSTEPS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const uint16_t *qrow = Q + (size_t)rowid[lr[s]] * D + 8 * q4;
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c) qf[s][c] = score_operand(*reinterpret_cast<const bf16x8 *>(qrow + 32 * c), c2);
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c) asm volatile("" : "+v"(qf[s][c]));

    int lim[NS];
    float m_run[NS];
    bool fresh[NS];
    f32x4 l_run[NS];  // every element holds the row's running sum
    f32x4 oacc[NS][DT];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        m_run[s] = 0.f;   // reference point of the exponentials; set by the row's first tile (fresh)
        fresh[s] = true;
        l_run[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < DT; ++e) oacc[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bool rsel[NS];
    // The rows' mask words: the one in use, and the next one, fetched when the walk enters a word so that it has
    // long arrived when the walk gets there 32 cubes later (read and used at the same cube boundary, every
    // wavefront stood still for a memory latency once per 32 cubes).
    uint32_t mword[NS], mword_ahead[NS];
    int mword_idx = -1;
#pragma unroll
    for (int s = 0; s < NS; ++s) { rsel[s] = true; mword[s] = 0; mword_ahead[s] = 0; }
    if (MASKED) {
#pragma unroll
        for (int s = 0; s < NS; ++s) mword_ahead[s] = sel_mask[(size_t)rowid[lr[s]] * g.words];
    }
    // Wave-uniform: no row of the wavefront is without a reference point any more; no row that takes part in the cube is
    // (softmax_tile_fast may be tried).  Rows that select a cube or two are without one for most of their walk, and would
    // keep their wavefront on the long step (144,585 tokens of 14/2 heads of 128, one KV head's rows
    // selecting nearly nothing: 63.7 ms, with only the first condition 73.1).
    bool settled = false, short_step = false;
    auto references = [&]() __attribute__((always_inline)) {
        bool open = false, here = false;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            open = open || fresh[s];
            here = here || (fresh[s] && (!MASKED || rsel[s]));
        }
        settled = __ballot(open) == 0ull;
        short_step = __ballot(here) == 0ull;
    };
    // Per-cube constants of the softmax: key limits of every row, and (MASKED) whether the row attends the cube.  A row
    // attends its own cube up to its rank and no later one.
    auto enter_cube = [&](int j, int size) __attribute__((always_inline)) {
        if (MASKED) {
            if ((j >> 5) != mword_idx) {
                const bool ahead = (j >> 5) == mword_idx + 1;  // (the walk ascends; words can be skipped)
                mword_idx = j >> 5;
                const int nxt = min(mword_idx + 1, g.words - 1);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const uint32_t *mr = sel_mask + (size_t)rowid[lr[s]] * g.words;
                    mword[s] = ahead ? mword_ahead[s] : mr[mword_idx];
                    mword_ahead[s] = mr[nxt];
                }
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) rsel[s] = (mword[s] >> (j & 31)) & 1u;
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) lim[s] = size - 1;
        if (j >= own_lo) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int own = rown[lr[s]];
                if (MASKED) rsel[s] = j == own || (rsel[s] && (!g.causal || j < own));
                if (g.causal && j >= own) lim[s] = j == own ? min(rrank[lr[s]], size - 1) : -1;
            }
        }
        if (!settled) references();
    };
    auto advance = [&]() __attribute__((always_inline)) {
        if (cc_t + 1 < cc_nt) ++cc_t;
        else if (cc_k + 1 < nlist) {
            cc_j = __builtin_amdgcn_readfirstlane(cc_next.x);
            cc_size = __builtin_amdgcn_readfirstlane(cc_next.y);
            cc_next = peek_after(++cc_k);
            cc_t = 0;
            cc_nt = cube_tiles(cc_j, cc_size);
            enter_cube(cc_j, cc_size);
        }  // the last tile stays where it is: nothing is issued or computed past the end
    };
    enter_cube(cc_j, cc_size);

    f32x4 sacc[NS][4];
    bf16x8 pf[NS][2];
    // Writes the rows whose own cube lies before cube `behind`, once.  A row's probabilities of the cubes behind its own are zero, and
    // so is what they add to its O -- unless V is not finite there (0 * inf); so a row is written before the first product
    // with such a cube.  (K cannot leak: the packed copy is finite, attn_tile.h.)
    int written = 0;  // rows of the cubes before it are
    auto write_rows = [&](int behind) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (lr[s] == MMAX) continue;
            const int own = rown[lr[s]];
            if (own >= behind || own < written) continue;
            const int rid = rowid[lr[s]];
            const float inv = 1.0f / l_run[s][0];
            uint16_t *orow = O + (size_t)rid * D + 4 * q4;
#pragma unroll
            for (int e = 0; e < DT; ++e) {
                *reinterpret_cast<uint2 *>(orow + 16 * e) = pack_bf16(oacc[s][e] * inv);
            }
            if (lse != nullptr && q4 == 0) lse[rid] = (m_run[s] + log2f(l_run[s][0])) * 0.69314718055994530942f;
        }
    };
    // LATE: the tile may be of a cube behind some rows' own; if not, it is of one up to main_to.
    const int main_to = g.causal ? own_lo : 0x7fffffff;
    auto softmax_step = [&](auto late) __attribute__((always_inline)) {
        constexpr bool LATE = decltype(late)::value;
        const int key0 = KEY_TILE * cc_t;
        // the causal edge (of the sparse entry's rows, a cube behind the own one is just not selected); padding keys
        const bool edge = g.causal && cc_j >= own_lo && (MASKED ? cc_j <= own_hi : true) &&
                          (cc_j > own_lo || key0 + KEY_TILE - 1 > rank_lo);
        const int fill = cc_size - key0;
        if (edge || !softmax_tile_fast<NS, KG>(sacc, pf, short_step, smem + C::OFF_FILL, fill, q4)) {
            softmax_tile_folded<D, NS, KG>(sacc, pf, oacc, m_run, l_run, fresh, lim, key0, edge || fill < 16 * KG, q4);
            references();
        }
        if (LATE && g.causal && cc_j > own_lo) {  // (the product with this tile comes next)
            write_rows(cc_j);
            written = cc_j;
        }
        advance();
    };

    // what the scores of the next tile start from: minus the reference point of the row's exponentials, or -inf
    // for a row that did not select the tile's cube (its probabilities are then 0 and its state stays as it is)
    f32x4 sinit[NS];
    auto set_sinit = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float x = (MASKED && !rsel[s]) ? -INFINITY : -m_run[s];
            sinit[s] = f32x4{x, x, x, x};
        }
    };
    static_assert(NST == 3, "the stage arithmetic below is for three stages");
    int kst = 0;  // stage of K(t); V(t-1) sits in stage (kst + 2) % 3
    bf16x8 ring[PF];
    // Opens slot t.  The loads started after the previous barrier, K(t+1) and V(t), may stay in flight; everything
    // older has landed: K(t) and V(t-1).  Then K(t+2) and V(t+1) are started into the stages that fell free.
    auto open_slot = [&](int t) __attribute__((always_inline)) {
        if (t > 0 && t + 1 < ntiles) dma_barrier<C::DMA + DMA_K>();
        else dma_barrier<0>();
        const int st_v = kst == 0 ? 2 : kst - 1;  // (kst + 2) % 3: stage of V(t-1), and of K(t+2)
        const int st_n = kst == 2 ? 0 : kst + 1;  // (kst + 1) % 3: stage of V(t+1)
        if (t + 1 < ntiles)  // V^T(t+1): the tile K(t+1), whose offset the K load of the slot before this one used
            issue(vhead, klast, C::OFF_V + st_n * C::CHUNK);
        if (t + 2 < ntiles) {
            klast = sk.off;
            issue_k(sk.off, C::OFF_K + st_v * C::CHUNK);
            stream_next(sk);
        }
    };
    auto k_tile = [&]() -> const unsigned char * { return smem + C::OFF_K + kst * C::CHUNK; };
    auto v_tile = [&]() -> const unsigned char * { return smem + C::OFF_V + (kst == 0 ? 2 : kst - 1) * C::CHUNK; };
    // The first and the last slot are peeled off the loops: a loop body with a conditional MFMA phase would merge
    // two versions of every accumulator at its end, at the price of a register copy each.
    open_slot(0);
    phase_prefetch<D, PF, false, true, KG>(nullptr, k_tile(), n16, q4, ring);
    set_sinit();
    mfma_phase_from<D, NS, PF, false, true, KG>(nullptr, k_tile(), n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);
    // Each set's loop twice: up to the own cube of the wavefront's first row, and behind it (few tiles, and none where a block's
    // rows are of one cube).  As one loop that may write rows out in any step, 65,536 tokens of 28/4 heads took 1.2 % longer; so, 0.3 %
    // longer than without the early writes.
    const std::false_type early;
    const std::true_type late;
    int t = 1;
    if (!set_y) {
        auto slot = [&](auto when) __attribute__((always_inline)) {
            kst = next_stage(kst);
            open_slot(t);
            phase_prefetch<D, PF, true, true, KG>(v_tile(), k_tile(), n16, q4, ring);
            set_sinit();
            mfma_phase_from<D, NS, PF, true, true, KG>(v_tile(), k_tile(), n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);
            softmax_step(when);
        };
        softmax_step(early);
        for (; t < ntiles && cc_j <= main_to; ++t) slot(early);
        for (; t < ntiles; ++t) slot(late);
        kst = next_stage(kst);
        open_slot(ntiles);
    } else {
        auto slot = [&](auto when) __attribute__((always_inline)) {
            kst = next_stage(kst);
            open_slot(t);
            softmax_step(when);  // of tile t-1
            phase_prefetch<D, PF, true, true, KG>(v_tile(), k_tile(), n16, q4, ring);
            set_sinit();
            mfma_phase_from<D, NS, PF, true, true, KG>(v_tile(), k_tile(), n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);
        };
        for (; t < ntiles && cc_j <= main_to; ++t) slot(early);
        for (; t < ntiles; ++t) slot(late);
        kst = next_stage(kst);
        open_slot(ntiles);
        softmax_step(late);
    }
    phase_prefetch<D, PF, true, false, KG>(v_tile(), nullptr, n16, q4, ring);
    mfma_phase_from<D, NS, PF, true, false, KG>(v_tile(), nullptr, n16, q4, ring, pf, oacc, l_run, qf, sinit, sacc);

    // ---- the rest of the rows (no direct-to-LDS load may outlive the workgroup's LDS allocation)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    write_rows(0x7fffffff);
}

// ---- What the choice of kernel goes by, from samples; two workgroups, which write
//   0  the share of candidate cubes that the rows select, per KV head: flags[FLAG_MODE] = 1 (the other row-stationary kernel: an overall
//      share of up to other_permille) or 2 (masked walk), flags[FLAG_ESTIMATE] = the smallest share of a KV head in permille (together:
//      the largest), and (kv_modes) the heads' shares
//   1  flags[FLAG_UNION]; it also clears the per-head choices and the key-stationary path's counters
// (One workgroup that did both: 15 us at 9,000 tokens of 28/4 heads, 28 at 65,536; two 11 and 19, and 31 at 262,144.)
constexpr int DENSITY_THREADS = 1024;
constexpr int DENSITY_MAX_ROWS = 2048;  // two sampled rows per thread: an estimate is all that is needed
constexpr int DENSITY_GROUPS = 16;          // sampled blocks of rows for the union estimate
constexpr int DENSITY_UNION_WORDS = ADASPARK_MAX_CUBES / 32;
// Measured on MI355X with rows that select independently of each other: the compacting kernel wins only below
// about 1.5 % selected cubes.
constexpr int MASKED_ABOVE_PERMILLE = 15;

__global__ __launch_bounds__(DENSITY_THREADS) void sel_density_kernel(Geom g, const uint32_t *__restrict__ sel_mask,
                                                                      int *__restrict__ flags, int kv_modes, int together,
                                                                      int other_permille, uint32_t *__restrict__ counters, int counter_words)
{
    if (blockIdx.x == 0) {
        // selected, candidates (at most DENSITY_MAX_ROWS * ADASPARK_MAX_CUBES); heads beyond the array fold
        __shared__ uint32_t acc[2][PAIRS_MAX_KV_HEADS];
        for (int x = threadIdx.x; x < 2 * PAIRS_MAX_KV_HEADS; x += DENSITY_THREADS) (&acc[0][0])[x] = 0u;
        __syncthreads();
        // sample k: token (k * tstride) mod S, query head k mod Hq -- every head gets its share of the samples
        const int samples = (int)min((long long)DENSITY_MAX_ROWS, (long long)g.S * g.Hq);
        const int tstride = max(1, g.S / samples) | 1;
        for (int k = threadIdx.x; k < samples; k += DENSITY_THREADS) {
            // (k * tstride < S + DENSITY_MAX_ROWS, or below DENSITY_MAX_ROWS: 32 bits)
            const int n = (int)((uint32_t)k * (uint32_t)tstride % (uint32_t)g.S), a = k % g.Hq;
            const int i = cube_of_token(g, n);
            const uint32_t *mr = sel_mask + ((size_t)n * g.Hq + a) * g.words;
            uint32_t sel = 0;
#pragma unroll 4
            for (int w = 0; 32 * w < i; ++w) sel += __popc(mr[w]);
            const int kv = (a / g.G) % PAIRS_MAX_KV_HEADS;
            atomicAdd(&acc[0][kv], sel);
            atomicAdd(&acc[1][kv], (uint32_t)i);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            static_assert((unsigned long long)DENSITY_MAX_ROWS * ADASPARK_MAX_CUBES * 1000 < (1ull << 32), "permille in 32 bits");
            uint32_t sel = 0, cand = 0, least = 1000, most = 0;
            for (int kv = 0; kv < min(g.Hkv, PAIRS_MAX_KV_HEADS); ++kv) {
                sel += acc[0][kv];
                cand += acc[1][kv];
                if (acc[1][kv] == 0u) continue;
                const uint32_t share = acc[0][kv] * 1000u / acc[1][kv];
                least = min(least, share);
                most = max(most, share);
            }
            flags[FLAG_MODE] = other_permille >= 0 && sel * 1000u <= cand * (uint32_t)other_permille ? 1 : 2;
            flags[FLAG_ESTIMATE] = (int)(together ? most : least);
        }
        if (kv_modes)
            for (int kv = threadIdx.x; kv < g.Hkv; kv += DENSITY_THREADS)
                flags[FLAG_SHARE + kv] = acc[1][kv] > 0u ? (int)(acc[0][kv] * 1000u / acc[1][kv]) : 0;
        return;
    }
    for (int x = threadIdx.x; x < counter_words; x += DENSITY_THREADS) counters[x] = 0u;
    if (threadIdx.x == 0) flags[FLAG_ACTIVE] = 0;
    if (kv_modes)
        for (int kv = threadIdx.x; kv < g.Hkv; kv += DENSITY_THREADS) flags[FLAG_KV + kv] = 0;
    // What the masked walk cannot leave out: the share of the cubes before a block of its rows that some row of the block selected
    // or is in, over DENSITY_GROUPS sampled (block, KV head) pairs, one per wavefront, all at once.
    static_assert(DENSITY_THREADS / 64 == DENSITY_GROUPS, "one sampled block per wavefront");
    __shared__ uint32_t uni[DENSITY_GROUPS][DENSITY_UNION_WORDS];
    __shared__ uint32_t ucount[2];  // cubes in the unions, cubes before the blocks
    if (threadIdx.x < 2) ucount[threadIdx.x] = 0u;
    const int k = threadIdx.x >> 6, t = threadIdx.x & 63;
    const bool measured = g.causal != 0;
    // late blocks weigh most, as in the walk, and the blocks of a whole cube (of its query heads) take turns
    const int nrows = g.S * g.G, nblk = (nrows - 1) / Walk<64>::MMAX + 1;
    const int blk = min((int)((long long)k * nblk / DENSITY_GROUPS) + k % walk_group(g), nblk - 1), kv = k % g.Hkv;
    const int row1 = nrows - blk * Walk<64>::MMAX, row0 = max(0, row1 - Walk<64>::MMAX);
    // every second row, from the last one: each is a cache line of its own, and one CU fetches them all
    RowAt at[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) at[q] = row_at(g, kv, max(row1 - 1 - 2 * (64 * q + t), row0));
    const int i = __builtin_amdgcn_readfirstlane(at[0].cube), i_first = __builtin_amdgcn_readlane(at[1].cube, 63);
    const int wlim = (i + 31) >> 5;
    if (measured)
        for (int w = t; w < wlim; w += 64) uni[k][w] = 0u;
    __syncthreads();
    if (measured) {
        const uint32_t *mr[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) mr[q] = sel_mask + (size_t)at[q].id * g.words;
        for (int w0 = 0; w0 < wlim; w0 += 8) {  // 2 rows x 8 words in flight per lane, then combined
            uint32_t m[2][8];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int u = 0; u < 8; ++u) m[q][u] = w0 + u < wlim ? mr[q][w0 + u] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                uint32_t x = m[0][u] | m[1][u];
                for (int off = 32; off > 0; off >>= 1) x |= __shfl_xor(x, off, 64);
                if (t == 0 && x) uni[k][w0 + u] |= x;  // the wavefront owns this row of `uni`
            }
        }
    }
    __syncthreads();
    if (measured) {
        uint32_t n = 0;
        for (int w = t; w < wlim; w += 64) {
            const uint32_t own = w < (i_first >> 5) ? 0u : w > (i_first >> 5) ? ~0u : ~0u << (i_first & 31);
            n += __popc((uni[k][w] | own) & (w == (i >> 5) ? (1u << (i & 31)) - 1u : ~0u));
        }
        if (n) atomicAdd(&ucount[0], n);
        if (t == 0) atomicAdd(&ucount[1], (uint32_t)i);
    }
    __syncthreads();
    if (threadIdx.x == 0)
        flags[FLAG_UNION] = ucount[1] > 0u ? max(1, (int)(ucount[0] * 1000u / ucount[1])) : 1000;
}

template <int D, bool MASKED>
static hipError_t launch_walk(const Geom &g, const uint16_t *Q, const void *packed, const uint32_t *sel_mask,
                              const int *mode_flag, int my_mode, int kv_modes, uint16_t *O, float *lse, hipStream_t st)
{
    using C = Walk<D>;
    if (g.N > C::LIST_MAX) return hipErrorInvalidValue;  // the kernel's cube list is that long (the entry points check)
    const uint16_t *Kp = reinterpret_cast<const uint16_t *>(packed);
    const size_t half_elems = (size_t)g.Hkv * g.N * g.TPC * KEY_TILE * D;
    const uint16_t *Vt = Kp + half_elems;
    const int32_t *csize = reinterpret_cast<const int32_t *>(Vt + half_elems);
    const int per_group = walk_group(g), nblk = (g.S * g.G - 1) / C::MMAX + 1;
    const int groups = (nblk + per_group - 1) / per_group;
    const dim3 grid((unsigned)((size_t)(((long long)groups * g.Hkv + 7) / 8) * per_group * 8));
    auto launch = [&](auto small) -> hipError_t {
        constexpr bool SMALL = decltype(small)::value;
        static LdsOptIn opted;  // one per kernel instantiation
        const hipError_t e = opted.ensure(reinterpret_cast<const void *>(&attn_walk_kernel<D, MASKED, SMALL>), C::BYTES);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((attn_walk_kernel<D, MASKED, SMALL>), grid, dim3(C::THREADS), C::BYTES, st, g, Q, Kp, Vt, csize,
                           sel_mask, mode_flag, my_mode, kv_modes, O, lse);
        return hipGetLastError();
    };
    return g.Cmax <= KEY_TILE / 2 ? launch(std::true_type{}) : launch(std::false_type{});
}

// Below this many candidate (row, cube) pairs the automatic choice is the masked walk outright (see launch_attn_d).
constexpr unsigned long long AUTO_MIN_CANDIDATE_PAIRS = 2ull << 20;

// The walks of a launch over the longest one, where every CU takes the same share (1.18: they do not).
static double walk_rounds(const Geom &g)
{
    return 1.18 * (g.causal ? 0.5 : 1.0) * g.Hkv * std::ceil((double)g.S * g.G / 256) / 256;
}

// Whether the automatic choice is made on the device.
static bool chosen_on_device(const Geom &g) { return candidate_pairs(g) >= AUTO_MIN_CANDIDATE_PAIRS; }

// Whether it is then made for all KV heads together.  Where the time of the masked walk is that of its longest walk, heads that go to
// the key-stationary kernel do not shorten it, unless all of them go (3,600 tokens of 28/4 heads of 128 in cubes of 32, half the
// heads selecting nearly nothing: the walk 202 us with all heads; with half of them, and the others by that kernel, 295).  With room for the
// key-stationary kernel, up to 1.2: a fifth of the walk is less than that kernel's share takes.  (Attention of as many heads that
// select nearly nothing as of others, us, one by one and together, by rounds of the walk: 14/2 heads of 128 in cubes of 256, 9,216 tokens,
// 1.16, 367, 293; 8/2 of 64, 14,336, 1.03, 384, 299; 28/4 in cubes of 32, 4,032, 1.02, 303, 218; 4,752, 1.20, 343, 283; 6/2 in cubes of 128,
// 19,008, 1.03, 589, 507; 22,464, 1.22, 684, 680.)
static bool heads_together(const Geom &g, bool room) { return walk_rounds(g) <= (room ? 1.2 : 1.0); }

// Tiles of `keys` keys that all cubes together take.  The cubes of a grid come in eight sizes (clipped or not along each
// axis), text cubes in two.
long long tiles_of_cubes(const Geom &g, int keys)
{
    auto tiles = [&](int tokens) { return (long long)(tokens + keys - 1) / keys; };
    long long n = (long long)(g.Sp / g.Cmax + g.St / g.Cmax) * tiles(g.Cmax) + tiles(g.Sp % g.Cmax) + tiles(g.St % g.Cmax);
    for (int clip = 0; clip < 8; ++clip) {
        const int et = clip & 1 ? g.T % g.ct : g.ct, eh = clip & 2 ? g.H % g.ch : g.ch, ew = clip & 4 ? g.W % g.cw : g.cw;
        const int nt = clip & 1 ? 1 : g.T / g.ct, nh = clip & 2 ? 1 : g.H / g.ch, nw = clip & 4 ? 1 : g.W / g.cw;
        n += (long long)nt * nh * nw * tiles(et * eh * ew);
    }
    return n;
}

// Whether the kernel for short sequences (attn_split.hip) beats this one, from what each of them takes on an MI355X (us).
// Fitted to 161 shapes of 460 to 16,384 tokens, heads 4/4 .. 32/8 of 64 and 128, cubes of 32 to 256 tokens, whole and clipped,
// with and without text; the figures below are 5 % (walk) and 6 % (split) off on average and pick the faster kernel but for
// two shapes, 4 and 6 % slower.
//   walk   a slot (64 keys past 256 rows) takes 1.19 at head-dim 64 and 1.62 at 128; the time is the longest walk's slots,
//          or all slots over 256 CUs where that is more.  In cubes of up to 32 tokens a slot is half the keys: 1.16 with most cubes
//          selected and 1.4 with few at head-dim 128, taken as 1.3 where selections of few cubes have another kernel to go to; where
//          they do not, and at head-dim 64, the line above stays (2,016 tokens of 28/4 heads, 62, 18 and 5 % selected, a forward
//          pass: 126, 136, 147 walk, 143, 144, 131 split)
//   split  a step (32 keys past 32 rows) takes a CU 0.15 and 0.24 -- what its operands take from L2 -- and a workgroup
//          7 to start and to combine its parts
// Measured on both sides of the line: 8,192 tokens of 4/4 heads of 64 in cubes of 128: 113 split, 155 walk; 16,384: 396, 303.
// 2,048 tokens of 14/2 heads of 128 in cubes of 256: 62, 59; 4,096: 156, 105.
//   choice  where this kernel would be one of those chosen from on the device, the launches of that choice count as 40 (20 to 25 with two of
//          them gone; the line was
//          fitted with 40 and is left where selections of few cubes, which the split takes in less time, lie near it)
static double walk_time(const Geom &g, bool choice)
{
    const double slot = g.D == 64 ? 1.19 : choice && g.Cmax <= KEY_TILE / 2 ? 1.3 : 1.62;
    return 11 + slot * (double)tiles_of_cubes(g, KEY_TILE) * std::max(1.0, walk_rounds(g));
}

// What the split takes, and of that what grows with the steps it visits.
static double split_time(const Geom &g, double &of_steps)
{
    const double share = g.causal ? 0.5 : 1.0;  // of all cubes that the average walk visits
    const double steps = (double)tiles_of_cubes(g, 32), blocks = g.Hkv * std::ceil((double)g.S * g.G / 32);
    of_steps = blocks / 256 * share * steps * (g.D == 64 ? 0.15 : 0.24);
    return 5 + 7 * std::max(1.0, blocks / 256) + of_steps;
}

bool attn_split_pays(const Geom &g, bool choice)
{
    double of_steps;
    choice = choice && chosen_on_device(g);
    return attn_split_fits(g) && split_time(g, of_steps) < walk_time(g, choice) + (choice ? 40 : 0);
}

// Up to which share of selected candidate cubes (permille) the split beats the walk where it does not at any share: it leaves
// out what none of 32 rows selected, rows that select independently (1 - share)^32 of the cubes.  The walk, in cubes of up to 32 tokens at
// head-dim 128 and with few of them selected, takes 57 and 1.155 a tile, the launches of the choice included (within 4 % over eight shapes of
// 2,816 to 15,360 tokens, 96 to 480 tiles); 65 because the share is one of rows from the first 60 to 100 % of the tokens, and few cubes are a larger share
// of the candidates there.  Chosen so, us, split and walk on either side of the line: 7,680 tokens of 14/2 heads of 128 in cubes of 32, 2.5 % selected
// 314, 334, 3.3 % 348, 339; 3,600 of 28/4, 1.7 % 181, 191, 3.3 % 218, 210; 2,816, 4.5 % 161, 167, 6.7 % 174, 163; 15,360 of 6/2, 4.9 % 588,
// 616, 6.6 % 640, 613, 61 % 763, 585.
static int split_below_permille(const Geom &g)
{
    if (!attn_split_fits(g)) return -1;
    double of_steps;
    const double walk = g.D == 128 && g.Cmax <= KEY_TILE / 2 ? 65 + 1.155 * (double)tiles_of_cubes(g, KEY_TILE) * std::max(1.0, walk_rounds(g))
                                                             : walk_time(g, false);
    const double all = split_time(g, of_steps), visited = 1.0 - (all - walk) / of_steps;
    return visited <= 0.0 ? -1 : (int)(1000.0 * (1.0 - std::pow(std::max(0.0, 1.0 - visited), 1.0 / 32)));
}

// The key-stationary kernel is the faster one below this share of selected candidate cubes.  The walk takes time by the
// tiles of a cube, 0.03 ns a candidate pair and tile at head-dim 128; a selected pair costs the other path 0.22 ns in cubes of one tile and
// 0.24 in cubes of four, most of it its record.  (Measured: 65,536 tokens of 28/4 heads in cubes of 256, break-even at 44 %;
// 7,688 tokens in cubes of 32, 32 % selected, 1,665 us against 583; 8,640 on a grid of 9 x 10, where cubes of up to 256 have 1.75 tiles on
// average, 33 % selected, 874 against 575, 18 % 587, 598.)  With half a tile's keys to a step (no cube above 32 tokens) the walk takes 0.72 of that; at
// head-dim 64 the other path's records are half as long, and the line stays.  (At head-dim 128, the walk and the key-stationary kernel by
// the share selected: 8,064 tokens, 28/4 heads, 13.6 % 624, 858, 10.6 % 628, 691, 9.3 % 645, 640; 14/2, 13.6 % 324, 469, 10.6 % 327, 387;
// 12,000, 14/2, 10.2 % 717, 707; 32/8, 13.1 % 1,460, 2,109, 8.7 % 1,501, 1,530.  KV heads on both sides of the line take both kernels, and that
// costs more than either near it: at 90, 7 % over 24 such shapes of 10 %, none slower at 110.  At 64: 8,064, 8/2, 16.5 % 265, 216.)
static int pairs_below_permille(const Geom &g)
{
    if (g.Cmax <= KEY_TILE / 2 && g.D == 128) return 110;
    return (int)(60 + 85 * tiles_of_cubes(g, KEY_TILE) / g.N);
}

template <int D>
static hipError_t launch_attn_d(const Geom &g, const uint16_t *Q, void *packed, const uint32_t *sel_mask,
                                int sparse_kernel, void *scratch, size_t scratch_bytes, uint16_t *O, float *lse,
                                hipStream_t st)
{
    if ((sel_mask == nullptr || sparse_kernel == ADASPARK_SPARSE_AUTO) &&
        attn_split_pays(g, sel_mask != nullptr && g.causal))
        return launch_attn_split(g, Q, packed, sel_mask, nullptr, 0, O, lse, st);
    if (sel_mask == nullptr) return launch_walk<D, false>(g, Q, packed, nullptr, nullptr, 0, 0, O, lse, st);
    if (sparse_kernel == ADASPARK_SPARSE_COMPACT && g.causal)
        return launch_attn_compact(g, Q, packed, sel_mask, nullptr, 0, 0, O, lse, st);
    if (sparse_kernel == ADASPARK_SPARSE_MASKED || !g.causal)  // non-causal mode: the masked walk is the one kernel
        return launch_walk<D, true>(g, Q, packed, sel_mask, nullptr, 0, 0, O, lse, st);
    // Small problems (8,192 rows of 64 cubes, say) are bound by the latency from one dependent kernel to the next: the
    // kernels that measure the selection and prepare the other paths would cost more than any choice among them can win
    // back.  The masked walk is the one kernel then.
    if (sparse_kernel == ADASPARK_SPARSE_AUTO && !chosen_on_device(g))
        return launch_walk<D, true>(g, Q, packed, sel_mask, nullptr, 0, 0, O, lse, st);
    // Automatic (or the key-stationary kernel asked for): the choice is made on the device, every candidate kernel
    // is enqueued, and the workgroups of those not chosen return at once.  First the selected share from a sample
    // of rows: that decides between the two row-stationary kernels, and whether the exact count for the
    // key-stationary one is worth taking at all; with room for its tables the choice is then made per KV head.
    int *flags = pairs_flags(g, scratch, scratch_bytes);
    const int kv_modes = flags != nullptr;
    if (!kv_modes) {
        if (sparse_kernel == ADASPARK_SPARSE_PAIRS) return hipErrorInvalidValue;  // the entry point checks this first
        flags = reinterpret_cast<int *>(reinterpret_cast<char *>(packed) + attn_workspace_bytes(g) - 16);
    }
    // Heads together: the walk, or all of them by the key-stationary kernel; without room for that one, by the kernel for
    // short sequences.  (Attention, us, chosen so, by the walk and by the key-stationary kernel: 24,576 tokens of 4/4 heads of 64 in
    // cubes of 256, 63, 34 and 18 % selected: 474, 319, 220; 439, 441, 445; 489, 320, 221.  Never one of the latter two: a call of
    // these that selects much is 8 % faster, one that selects little 50 % slower.)
    // Room: for twice the records of a selection of MASKED_ABOVE_PERMILLE (the share is an estimate), and the rows' own.  With less, heads are
    // by themselves where heads_together says so without the key-stationary kernel.
    const bool room = kv_modes && pairs_capacity(g, scratch, scratch_bytes) >=
                                      (long long)(candidate_pairs(g) / 1000 * (2 * MASKED_ABOVE_PERMILLE)) + (long long)g.S * g.Hq;
    const bool together = sparse_kernel == ADASPARK_SPARSE_AUTO && heads_together(g, room);
    // Heads by themselves: the compacting kernel for a selection of up to MASKED_ABOVE_PERMILLE -- which the key-stationary kernel has
    // already, if there is room.
    const bool compact = !together && !room;
    const int other_permille = together ? (kv_modes ? -1 : split_below_permille(g)) : compact ? MASKED_ABOVE_PERMILLE : -1;
    if (together && !kv_modes && other_permille < 0) return launch_walk<D, true>(g, Q, packed, sel_mask, nullptr, 0, 0, O, lse, st);
    int counter_words = 0;
    uint32_t *counters = kv_modes ? pairs_counters(g, scratch, scratch_bytes, counter_words) : nullptr;
    hipLaunchKernelGGL(sel_density_kernel, dim3(2), dim3(DENSITY_THREADS), 0, st, g, sel_mask, flags, kv_modes, together,
                       other_permille, counters, counter_words);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (kv_modes) {
        e = launch_attn_pairs(g, Q, packed, sel_mask, scratch, scratch_bytes, sparse_kernel == ADASPARK_SPARSE_PAIRS, together,
                              pairs_below_permille(g), O, lse, st);
        if (e != hipSuccess) return e;
    }
    if (compact) e = launch_attn_compact(g, Q, packed, sel_mask, flags, 1, kv_modes, O, lse, st);
    else if (together && !kv_modes) e = launch_attn_split(g, Q, packed, sel_mask, flags, 1, O, lse, st);
    if (e != hipSuccess) return e;
    return launch_walk<D, true>(g, Q, packed, sel_mask, flags, 2, kv_modes, O, lse, st);
}

hipError_t launch_attn(const Geom &g, const uint16_t *Q, void *packed, const uint32_t *sel_mask, int sparse_kernel,
                       void *scratch, size_t scratch_bytes, uint16_t *O, float *lse, hipStream_t st)
{
    if (g.D == 64) return launch_attn_d<64>(g, Q, packed, sel_mask, sparse_kernel, scratch, scratch_bytes, O, lse, st);
    return launch_attn_d<128>(g, Q, packed, sel_mask, sparse_kernel, scratch, scratch_bytes, O, lse, st);
}

}  // namespace adaspark
