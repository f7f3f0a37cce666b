// Backward pass of cube-selective attention (Eq. 3 differentiated; the selected sets are constants).
//
// For a row r with attended keys A_r, scale c = 1/sqrt(D):  p = softmax(c q.k),  delta = dO.O,
//     dV_j += p_j dO,   dS_j = p_j (dO.v_j - delta),   dQ = c sum_j dS_j k_j,   dK_j += c dS_j q.
// p is rebuilt from the forward's log-sum-exp, so nothing of the forward's size is stored.  Two MFMA kernels, neither
// of which needs a transposition in registers or an atomic:
//   attn_bwd_dq_kernel   row-stationary (like the forward's masked walk): a wavefront keeps Q and dO of 32 rows as
//                        MFMA B operands, walks the key tiles of the cubes that some row of its block selected or is in, and
//                        accumulates dQ^T.
//                        S^T = K.Q^T, dP^T = V.dO^T, dQ^T += K^T.dS^T.  A row's selection bit for the key cube acts
//                        as a mask (dense work, like the forward's masked walk).
//   attn_bwd_dkv_kernel  key-stationary: a wavefront keeps K and V of 32 keys as B operands and accumulates dV^T and
//                        dK^T over the rows that selected the keys' cube -- only those: the rows' state is nothing but
//                        Q, dO and two floats, so rows are gathered into tiles, and the work follows the selection.
//                        S = Q.K^T, dP = dO.V^T, dV^T += dO^T.P, dK^T += Q^T.dS.
// The streamed tiles of the first come from packed, pre-swizzled copies (kvtile.h layouts) straight into LDS: K
// natural / V natural / K transposed per 64 keys (bwd_prep_kernel).  The second gathers rows of
// Q and dO as the caller holds them, and reads each tile in LDS both ways: rows as they are, and transposed
// (ds_read_b64_tr_b16).
// The score products take Q and K as they are (bf16 x bf16 -> fp32: exact products, so the rebuilt probabilities
// carry nothing but their own rounding, whatever the size of the scores) and their accumulators start from
// -lse * sqrt(D), -inf for a row that did not select the key cube: the accumulator times the softmax scale in base
// 2 is then the exponent of the probability, and the selection costs no instruction per score.  The dP accumulators
// start from minus delta.  bwd_prep_kernel leaves both start values per row.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "attn_tile.h"

namespace adaspark {

constexpr int BWD_THREADS = 512;
constexpr int BWD_ROWS = 256;   // rows (dQ kernel) or keys (dK/dV kernel) per workgroup: 8 wavefronts x 2 x 16
constexpr int DQ_SHARED_BLOCKS = 304;  // bwd_dq_waves
constexpr int SHARED_ROWS = 6000;     // dkv_shared
constexpr int SHARED_CUBE_ROWS = 384;
constexpr float BWD_LOG2E = 1.44269504088896340736f;

// How attn_bwd_dkv_kernel's work is cut.  A workgroup takes up to 256 keys (one of nkb key blocks) of one (key cube j, KV
// head) and the rows of `span` consecutive row cubes c * span .. that selected j (and cube j's own rows, if it is one
// of them).  Parts of the same keys are summed by bwd_reduce_kernel in a fixed order.  Parts (c, j) exist for
// c >= j / span; they are numbered span * c * (c + 1) / 2 + j, so the workgroups of one c, which gather the same rows
// at the same time, follow each other.
struct BwdParts {
    int span, nc;     // row cubes per part; ranges c
    int nkb, keys;    // key blocks per cube; keys of one, as the sums are held (a multiple of 32, 256 but for small cubes)
    long long parts;  // per (KV head, key block)
};
static BwdParts bwd_cut(const Geom &g, long long span)
{
    BwdParts p;
    p.nkb = (g.Cmax + BWD_ROWS - 1) / BWD_ROWS;
    p.keys = std::min(BWD_ROWS, (g.Cmax + 31) / 32 * 32);
    p.span = (int)span;
    p.nc = (g.N + p.span - 1) / p.span;
    p.parts = (long long)p.span * (p.nc - 1) * p.nc / 2 + g.N;
    return p;
}
static BwdParts bwd_parts(const Geom &g)
{
    // A part costs its two sums' trip through memory (256 keys x D x 8 bytes written and read: about what 450 gathered
    // rows of head-dim 128 cost to compute), so it should see some thousands of rows; but there should be a few parts
    // per CU to keep the chip even at the end, and more than about 8,000 of them only take up memory.
    const long long lists = (long long)g.Hkv * ((g.Cmax + BWD_ROWS - 1) / BWD_ROWS) * g.N;
    const long long want = (8192 + g.G * g.Cmax - 1) / (g.G * g.Cmax);
    const long long lo = lists * g.N / (2 * 8192);
    long long hi = std::max(1LL, lists * g.N / (2 * 1024));
    // Up to two parts per CU, and row cubes of few rows: one round of workgroups with twice the rows instead, which leaves
    // half the sums (a backward pass, us: 384 rows a cube, 1,080 tokens of 6/2 heads of 128: 92.0 against 94.5; 768 rows, 4,096
    // tokens: 211.6, 216.1; runs of one side differ by 0.1).  With more rows the longest part is what counts (1,024 rows, 8/2 heads of 64: 161, 158; 1,792
    // rows, 14/2 heads of 128: 314, 300; 28/4 heads, 2,560 tokens: 315, 274).
    const long long most = lists * (g.N + 1) / 2;
    if (most <= 512 && g.G * g.Cmax <= 768) hi = (most + 255) / 256;
    return bwd_cut(g, std::min((long long)g.N, std::max(1LL, std::max(lo, std::min(hi, want)))));
}
// (keys that have a single part are written where they belong, so with a single range there are no sums to hold)
static size_t bwd_part_bytes(const Geom &g, const BwdParts &p)
{
    return p.nc > 1 ? (size_t)g.Hkv * p.nkb * p.parts * 2 * p.keys * g.D * 4 : 0;
}

struct BwdWorkspace {
    uint16_t *Kn, *Vn, *Kt;  // packed copies (kvtile.h): K and V natural, K transposed
    int32_t *csize;          // [N] sizes of the cubes
    // -lse * sqrt(D) and -delta per row (what the score and dP products start from); entry [rows] belongs to the rows
    // that pad a tile: -inf, 0
    float *lse2, *delta;     // [S * Hq + 1]
    unsigned long long *colmask;  // [Hkv][N (key cube j)][N (row cube i)][tpcr]: bit k = row 64 t + k of cube i selects j (j < i)
    uint32_t *rowtab;        // [N][tpcr * 64]: row ids of the row tiles, KV head 0
    float *part;             // [Hkv][nkb][parts][2 (dV, dK)][cut.keys x D], in MFMA output order
    uint16_t *Q, *dO;        // copies of the caller's, if a gradient is written over one of them
    BwdParts cut;
    int tpcr;                // 64-row words per cube = ceil(Cmax * G / 64)
    size_t bytes;
};

// in_place: dQ, dK or dV lies over Q or dO, which the dK/dV kernel gathers from while gradients are being written, so the
// kernels read copies.  These take part of the sums' place (made at least as large as they are), and the sums are those of
// wider ranges: a backward pass with dQ over dO, 1,080 tokens of 6/2 heads of 128, 108 us against 92; 4,096 tokens, 275 against 212.
BwdWorkspace bwd_workspace(const Geom &g, void *ws, bool in_place)
{
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    BwdWorkspace w;
    unsigned char *p = static_cast<unsigned char *>(ws);
    w.tpcr = (g.Cmax * g.G + 63) / 64;
    w.cut = bwd_parts(g);
    const size_t rows = (size_t)g.S * g.Hq + 1;
    size_t off = 0;
    const size_t copy_bytes = (size_t)g.Hkv * g.N * g.TPC * KEY_TILE * g.D * sizeof(uint16_t);
    w.Kn = reinterpret_cast<uint16_t *>(p + off); off = up(off + copy_bytes);
    w.Vn = reinterpret_cast<uint16_t *>(p + off); off = up(off + copy_bytes);
    w.Kt = reinterpret_cast<uint16_t *>(p + off); off = up(off + copy_bytes);
    w.csize = reinterpret_cast<int32_t *>(p + off); off = up(off + (size_t)g.N * 4);
    w.lse2 = reinterpret_cast<float *>(p + off); off = up(off + rows * 4);
    w.delta = reinterpret_cast<float *>(p + off); off = up(off + rows * 4);
    w.colmask = reinterpret_cast<unsigned long long *>(p + off); off = up(off + (size_t)g.Hkv * g.N * g.N * w.tpcr * 8);
    w.rowtab = reinterpret_cast<uint32_t *>(p + off); off = up(off + (size_t)g.N * w.tpcr * 64 * 4);
    const size_t copy = up((size_t)g.S * g.Hq * g.D * 2), place = up(std::max(bwd_part_bytes(g, w.cut), 2 * copy));
    w.Q = reinterpret_cast<uint16_t *>(p + off);
    w.dO = reinterpret_cast<uint16_t *>(p + off + copy);
    w.part = reinterpret_cast<float *>(p + off + (in_place ? 2 * copy : 0));
    if (in_place)
        while (2 * copy + bwd_part_bytes(g, w.cut) > place) w.cut = bwd_cut(g, w.cut.span + 1);  // (a single range has no sums)
    w.bytes = off + place;
    return w;
}

size_t attn_bwd_workspace_bytes(const Geom &g) { return bwd_workspace(g, nullptr, false).bytes; }

// Workgroup -> (KV head, slot among the head's workgroups).  Consecutive workgroups go to different XCDs, each with
// its own L2; the workgroups of one KV head stream the same tiles, so where the head count allows a head's
// workgroups stay on as few XCDs as possible.  bwd_grid is the matching launch size.
__host__ __device__ inline bool bwd_head_slot(int b, int Hkv, int per_head, int &kv, int &slot)
{
    if (Hkv <= 8 && 8 % Hkv == 0) {
        const int x = b & 7, idx = b >> 3, share = 8 / Hkv;
        kv = x % Hkv;
        slot = idx * share + x / Hkv;
    } else if (Hkv % 8 == 0) {
        const int x = b & 7, idx = b >> 3, m = Hkv / 8;
        kv = x + 8 * (idx % m);
        slot = idx / m;
    } else {
        kv = b % Hkv;
        slot = b / Hkv;
    }
    return slot < per_head;
}
inline unsigned bwd_grid(int Hkv, int per_head)
{
    if (Hkv <= 8 && 8 % Hkv == 0) return (unsigned)((per_head + 8 / Hkv - 1) / (8 / Hkv) * 8);
    return (unsigned)per_head * (unsigned)Hkv;
}

// Direct-to-LDS copies with an address per lane: lane l moves the 16 (4) bytes at src to lds_addr + 16 * l (4 * l).
__device__ __forceinline__ void dma_lane16(uint32_t lds_addr, const void *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(src) : "memory", "m0");
}
__device__ __forceinline__ void dma_lane4(uint32_t lds_addr, const void *src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" ::"s"(lds_addr), "v"(src) : "memory", "m0");
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__global__ __launch_bounds__(256) void bwd_copy_rows_kernel(long long pieces, const uint4 *__restrict__ Q,
                                                            const uint4 *__restrict__ dO, uint4 *__restrict__ Qc,
                                                            uint4 *__restrict__ dOc)
{
    const long long x = (long long)blockIdx.x * 256 + threadIdx.x;
    if (x >= pieces) return;
    Qc[x] = Q[x];
    dOc[x] = dO[x];
}

// What the kernels below read, in one launch whose workgroups do one of three things (as four launches, 1,080 tokens of 6/2 heads of
// 128, a layer's training pass 135 us, and 127):
//   a tile of 64 keys   its packed copies, K and V natural and K transposed (kvtile.h); padding keys are zero
//   256 / (D / 8) rows  what their products start from: lse2 = -lse * sqrt(D), delta = -dO.O; entry [rows]: what padding rows
//                       start from
//   four row tiles      the selection bits transposed for the key-stationary kernel, a wavefront per (KV head, row cube i, row
//                       tile t): lane k holds the mask words of row 64 t + k (rank-major: row r of a cube is head r % G of rank
//                       r / G), a ballot per cube turns 64 rows' bits into one 64-bit word.  sel_mask == nullptr: every row
//                       selects every cube.  KV head 0 also leaves the row ids of the row tiles (those of KV head kv are
//                       kv * G higher).
struct BwdPrep {
    const uint16_t *K, *V, *O, *dO;
    const float *lse;
    const uint32_t *sel_mask;
    uint16_t *Kn, *Vn, *Kt;
    int32_t *csize;
    float *lse2, *delta;
    unsigned long long *colmask;
    uint32_t *rowtab;
    int tpcr;
    uint32_t mask_blocks, key_blocks;  // the first workgroups are row tiles', the next ones key tiles', the rest rows'
};
template <int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(Geom g, BwdPrep p)
{
    constexpr int CPR = D / 8;  // 16-byte pieces of a row
    __shared__ __attribute__((aligned(16))) uint16_t ks[KEY_TILE][D + 8];
    const int lane = threadIdx.x & 63;
    if (blockIdx.x < p.mask_blocks) {
        uint32_t x = blockIdx.x * 4 + (threadIdx.x >> 6);
        if (x >= (uint32_t)p.tpcr * (uint32_t)g.N * (uint32_t)g.Hkv) return;
        const int t = (int)(x % (uint32_t)p.tpcr);
        x /= (uint32_t)p.tpcr;
        const int i = (int)(x % (uint32_t)g.N), kv = (int)(x / (uint32_t)g.N);
        const CubeBox box = cube_box(g, i);
        const int r = 64 * t + lane;
        const bool valid = r < box.size() * g.G;
        const size_t rowid = valid ? (size_t)token_in_cube(g, box, r / g.G) * g.Hq + kv * g.G + r % g.G : 0;
        if (kv == 0) p.rowtab[((size_t)i * p.tpcr + t) * 64 + lane] = (uint32_t)rowid;
        for (int jw = 0; 32 * jw < i; ++jw) {
            const uint32_t word = valid ? (p.sel_mask != nullptr ? p.sel_mask[rowid * g.words + jw] : ~0u) : 0u;
            unsigned long long mine = 0ull;
#pragma unroll
            for (int b = 0; b < 32; ++b) {
                const unsigned long long bal = __ballot((word >> b) & 1u);
                if (lane == b) mine = bal;
            }
            const int j = 32 * jw + lane;
            if (lane < 32 && j < i) p.colmask[(((size_t)kv * g.N + j) * g.N + i) * p.tpcr + t] = mine;
        }
    } else if (blockIdx.x < p.mask_blocks + p.key_blocks) {
        uint32_t x = blockIdx.x - p.mask_blocks;
        const size_t tile_base = (size_t)x * (KEY_TILE * D);
        const int t = (int)(x % (uint32_t)g.TPC);
        x /= (uint32_t)g.TPC;
        const int c = (int)(x % (uint32_t)g.N), kv = (int)(x / (uint32_t)g.N);
        const CubeBox box = cube_box(g, c);
        const int size = box.size();
        if (t == 0 && kv == 0 && threadIdx.x == 0) p.csize[c] = size;
        for (int y = threadIdx.x; y < KEY_TILE * CPR; y += 256) {
            const int k = y / CPR, col = y % CPR, rank = KEY_TILE * t + k;
            uint4 kk = make_uint4(0, 0, 0, 0), vv = make_uint4(0, 0, 0, 0);
            if (rank < size) {
                const size_t src = ((size_t)token_in_cube(g, box, rank) * g.Hkv + kv) * D + col * 8;
                kk = *reinterpret_cast<const uint4 *>(p.K + src);
                vv = *reinterpret_cast<const uint4 *>(p.V + src);
            }
            *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(p.Kn + tile_base) + k_tile_off<D>(k, col)) = kk;
            *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(p.Vn + tile_base) + k_tile_off<D>(k, col)) = vv;
            *reinterpret_cast<uint4 *>(&ks[k][col * 8]) = kk;
        }
        __syncthreads();
        for (int y = threadIdx.x; y < D * (KEY_TILE / 8); y += 256) {
            const int d = y / (KEY_TILE / 8), kc = y % (KEY_TILE / 8);
            uint32_t w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[e] = (uint32_t)ks[kc * 8 + 2 * e][d] | ((uint32_t)ks[kc * 8 + 2 * e + 1][d] << 16);
            *reinterpret_cast<uint4 *>(reinterpret_cast<char *>(p.Kt + tile_base) + vt_tile_off(d, kc)) =
                make_uint4(w[0], w[1], w[2], w[3]);
        }
    } else {
        const long long rows = (long long)g.S * g.Hq;
        const long long r = ((long long)(blockIdx.x - p.mask_blocks - p.key_blocks) * 256 + threadIdx.x) / CPR;
        const int col = threadIdx.x % CPR;
        float part = 0.f;
        if (r < rows) {
            const uint4 gg = *reinterpret_cast<const uint4 *>(p.dO + r * D + col * 8);
            const uint4 oo = *reinterpret_cast<const uint4 *>(p.O + r * D + col * 8);
            const uint32_t gw[4] = {gg.x, gg.y, gg.z, gg.w}, ow[4] = {oo.x, oo.y, oo.z, oo.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                part = fmaf(__uint_as_float(gw[e] << 16), __uint_as_float(ow[e] << 16), part);
                part = fmaf(__uint_as_float(gw[e] & 0xffff0000u), __uint_as_float(ow[e] & 0xffff0000u), part);
            }
        }
#pragma unroll
        for (int d = CPR / 2; d >= 1; d >>= 1) part += __shfl_xor(part, d, 64);
        if (col == 0 && r <= rows) {
            p.lse2[r] = r < rows ? -p.lse[r] * sqrtf((float)D) : -INFINITY;  // = -(lse in base 2) / (softmax scale in base 2)
            p.delta[r] = -part;
        }
    }
}

// Half H of qk_tile: the products of a natural tile's rows 32 H .. 32 H + 31 with the B operands of NS slabs (OP:
// the operand type, bf16x8).  acc[s][k2][v] belongs to tile row 32 H + 8 q4 + 4 k2 + v.
// Working a tile in two halves keeps half as many accumulators alive.  The accumulators of slab s start from bias[s],
// a value of the slab's row (the lane's column): the products come out with it added.
template <int D, int NS, int H, typename OP>
__device__ __forceinline__ void nat_half_bias(const unsigned char *kt, int n16, int q4, const OP (&bf)[NS][D / 32],
                                              const float (&bias)[NS], f32x4 (&acc)[NS][2])
{
    f32x4 init[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) init[s] = f32x4{bias[s], bias[s], bias[s], bias[s]};
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
            const int krow = 32 * H + 8 * (n16 >> 2) + 4 * k2 + (n16 & 3);
            const OP af = *reinterpret_cast<const OP *>(kt + k_tile_off<D>(krow, 4 * c + q4));
#pragma unroll
            for (int s = 0; s < NS; ++s) acc[s][k2] = mfma16(af, bf[s][c], c == 0 ? init[s] : acc[s][k2]);
        }
}

// acc^T[d, n] += T[d, k] . B[k, n] over the entities k = 32 H .. 32 H + 31 of a tile, slabs 0..NS-1: T a transposed tile in
// LDS (rows = head-dim), B in registers in the operand order qk_tile's outputs pack into (bf[s][H] = entities
// 32 H + 8 q4 + 0..7).  DONE: slab s's column of this lane keeps its value where done[s].
template <int D, int NS, int H, bool DONE = false>
__device__ __forceinline__ void tn_half(const unsigned char *tt, int n16, int q4, const bf16x8 (&bf)[NS][2],
                                        f32x4 (&acc)[NS][D / 16], const bool *done = nullptr)
{
#pragma unroll
    for (int e = 0; e < D / 16; ++e) {
        const bf16x8 af = *reinterpret_cast<const bf16x8 *>(tt + vt_tile_off(16 * e + n16, 4 * H + q4));
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const f32x4 sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af, bf[s][H], acc[s][e], 0, 0, 0);
            acc[s][e] = DONE && done[s] ? acc[s][e] : sum;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// dQ: workgroup = 256 / KEYS rows of one KV head; late rows (the long walks) first.
// KEYS = 1: a wavefront per 32 rows.  KEYS = 2: two, wavefronts w and w + 4, each with half of every tile's keys; their
// sums are added through LDS at the end.  A tile takes a workgroup 1.5 us at head-dim 128 (its MFMAs and exponentials), and
// with few workgroups the longest walk is the kernel's time: half as long, over twice as many workgroups (bwd_dq_waves).
// SMALL (KEYS = 1): no cube has more than 32 tokens, every tile is worked as its first half, the other held no keys (a backward pass, us,
// whole and half: 5,940 tokens of 28/4 heads of 128 in cubes of 32 2,160, 1,839; 6,048 of 14/2 1,124, 937).
// ---------------------------------------------------------------------------------------------------------------
template <int D, bool MASKED, int KEYS, bool SMALL = false>
__global__ __launch_bounds__(BWD_THREADS) void attn_bwd_dq_kernel(Geom g, const uint16_t *__restrict__ Q,
                                                                  const uint16_t *__restrict__ dO,
                                                                  const uint16_t *__restrict__ Kn,
                                                                  const uint16_t *__restrict__ Vn,
                                                                  const uint16_t *__restrict__ Kt,
                                                                  const int32_t *__restrict__ csize,
                                                                  float *__restrict__ lse2p,
                                                                  const float *__restrict__ deltap,
                                                                  const uint32_t *__restrict__ sel_mask,
                                                                  uint16_t *__restrict__ dQ)
{
    constexpr int NS = 2, KSTEPS = D / 32, DT = D / 16;
    constexpr int ROWS = BWD_ROWS / KEYS;
    constexpr int TILE = 64 * D * 2;       // bytes of one tile
    constexpr int STAGE = 3 * TILE;        // K natural, V natural, K transposed
    constexpr int PIECES = TILE / 1024;    // 1 KB pieces per tile
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];

    int4 *place = reinterpret_cast<int4 *>(smem + 2 * STAGE);  // [BWD_ROWS] a row's own cube, its rank there, its id
    uint32_t *uni = reinterpret_cast<uint32_t *>(place + BWD_ROWS);
    uint16_t *clist = reinterpret_cast<uint16_t *>(uni + ADASPARK_MAX_CUBES / 32);  // the cubes of the walk
    int *nlist_s = reinterpret_cast<int *>(clist + ADASPARK_MAX_CUBES);

    // A KV head's rows are numbered cube by cube and in a cube head by head, and cut into blocks from the last row on, across
    // the cubes' borders, as in the forward's walk, and the cubes that no row of the block selected are left out.  (A layer's
    // training pass, us, with a workgroup's rows in one cube and all cubes before it walked, and so: 6,426 tokens of 32/8 heads
    // in cubes of up to 128 of which half the heads select few 2,235, 1,796; 6,805 tokens of 28/4 heads, neighbours' queries
    // alike, on a grid of 9 x 10 2,824, 2,178.)
    const int nrows = g.S * g.G;
    int kv, slot;
    if (!bwd_head_slot(blockIdx.x, g.Hkv, (nrows - 1) / ROWS + 1, kv, slot)) return;
    const int row1 = nrows - slot * ROWS, row0 = max(0, row1 - ROWS), last = row1 - 1;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n16 = lane & 15, q4 = lane >> 4;
    const int rgroup = wave & (8 / KEYS - 1), khalf = wave / (8 / KEYS);  // 32 rows of the workgroup; half of a tile's keys

    // the wavefront's rows: lane l works out row l % 32 (rows past the last one repeat it)
    const RowAt at = row_at(g, kv, min(row0 + rgroup * 32 + (lane & 31), last));
    if (lane < 32) place[rgroup * 32 + lane] = make_int4(at.cube, at.rank, at.id, 0);  // (KEYS == 2: the same twice)
    bool valid[NS];
    int rid[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        valid[s] = row0 + rgroup * 32 + s * 16 + n16 <= last;
        rid[s] = __shfl(at.id, 16 * s + n16, 64);
    }
    // The rows' first mask words (a row's words are shared out among the four lanes that hold it): asked for first, used
    // last.
    uint32_t mask0 = 0u;
    if (MASKED) {
        if (q4 < g.words) mask0 = sel_mask[(size_t)rid[0] * g.words + q4] | sel_mask[(size_t)rid[1] * g.words + q4];
        for (int w = tid; w < g.words; w += BWD_THREADS) uni[w] = 0u;
    }
    bf16x8 qf[NS][KSTEPS], gf[NS][KSTEPS];
    float lse2[NS], delta[NS], psum[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        psum[s] = 0.f;
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c) {
            qf[s][c] = *reinterpret_cast<const bf16x8 *>(Q + (size_t)rid[s] * D + 32 * c + 8 * q4);
            gf[s][c] = *reinterpret_cast<const bf16x8 *>(dO + (size_t)rid[s] * D + 32 * c + 8 * q4);
        }
        lse2[s] = lse2p[rid[s]];    // -lse * sqrt(D): what the score products start from
        delta[s] = deltap[rid[s]];  // minus delta: what the dP products start from
    }

    auto row_place = [&](int s) -> int4 { return place[rgroup * 32 + s * 16 + n16]; };
    const float c2 = BWD_LOG2E / sqrtf((float)D);  // softmax scale in base 2

    // tile stream: the cubes of the walk (clist), the tiles of each that hold keys
    const size_t head_tiles = (size_t)kv * g.N * g.TPC;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
    auto issue = [&](int stage, int j, int t) __attribute__((always_inline)) {
        const size_t toff = (head_tiles + (size_t)j * g.TPC + t) * (size_t)TILE;
        // every wavefront moves its eighth of each of the three tiles (the tile is a compile-time index: a run-time
        // choice among kernel arguments would be made through a table in scratch memory)
#pragma unroll
        for (int which = 0; which < 3; ++which)
#pragma unroll
            for (int u = 0; u < PIECES / 8; ++u) {
                const int sub = wave * (PIECES / 8) + u;
                const unsigned char *src =
                    reinterpret_cast<const unsigned char *>(which == 0 ? Kn : which == 1 ? Vn : Kt) + toff + sub * 1024;
                dma_1k_s(__builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(stage * STAGE + which * TILE + sub * 1024)),
                         uniform_ptr(src), (uint32_t)(lane * 16));
            }
    };

    // The walk: the rows' own cubes, and of those before them the ones that some row of the block selected.
    __syncthreads();
    // the last cube with rows here, and the first
    const int i = __builtin_amdgcn_readfirstlane(place[last - row0].x), i_first = __builtin_amdgcn_readfirstlane(place[0].x);
    if (MASKED) {
        if (mask0) atomicOr(&uni[q4], mask0);
        for (int w = q4 + 4; 32 * w <= i; w += 4) {
            const uint32_t m = sel_mask[(size_t)rid[0] * g.words + w] | sel_mask[(size_t)rid[1] * g.words + w];
            if (m) atomicOr(&uni[w], m);
        }
        __syncthreads();
    }
    if (wave == 0) {
        int n = 0;
        for (int c0 = 0; c0 <= i; c0 += 64) {
            const int c = c0 + lane;
            const bool in = c <= i && (!MASKED || c >= i_first || ((uni[c >> 5] >> (c & 31)) & 1u));
            const unsigned long long b = __ballot(in);
            if (in) clist[n + __popcll(b & ((1ull << lane) - 1ull))] = (uint16_t)c;
            n += __popcll(b);
        }
        if (lane == 0) *nlist_s = n;
    }
    __syncthreads();
    const int nlist = __builtin_amdgcn_readfirstlane(*nlist_s);
    auto entry = [&](int k) -> int { return clist[min(k, nlist - 1)]; };  // past the end: any valid cube
    auto tiles_of = [&](int j) { return (csize[j] + 63) >> 6; };

    f32x4 acc[NS][D / 16];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int e = 0; e < DT; ++e) acc[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    // (a list entry is read when the cube before it is entered: the LDS read is long over when it is used)
    int inext = entry(1);
    int ik = 0, ij = __builtin_amdgcn_readfirstlane(entry(0)), it = 0, int_ = tiles_of(ij);  // next tile to issue
    int issued = ij;  // cube of the tile issued last: where the walk goes on when it is through with its cube
    auto issue_next = [&](int stage) __attribute__((always_inline)) {
        if (ik >= nlist) return;
        issued = ij;
        issue(stage, ij, it);
        if (++it == int_) {
            ++ik;
            ij = __builtin_amdgcn_readfirstlane(inext);
            int_ = tiles_of(ij);
            inext = entry(ik + 1);
            it = 0;
        }
    };
    issue_next(0);
    int stage = 0;
    uint32_t mw[NS] = {0u, 0u};
    int mw_idx = -1;
    // BEHIND: a cube behind some rows' own.  These rows' probabilities are zero there, but K and V need not be finite: they
    // keep their sums.
    auto walk_cube = [&](auto behind) __attribute__((always_inline)) {
        constexpr bool BEHIND = decltype(behind)::value;
        const int j = issued, size_j = csize[j], nt = tiles_of(j);
        const bool late = j >= i_first;  // some rows' own cube, or behind it
        // What the score products start from: minus the row's log-sum-exp; -inf for a row that did not select cube
        // j, which then takes no part (probabilities 0).  lim: the last key the row attends.
        if (MASKED && (j >> 5) != mw_idx) {
            mw_idx = j >> 5;
#pragma unroll
            for (int s = 0; s < NS; ++s) mw[s] = sel_mask[(size_t)row_place(s).z * g.words + mw_idx];
        }
        float le[NS];
        int lim[NS];
        bool done[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            le[s] = lse2[s];
            lim[s] = size_j - 1;
            done[s] = false;
            if (MASKED && !((mw[s] >> (j & 31)) & 1u)) le[s] = -INFINITY;
            if (late) {
                const int4 at = row_place(s);
                if (j >= at.x) {
                    le[s] = lse2[s];
                    lim[s] = j == at.x ? at.y : -1;
                }
                done[s] = j > at.x;
            }
        }
        for (int t = 0; t < nt; ++t) {
            tile_barrier();
            issue_next(stage ^ 1);
            const unsigned char *kt = smem + stage * STAGE, *vt = kt + TILE, *ktt = vt + TILE;
            const bool edge = late || 64 * t + 64 > size_j;  // the own cubes' causal edge, padding keys: few tiles
            bf16x8 ds[NS][2];
            auto half = [&](auto hc) __attribute__((always_inline)) {
                constexpr int H = decltype(hc)::value;
                f32x4 sacc[NS][2], pacc[NS][2];
                nat_half_bias<D, NS, H>(kt, n16, q4, qf, le, sacc);
                nat_half_bias<D, NS, H>(vt, n16, q4, gf, delta, pacc);
                if (edge) {
                    int kb = 64 * t + 32 * H + 8 * q4;
                    asm volatile("" : "+v"(kb));
#pragma unroll
                    for (int s = 0; s < NS; ++s)
#pragma unroll
                        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int key = kb + 4 * k2 + v;
                                if (key > lim[s]) sacc[s][k2][v] = -INFINITY;
                            }
                }
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float p = __builtin_amdgcn_exp2f(sacc[s][k2][v] * c2);
                            psum[s] += p;
                            ds[s][H][4 * k2 + v] = (__bf16)(p * pacc[s][k2][v]);
                        }
            };
            if (SMALL) {
                half(std::integral_constant<int, 0>{});
                tn_half<D, NS, 0, BEHIND>(ktt, n16, q4, ds, acc, done);
            } else if (KEYS == 1) {
                half(std::integral_constant<int, 0>{});
                half(std::integral_constant<int, 1>{});
                tn_half<D, NS, 0, BEHIND>(ktt, n16, q4, ds, acc, done);
                tn_half<D, NS, 1, BEHIND>(ktt, n16, q4, ds, acc, done);
            } else if (khalf == 0) {
                half(std::integral_constant<int, 0>{});
                tn_half<D, NS, 0, BEHIND>(ktt, n16, q4, ds, acc, done);
            } else {
                half(std::integral_constant<int, 1>{});
                tn_half<D, NS, 1, BEHIND>(ktt, n16, q4, ds, acc, done);
            }
            stage ^= 1;
        }
    };
    int k = 0;
    for (; k < nlist && issued <= i_first; ++k) walk_cube(std::false_type{});
    for (; k < nlist; ++k) walk_cube(std::true_type{});
    if (KEYS == 2) {  // (no load is in flight: the last tile's were waited for)
        static_assert(KEYS == 1 || 4 * 64 * (NS * DT * 16 + NS * 4) <= 2 * STAGE, "the second half's sums fit the tiles' place");
        f32x4 *sums = reinterpret_cast<f32x4 *>(smem);              // [4][NS * DT][64]
        float *psums = reinterpret_cast<float *>(sums + 4 * NS * DT * 64);  // [4][NS][64]
        __syncthreads();
        if (khalf == 1) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
#pragma unroll
                for (int e = 0; e < DT; ++e) sums[((size_t)rgroup * (NS * DT) + s * DT + e) * 64 + lane] = acc[s][e];
                psums[(rgroup * NS + s) * 64 + lane] = psum[s];
            }
        }
        __syncthreads();
        if (khalf == 1) return;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int e = 0; e < DT; ++e) acc[s][e] += sums[((size_t)rgroup * (NS * DT) + s * DT + e) * 64 + lane];
            psum[s] += psums[(rgroup * NS + s) * 64 + lane];
        }
    }
    // The probabilities above were built from the caller's log-sum-exp, which the forward kernels give to about
    // 1e-3; their sum over the row says by how much it is off.  dQ is linear in them, so it is divided by the sum
    // here, and the log-sum-exp is corrected for the dK / dV kernel that runs next.
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const float total = quad_sum(psum[s]);
        if (!valid[s]) continue;
        const size_t rid = row_place(s).z;
        if (q4 == 0) lse2p[rid] = lse2[s] - log2f(total) / c2;
        const float scale = 1.0f / (sqrtf((float)D) * total);
#pragma unroll
        for (int e = 0; e < DT; ++e)
            *reinterpret_cast<uint2 *>(dQ + rid * D + 16 * e + 4 * q4) = pack_bf16(acc[s][e] * scale);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// dQ of short sequences: workgroup = 32 rows of one KV head, as in the forward's kernel for short sequences (attn_split.hip); its eight
// wavefronts take every eighth 32-key step of the walk, operands straight from the packed copies (they are in operand order, and nobody
// else on the CU wants the same ones), and their sums are added through LDS.
//
// Bound by the latency of a step (24 KB from L2, 48 MFMAs at head-dim 128, the next step's operands asked for as soon as this one's
// are used): its wavefronts wait for data 44 % of their time and for their turn another 36 %, the matrix pipes are busy 5 %, and it reads
// 138 MB from L2, 6.6 TB/s.  1,080 tokens of 6/2 heads of 128: 20 us, 46 with two wavefronts per 32 rows on 56 workgroups.  The rows' Q and dO are B operands of all steps and of all eight wavefronts: they lie in LDS, which leaves the registers
// to the operands in flight.
// ---------------------------------------------------------------------------------------------------------------
template <int D>
struct DqSplit {
    static constexpr int WAVES = BWD_THREADS / 64;
    static constexpr int NS = 2;
    static constexpr int ROWS = 16 * NS;
    static constexpr int STEP = 32;  // keys per step
    static constexpr int DT = D / 16, KSTEPS = D / 32;
    static constexpr int OFF_OPS = WAVES * NS * DT * 1024;             // behind the wavefronts' sums: Q and dO as operands
    static constexpr int OFF_PSUM = OFF_OPS + 2 * NS * KSTEPS * 1024;  // the wavefronts' sums of probabilities
    static constexpr int OFF_UNION = OFF_PSUM + WAVES * ROWS * 4;
    static constexpr int OFF_N = OFF_UNION + ADASPARK_MAX_CUBES / 8;
    static constexpr int BYTES = OFF_N + 16;
    static constexpr int LIST_MAX = OFF_OPS / 4;  // the list of steps lies where the sums go at the end
    static_assert(BYTES <= 160 * 1024, "LDS of one CU");
};

template <int D, bool MASKED>
__global__ __launch_bounds__(BWD_THREADS) void attn_bwd_dq_split_kernel(Geom g, const uint16_t *__restrict__ Q,
                                                                        const uint16_t *__restrict__ dO,
                                                                        const uint16_t *__restrict__ Kn,
                                                                        const uint16_t *__restrict__ Vn,
                                                                        const uint16_t *__restrict__ Kt,
                                                                        const int32_t *__restrict__ csize,
                                                                        float *__restrict__ lse2p,
                                                                        const float *__restrict__ deltap,
                                                                        const uint32_t *__restrict__ sel_mask,
                                                                        uint16_t *__restrict__ dQ)
{
    using C = DqSplit<D>;
    constexpr int NS = C::NS, KSTEPS = C::KSTEPS, DT = C::DT;
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    uint32_t *list = reinterpret_cast<uint32_t *>(smem);  // steps of the walk: cube << 16 | step of the cube
    bf16x8 *ops = reinterpret_cast<bf16x8 *>(smem + C::OFF_OPS);  // [Q, dO][slab][KSTEPS][lane]
    float *psums = reinterpret_cast<float *>(smem + C::OFF_PSUM);  // [wave][row]
    uint32_t *uni = reinterpret_cast<uint32_t *>(smem + C::OFF_UNION);
    int *nsteps_s = reinterpret_cast<int *>(smem + C::OFF_N);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;

    // workgroup -> (KV head, block of 32 rows), late rows (long walks) first, across the cubes' borders
    const int kv = blockIdx.x % g.Hkv;
    const int row1 = g.S * g.G - (int)(blockIdx.x / g.Hkv) * C::ROWS, row0 = max(0, row1 - C::ROWS), last = row1 - 1;
    const RowAt at = row_at(g, kv, min(row0 + (lane & 31), last));  // lane l works out row l % 32 (rows past the last one repeat it)
    int rank[NS], own[NS];
    size_t rowid[NS];
    float lse2[NS], delta[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        rank[s] = __shfl(at.rank, 16 * s + n16, 64);
        own[s] = __shfl(at.cube, 16 * s + n16, 64);
        rowid[s] = (size_t)__shfl(at.id, 16 * s + n16, 64);
        lse2[s] = lse2p[rowid[s]];    // -lse * sqrt(D): what the score products start from
        delta[s] = deltap[rowid[s]];  // minus delta: what the dP products start from
    }
    // the last cube with rows here, and the first
    const int i = __builtin_amdgcn_readlane(at.cube, 31), i_first = __builtin_amdgcn_readfirstlane(at.cube);
    const int max_rank = __builtin_amdgcn_readlane(block_max_rank(at, row1 - row0), 31);  // of the block's rows in cube i
    for (int x = wave; x < 2 * NS * KSTEPS; x += C::WAVES) {
        const int s = x / KSTEPS % NS, c = x % KSTEPS;
        ops[x * 64 + lane] = *reinterpret_cast<const bf16x8 *>((x < NS * KSTEPS ? Q : dO) + (s ? rowid[1] : rowid[0]) * D + 32 * c + 8 * q4);
    }

    // ---- the steps of the walk: the rows' own cubes, the last one up to the block's largest rank, and of those before them the ones
    // that a row selected
    if (MASKED) {
        // wavefront w takes mask words w, w + 8, ...; its lanes are the block's rows, twice over
        for (int w = wave; 32 * w <= i; w += C::WAVES) {
            uint32_t m = sel_mask[rowid[(lane >> 4) & 1] * g.words + w];
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) m |= __shfl_xor(m, d, 64);
            if (lane == 0) uni[w] = m;
        }
        __syncthreads();
    }
    if (wave == 0) {
        int n = 0;
        for (int c0 = 0; c0 <= i; c0 += 64) {
            const int c = c0 + lane;
            int steps = 0;
            if (c <= i && (!MASKED || c >= i_first || ((uni[c >> 5] >> (c & 31)) & 1u))) {
                const int size = c == i ? max_rank + 1 : g.ragged ? csize[c] : g.Cmax;
                steps = (size + C::STEP - 1) / C::STEP;
            }
            int incl = steps;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int up = __shfl_up(incl, d, 64);
                if (lane >= d) incl += up;
            }
            for (int k = 0; k < steps; ++k) list[n + incl - steps + k] = ((uint32_t)c << 16) | (uint32_t)k;
            n += __shfl(incl, 63, 64);
        }
        if (lane == 0) *nsteps_s = n;
    }
    __syncthreads();
    const int nsteps = __builtin_amdgcn_readfirstlane(*nsteps_s);

    // ---- this wavefront's steps: wave, wave + 8, ...  The next step's operands are loaded as soon as this one's are used.
    const size_t head = (size_t)kv * g.N * g.TPC * (KEY_TILE * D);
    bf16x8 kf[KSTEPS][2], vf[KSTEPS][2], tf[DT];
    uint32_t word[NS], word_next[NS];
    auto entry = [&](int p) -> uint32_t {  // (past the end the last step's operands are loaded, and not used)
        return __builtin_amdgcn_readfirstlane(list[min(p, nsteps - 1)]);
    };
    auto tile_of = [&](const uint16_t *copy, uint32_t e) __attribute__((always_inline)) {
        return reinterpret_cast<const unsigned char *>(copy + head + ((size_t)(e >> 16) * g.TPC + ((e & 0xffffu) >> 1)) * (KEY_TILE * D));
    };
    auto load_rows = [&](const uint16_t *copy, uint32_t e, bf16x8 (&f)[KSTEPS][2]) __attribute__((always_inline)) {
        const unsigned char *tile = tile_of(copy, e);
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2) {
                const int krow = 32 * (int)(e & 1u) + 8 * (n16 >> 2) + 4 * k2 + (n16 & 3);
                f[c][k2] = *reinterpret_cast<const bf16x8 *>(tile + k_tile_off<D>(krow, 4 * c + q4));
            }
    };
    auto load_cols = [&](uint32_t e) __attribute__((always_inline)) {
        const unsigned char *tile = tile_of(Kt, e);
#pragma unroll
        for (int e2 = 0; e2 < DT; ++e2)
            tf[e2] = *reinterpret_cast<const bf16x8 *>(tile + vt_tile_off(16 * e2 + n16, 4 * (int)(e & 1u) + q4));
    };
    auto load_words = [&](uint32_t e) __attribute__((always_inline)) {
        if (MASKED) {
#pragma unroll
            for (int s = 0; s < NS; ++s) word_next[s] = sel_mask[rowid[s] * g.words + (e >> 21)];
        }
    };
    const float c2 = BWD_LOG2E / sqrtf((float)D);  // softmax scale in base 2
    float psum[NS];
    f32x4 acc[NS][DT];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        psum[s] = 0.f;
#pragma unroll
        for (int e = 0; e < DT; ++e) acc[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // The step e0; e1 is the next one.  BEHIND: of a cube behind some rows' own.  These rows' probabilities are zero there, but K and
    // V need not be finite: they keep their sums.
    auto work = [&](uint32_t e0, uint32_t e1, auto behind) __attribute__((always_inline)) {
        constexpr bool BEHIND = decltype(behind)::value;
        const int j = (int)(e0 >> 16), key0 = C::STEP * (int)(e0 & 0xffffu);
        const bool edge = j >= i_first;  // some row's own cube, or behind it
        const int jsize = g.ragged ? csize[j] : g.Cmax;
#pragma unroll
        for (int s = 0; s < NS; ++s) word[s] = MASKED ? word_next[s] : 0u;
        f32x4 sa[NS][2], pa[NS][2];
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const bf16x8 q = ops[(s * KSTEPS + c) * 64 + lane];
                bool in = !MASKED || ((word[s] >> (j & 31)) & 1u);
                if (edge) in = j >= own[s] || in;
                const float b = in ? lse2[s] : -INFINITY;
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) sa[s][k2] = mfma16(kf[c][k2], q, c == 0 ? f32x4{b, b, b, b} : sa[s][k2]);
            }
        __builtin_amdgcn_sched_barrier(0);
        load_rows(Kn, e1, kf);
        load_words(e1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const bf16x8 o = ops[((NS + s) * KSTEPS + c) * 64 + lane];
                const float b = delta[s];
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2) pa[s][k2] = mfma16(vf[c][k2], o, c == 0 ? f32x4{b, b, b, b} : pa[s][k2]);
            }
        __builtin_amdgcn_sched_barrier(0);
        load_rows(Vn, e1, vf);
        __builtin_amdgcn_sched_barrier(0);
        if (edge || key0 + C::STEP > jsize) {  // the own cubes' causal edge, padding keys
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int lim = j < own[s] ? jsize - 1 : j == own[s] ? rank[s] : -1;
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (key0 + 8 * q4 + 4 * k2 + v > lim) sa[s][k2][v] = -INFINITY;
            }
        }
        bf16x8 ds[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float p = __builtin_amdgcn_exp2f(sa[s][k2][v] * c2);
                    psum[s] += p;
                    ds[s][4 * k2 + v] = (__bf16)(p * pa[s][k2][v]);
                }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < DT; ++e)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const f32x4 sum = mfma16(tf[e], ds[s], acc[s][e]);
                acc[s][e] = BEHIND && j > own[s] ? acc[s][e] : sum;
            }
        __builtin_amdgcn_sched_barrier(0);
        load_cols(e1);
        __builtin_amdgcn_sched_barrier(0);
    };
    if (wave < nsteps) {
        uint32_t e0 = entry(wave);
        load_rows(Kn, e0, kf);
        load_words(e0);
        load_rows(Vn, e0, vf);
        load_cols(e0);
        int p = wave;
        const uint32_t behind = (uint32_t)(i_first + 1) << 16;  // the first such step
        for (; p < nsteps && e0 < behind; p += C::WAVES) {
            const uint32_t e1 = entry(p + C::WAVES);
            work(e0, e1, std::false_type{});
            e0 = e1;
        }
        for (; p < nsteps; p += C::WAVES) {
            const uint32_t e1 = entry(p + C::WAVES);
            work(e0, e1, std::true_type{});
            e0 = e1;
        }
    }
    __syncthreads();  // the list is done with

    // ---- the wavefronts' sums, added in their order; then as in the kernel above
    f32x4 *part = reinterpret_cast<f32x4 *>(smem);  // [wave][s][e][lane]
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int e = 0; e < DT; ++e) part[((wave * NS + s) * DT + e) * 64 + lane] = acc[s][e];
        const float total = quad_sum(psum[s]);
        if (q4 == 0) psums[wave * C::ROWS + 16 * s + n16] = total;
    }
    __syncthreads();
    for (int x = wave; x < NS * DT; x += C::WAVES) {
        const int s = x / DT, e = x % DT;
        float total = 0.f;
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < C::WAVES; ++w) {
            total += psums[w * C::ROWS + 16 * s + n16];
            sum += part[((w * NS + s) * DT + e) * 64 + lane];
        }
        if (row0 + 16 * s + n16 > last) continue;
        const size_t rid = s == 0 ? rowid[0] : rowid[1];
        if (e == 0 && q4 == 0) lse2p[rid] = (s == 0 ? lse2[0] : lse2[1]) - log2f(total) / c2;
        *reinterpret_cast<uint2 *>(dQ + rid * D + 16 * e + 4 * q4) = pack_bf16(sum * (1.0f / (sqrtf((float)D) * total)));
    }
}

// ---------------------------------------------------------------------------------------------------------------
// dV, dK: workgroup = 256 keys of one (key cube j, KV head) and one range of row cubes (BwdParts).
//
// The rows of the range that selected cube j are listed in LDS from the transposed selection bits, BWD_LIST_WORDS
// 64-row words at a time, and gathered 64 at a time: natural Q and dO rows and their two start values, three LDS
// stages, started two tiles ahead.  A 256-byte (128-byte) row is fetched whole by 16 (8) lanes; the 16-byte chunk that
// lands in a slot is chosen by the lane that fetches it (row_swizzle), so that both kinds of operand read are free of
// bank conflicts: 16 consecutive rows at one chunk (ds_read_b128, S and dP), and 4 x 16-element blocks read transposed
// (ds_read_b64_tr_b16, the A operands of dV^T and dK^T).
//
// Bound by the matrix pipes and the operand reads that feed them (16 bytes of LDS per lane for every two MFMAs).  Both
// accumulators and both operand sets of 32 keys are 192 of the 256 registers that two wavefronts per SIMD leave: scores
// are therefore worked 16 rows at a time and the order of reads and MFMAs is fixed.  At 65,536 tokens, 28/4 heads of
// 128, Top-p 0.9 (61 % selected): 31.0 ms and 0.45 ms of sums, 1.23 PFLOP/s over selected pairs; two kernels that
// walked every row with the selection as a mask took 40.7 + 29.1 ms (and the transposed copies of Q and dO they
// streamed 0.4 ms).  At 16,384 tokens, where cube 0's walk used to outlast everything: 2.2 + 0.1 against 8.5 ms.
// On short sequences a workgroup's chain of memory latencies counts: the selection words and row ids are asked for before the keys, and the
// own cube's rows lie behind the last list's, one stream of tiles for both.  A backward pass over 1,080 tokens of 6/2 heads of 128: 56.5 us,
// with each in its turn 59.4.
// ---------------------------------------------------------------------------------------------------------------
constexpr int BWD_LIST_WORDS = 64;

template <int D>
struct Dkv {
    static constexpr int TILE = 64 * D * 2;
    static constexpr int OFF_LSE = 2 * TILE;  // Q, dO, then 64 floats lse2, 64 floats delta
    static constexpr int STAGE = 2 * TILE + 512;
    static constexpr int NST = 3;
    static constexpr int OFF_ROWS = NST * STAGE;  // row ids of the list
    static constexpr int OFF_WORDS = OFF_ROWS + 64 * BWD_LIST_WORDS * 4;
    static constexpr int OFF_BASE = OFF_WORDS + BWD_LIST_WORDS * 8;
    static constexpr int BYTES = OFF_BASE + (BWD_LIST_WORDS + 1) * 4 + 12;
    static_assert(BYTES <= 160 * 1024, "LDS of one CU");
};

// Slot of 16-byte chunk c of tile row r.  An LDS line is 16 slots: one row of head-dim 128, two of 64.  A ds_read_b128 of 64 lanes is served
// 16 lanes at a time, lanes 0-3, 12-15, 20-27 first: with the chunk index equal in 0-15 and one higher in 16-31, the
// lines' swizzle values must be distinct and those of rows 4..11 closed under ^ 1.  A transposing read is served 32
// lanes at a time, 8 rows at two neighbouring chunks: their values must differ above bit 0 (measured: 241 bytes per
// clock for both kinds; a plain row number gives 227 and 122).
template <int D>
__device__ __forceinline__ int row_swizzle(int r)
{
    if (D == 128) return (((r & 7) ^ (((r >> 3) & 1) << 2)) << 1) | ((r >> 3) & 1);
    const int line = r >> 1;
    return (((line & 3) ^ (((line >> 2) & 1) << 1)) << 1) | ((line >> 2) & 1);
}
template <int D>
__device__ __forceinline__ int row_tile_off(int r, int c)
{
    if (D == 128) return r * 256 + ((c ^ row_swizzle<D>(r)) << 4);
    return (r >> 1) * 256 + (((((r & 1) << 3) | c) ^ row_swizzle<D>(r)) << 4);
}

// LDS reads by address.
template <typename T>
__device__ __forceinline__ T lds_read(uint32_t addr)
{
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(addr);
}
// Two transposing reads, `step` bytes apart.  In each, lane (n16, q4) gets the elements at column n16 of the four
// 16-element row pieces that lanes 16 q4 .. 16 q4 + 15 point to (lane 4 k + m of them: 8 bytes, elements 4 m .. 4 m + 3 of
// row k).
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8 lds_read_tr2(uint32_t addr, int step)
{
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4 *>(addr));
    const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s16x4 *>(addr + step));
    return __builtin_bit_cast(bf16x8, (s16x8)__builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// SHARED: cubes of up to 128 tokens (a workgroup then has at most four wavefronts' worth of keys).  Wavefronts w and w + 4 take the
// same keys, and the first and the second half of every tile's rows; their sums are added through LDS at the end
// (dkv_shared).
template <int D, bool SHARED>
__global__ __launch_bounds__(BWD_THREADS) void attn_bwd_dkv_kernel(Geom g, const uint16_t *__restrict__ K,
                                                                   const uint16_t *__restrict__ V,
                                                                   const uint16_t *__restrict__ Q,
                                                                   const uint16_t *__restrict__ dO,
                                                                   const float *__restrict__ lse2,
                                                                   const float *__restrict__ delta, int tpcr,
                                                                   const unsigned long long *__restrict__ colmask,
                                                                   const uint32_t *__restrict__ rowtab, BwdParts cut, float *__restrict__ part,
                                                                   uint16_t *__restrict__ dK, uint16_t *__restrict__ dV)
{
    using C = Dkv<D>;
    constexpr int NS = 2, KSTEPS = D / 32, DT = D / 16;
    constexpr int CPR = D / 8;               // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;            // rows per direct-to-LDS instruction
    constexpr int PER = 64 / RPI / 8;        // such instructions per wavefront, tile and operand
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    uint32_t *rows = reinterpret_cast<uint32_t *>(smem + C::OFF_ROWS);
    unsigned long long *words = reinterpret_cast<unsigned long long *>(smem + C::OFF_WORDS);
    int *base = reinterpret_cast<int *>(smem + C::OFF_BASE);

    int kv, slot;
    if (!bwd_head_slot(blockIdx.x, g.Hkv, (int)(cut.nkb * cut.parts), kv, slot)) return;
    const int kb = slot % cut.nkb;
    const int pidx = (int)cut.parts - 1 - slot / cut.nkb;  // the later ranges, which have the most parts, first
    int c = (int)((sqrtf(1.0f + 8.0f * (float)pidx / (float)cut.span) - 1.0f) * 0.5f);
    while (c > 0 && (long long)cut.span * c * (c + 1) / 2 > pidx) --c;
    while (c + 1 < cut.nc && (long long)cut.span * (c + 1) * (c + 2) / 2 <= pidx) ++c;
    const int j = pidx - (int)((long long)cut.span * c * (c + 1) / 2);
    const CubeBox box = cube_box(g, j);
    const int size_j = box.size();
    if (kb * BWD_ROWS >= size_j) return;
    const bool single = cut.nc - j / cut.span == 1;  // these keys have no other part

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n16 = lane & 15, q4 = lane >> 4;

    // the rows' selection words and, of the wavefront's first one, their ids, for the first list: asked for before the keys
    const int i0 = max(c * cut.span, j + 1), i1 = min(g.N, (c + 1) * cut.span);
    const int nwords = max(0, i1 - i0) * tpcr;
    const unsigned long long *cm = colmask + (((size_t)kv * g.N + j) * g.N + i0) * tpcr;
    const uint32_t *tab = rowtab + (size_t)i0 * tpcr * 64;
    unsigned long long bits = lane < nwords ? cm[lane] : 0ull;
    uint32_t id = wave < nwords ? tab[wave * 64 + lane] : 0u;

    // the wavefront's keys (B operands)
    const int key0 = kb * BWD_ROWS + (SHARED ? wave & 3 : wave) * 32;
    const bool busy = key0 < size_j;  // (a wavefront without keys only helps with the loads)
    bf16x8 kf[NS][KSTEPS], vf[NS][KSTEPS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int key = min(key0 + s * 16 + n16, size_j - 1);
        const size_t krow = ((size_t)token_of(g, box, key) * g.Hkv + kv) * D;
#pragma unroll
        for (int k = 0; k < KSTEPS; ++k) {
            kf[s][k] = *reinterpret_cast<const bf16x8 *>(K + krow + 32 * k + 8 * q4);
            vf[s][k] = *reinterpret_cast<const bf16x8 *>(V + krow + 32 * k + 8 * q4);
        }
    }
    const float c2 = BWD_LOG2E / sqrtf((float)D);  // softmax scale in base 2
    const uint32_t nrows_all = (uint32_t)(g.S * g.Hq);

    f32x4 accV[NS][DT], accK[NS][DT];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int e = 0; e < DT; ++e) accV[s][e] = accK[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};

    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
    // The lane's part in a tile's loads: piece u of this wavefront is RPI rows of the tile, one 16-byte slot per lane.
    // (Computed anew for every tile, here and below, by hiding where `lane` comes from: registers are short.)
    auto fresh_lane = [&]() __attribute__((always_inline)) {
        int l = lane;
        asm volatile("" : "+v"(l));
        return l;
    };
    // A tile past the list's end (n rows) is padded with the list's last row -- a row that has its place in this tile anyway,
    // so that what is not finite in it reaches nobody new -- under start values that give it no part.
    auto issue = [&](int stage, int first, int n) __attribute__((always_inline)) {
        const uint32_t dst = lds0 + (uint32_t)(stage * C::STAGE);
        const int l = fresh_lane();
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int r = (wave * PER + u) * RPI + l / CPR;
            const uint32_t rid = rows[min(first + r, n - 1)];
            const int chunk = ((l & 15) ^ row_swizzle<D>(r)) & (CPR - 1);
            const size_t off = (size_t)rid * D + chunk * 8;
            const uint32_t piece = dst + (uint32_t)((wave * PER + u) * 1024);
            dma_lane16(__builtin_amdgcn_readfirstlane(piece), Q + off);
            dma_lane16(__builtin_amdgcn_readfirstlane(piece + C::TILE), dO + off);
        }
        if (wave < 2) {  // the start values: wavefront 0 lse2, wavefront 1 delta
            const float *vals = wave == 0 ? lse2 : delta;
            dma_lane4(__builtin_amdgcn_readfirstlane(dst + C::OFF_LSE + 256 * wave),
                      vals + (first + l < n ? rows[min(first + l, n - 1)] : nrows_all));
        }
    };
    // Opens a tile: this wavefront's loads of it have landed (those of the next tile may stay in flight), then everybody's.
    auto open_tile = [&](bool more) __attribute__((always_inline)) {
        if (!more) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else if (wave < 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * PER + 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * PER) : "memory");
    };

    // Operand reads: the lane's place in a tile for both kinds, without the 16-row block (an immediate offset) and the
    // chunk's high bits (flipped per read: a table of the addresses would not fit the register file).
    const uint32_t nat0 = (uint32_t)row_tile_off<D>(n16, q4);
    const uint32_t tr0 = (uint32_t)(row_tile_off<D>(4 * q4 + (n16 >> 2), (n16 & 3) >> 1) + 8 * (n16 & 1));
    constexpr int BLK = 16 * D * 2;  // bytes of 16 tile rows

    // One 64-row tile, in two halves of 32 rows.  OWN: the rows are cube j's own, from row r0 of its (rank, head) order.
    // The order written here is the order executed (operands one step ahead of their MFMAs): left to itself the
    // compiler starts more loads than there are registers for.
    auto tile_work = [&](int stage, auto own_tag, int r0) __attribute__((always_inline)) {
        constexpr bool OWN = decltype(own_tag)::value;
        const uint32_t st = lds0 + (uint32_t)(stage * C::STAGE);
        const uint32_t first = SHARED ? (uint32_t)((wave >> 2) * 2 * BLK) : 0u;  // the wavefront's half of the rows
        const uint32_t nat = st + nat0 + first, tr = st + tr0 + first;
        auto rows_at = [&](int blk, int k, bf16x8 (&o)[2]) __attribute__((always_inline)) {  // Q, dO
            uint32_t at;
            asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "n"(k << 6), "v"(nat));
            o[0] = lds_read<bf16x8>(at + (uint32_t)(blk * BLK));
            o[1] = lds_read<bf16x8>(at + (uint32_t)(blk * BLK + C::TILE));
        };
        auto cols_at = [&](int H, int e, bf16x8 (&o)[2]) __attribute__((always_inline)) {  // Q^T, dO^T
            uint32_t at;
            asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "n"(e << 5), "v"(tr));
            o[0] = lds_read_tr2(at + (uint32_t)(2 * H * BLK), BLK);
            o[1] = lds_read_tr2(at + (uint32_t)(2 * H * BLK + C::TILE), BLK);
        };
        bf16x8 op[2][2];
        rows_at(0, 0, op[0]);
#pragma unroll
        for (int H = 0; H < (SHARED ? 1 : 2); ++H) {
            bf16x8 pp[NS], ds[NS];
#pragma unroll
            for (int x = 0; x < 2; ++x) {  // 16 rows: scores and dP
                const uint32_t vec = st + (uint32_t)(C::OFF_LSE + 16 * (2 * H + x) * 4 + (SHARED ? wave >> 2 : 0) * 128) + (uint32_t)(16 * q4);
                const f32x4 li = lds_read<f32x4>(vec), di = lds_read<f32x4>(vec + 256);
                f32x4 sa[NS], pa[NS];
#pragma unroll
                for (int k = 0; k < KSTEPS; ++k) {
                    if (k + 1 < KSTEPS) rows_at(2 * H + x, k + 1, op[(k + 1) & 1]);
                    else if (x == 0) rows_at(2 * H + 1, 0, op[(k + 1) & 1]);
                    else cols_at(H, 0, op[(k + 1) & 1]);
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        sa[s] = mfma16(op[k & 1][0], kf[s][k], k == 0 ? li : sa[s]);
                        pa[s] = mfma16(op[k & 1][1], vf[s][k], k == 0 ? di : pa[s]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (OWN) {  // causal edge: a row attends keys up to its own rank, row / G
                    const int row = r0 + (SHARED ? wave >> 2 : 0) * 32 + 16 * (2 * H + x) + 4 * q4;
#pragma unroll
                    for (int s = 0; s < NS; ++s) {
                        const int reach = (key0 + 16 * s + n16) * g.G;  // the first row that attends the key
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (row + v < reach) sa[s][v] = -INFINITY;
                    }
                }
#pragma unroll
                for (int s = 0; s < NS; ++s)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float p = __builtin_amdgcn_exp2f(sa[s][v] * c2);
                        pp[s][4 * x + v] = (__bf16)p;
                        ds[s][4 * x + v] = (__bf16)(p * pa[s][v]);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
            // dV^T += dO^T.P, dK^T += Q^T.dS over the half's 32 rows (k index 8 q4 + 4 x + v: row 16 x + 4 q4 + v)
#pragma unroll
            for (int e = 0; e < DT; ++e) {
                if (e + 1 < DT) cols_at(H, e + 1, op[(e + 1) & 1]);
                else if (H == 0 && !SHARED) rows_at(2, 0, op[(e + 1) & 1]);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    accK[s][e] = mfma16(op[e & 1][0], ds[s], accK[s][e]);
                    accV[s][e] = mfma16(op[e & 1][1], pp[s], accV[s][e]);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // The list through the tiles: n rows, then, from a tile of their own on, m of cube j itself, its rows f ...
    auto run_list = [&](int n, int m, int f) __attribute__((always_inline)) {
        const int nt1 = (n + 63) >> 6, nt = nt1 + ((m + 63) >> 6);
        if (nt == 0) return;
        auto issue_tile = [&](int stage, int t) __attribute__((always_inline)) { issue(stage, 64 * t, t < nt1 ? n : 64 * nt1 + m); };
        issue_tile(0, 0);
        if (nt > 1) issue_tile(1, 1);
        int stage = 0, t = 0;
        auto tile = [&](auto own_tag) __attribute__((always_inline)) {
            constexpr bool OWN = decltype(own_tag)::value;
            open_tile(t + 1 < nt);
            const int s2 = stage == 0 ? 2 : stage - 1;  // (stage + 2) % 3: read last at tile t - 1
            if (t + 2 < nt) issue_tile(s2, t + 2);
            const int r0 = f + 64 * (t - nt1);
            // (own cube: no row of the tile reaches the wavefront's keys if the last one does not)
            if (busy && (!OWN || (r0 + 63) / g.G >= key0)) tile_work(stage, own_tag, r0);
            stage = stage == 2 ? 0 : stage + 1;
        };
        for (; t < nt1; ++t) tile(std::false_type{});
        for (; t < nt; ++t) tile(std::true_type{});
    };

    // ---- the rows: 64-row words w of the range's row cubes, BWD_LIST_WORDS at a time; behind the last of them cube j's own rows, in
    // rank order, if the range has it (ranks below the block's first key attend none of its keys)
    const int own = c == j / cut.span ? size_j * g.G : 0;
    int f = kb * BWD_ROWS * g.G / 64 * 64;
    for (int w0 = 0; w0 < nwords || f < own; w0 += BWD_LIST_WORDS) {
        __syncthreads();  // the list before is done with
        const int l = fresh_lane();
        int n = 0;
        if (w0 < nwords) {
            if (wave == 0) {
                const int mine = __popcll(bits);
                int incl = mine;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int up = __shfl_up(incl, d, 64);
                    if (l >= d) incl += up;
                }
                words[l] = bits;
                base[l] = incl - mine;
                if (l == 63) base[BWD_LIST_WORDS] = incl;
            }
            __syncthreads();
            n = __builtin_amdgcn_readfirstlane(base[BWD_LIST_WORDS]);
            for (int x = wave; x < min(BWD_LIST_WORDS, nwords - w0); x += BWD_THREADS / 64) {
                const unsigned long long word = words[x];
                if (x != wave) id = tab[(size_t)(w0 + x) * 64 + l];
                if ((word >> l) & 1ull) rows[base[x] + __popcll(word & ((1ull << l) - 1ull))] = id + (uint32_t)(kv * g.G);
            }
        }
        const int at = (n + 63) & ~63, m = w0 + BWD_LIST_WORDS >= nwords ? max(0, min(own - f, 64 * BWD_LIST_WORDS - at)) : 0;
        for (int x = wave * 64 + l; x < m; x += BWD_THREADS) rows[at + x] = rowtab[(size_t)j * tpcr * 64 + f + x] + (uint32_t)(kv * g.G);
        __syncthreads();
        run_list(n, m, f);
        f += m;
        const int next = w0 + BWD_LIST_WORDS, lane1 = fresh_lane();  // (the next list's, as above)
        bits = next + lane1 < nwords ? cm[next + lane1] : 0ull;
        id = next + wave < nwords ? tab[(size_t)(next + wave) * 64 + lane1] : 0u;
    }
    if (SHARED) {
        static_assert(4 * NS * DT * 1024 <= C::OFF_ROWS, "one sum of four wavefronts fits the tiles' place");
        f32x4 *sums = reinterpret_cast<f32x4 *>(smem) + (size_t)(wave & 3) * (NS * DT * 64) + lane;
        auto add = [&](f32x4 (&acc)[NS][DT]) __attribute__((always_inline)) {
            __syncthreads();
            if (wave >= 4) {
#pragma unroll
                for (int x = 0; x < NS * DT; ++x) sums[x * 64] = acc[x / DT][x % DT];
            }
            __syncthreads();
            if (wave < 4) {
#pragma unroll
                for (int x = 0; x < NS * DT; ++x) acc[x / DT][x % DT] += sums[x * 64];
            }
        };
        add(accV);
        add(accK);
        if (wave >= 4) return;
    }
    if (!busy) return;

    // ---- results: element (s, e, v) of lane (n16, q4) is key 16 s + n16, head-dim 16 e + 4 q4 + v
    const float scale = 1.0f / sqrtf((float)D);
    if (single) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int key = key0 + 16 * s + n16;
            if (key >= size_j) continue;
            const size_t o = ((size_t)token_of(g, box, key) * g.Hkv + kv) * D + 4 * q4;
#pragma unroll
            for (int e = 0; e < DT; ++e) {
                *reinterpret_cast<uint2 *>(dV + o + 16 * e) = pack_bf16(accV[s][e]);
                *reinterpret_cast<uint2 *>(dK + o + 16 * e) = pack_bf16(accK[s][e] * scale);
            }
        }
        return;
    }
    float *out = part + (((size_t)kv * cut.nkb + kb) * cut.parts + pidx) * (2 * cut.keys * D) + (size_t)wave * (32 * D) + lane * 4;
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int e = 0; e < DT; ++e) {
            *reinterpret_cast<f32x4 *>(out + (s * DT + e) * 256) = accV[s][e];
            *reinterpret_cast<f32x4 *>(out + cut.keys * D + (s * DT + e) * 256) = accK[s][e];
        }
}

// Sums the parts of (KV head and key block, cube j) in range order; a thread owns four elements of dV and of dK.
template <int D>
__global__ __launch_bounds__(256) void bwd_reduce_kernel(Geom g, BwdParts cut, const float *__restrict__ part,
                                                         uint16_t *__restrict__ dK, uint16_t *__restrict__ dV)
{
    constexpr int DT = D / 16;
    const int per = cut.keys * D / 4 / 256;  // workgroups per key block
    const int j = blockIdx.y, kv = blockIdx.z, kb = blockIdx.x / per;
    const int c0 = j / cut.span;
    if (cut.nc - c0 == 1) return;
    const CubeBox box = cube_box(g, j);
    // position x of a part: wavefront, (s, e), lane
    const int x = blockIdx.x % per * 256 + threadIdx.x;
    const int lane = x & 63, e = (x >> 6) % DT, s = (x >> 6) / DT % 2, wave = (x >> 6) / (2 * DT);
    const int key = kb * BWD_ROWS + wave * 32 + s * 16 + (lane & 15);
    if (key >= box.size()) return;
    const float *src = part + (((size_t)kv * cut.nkb + kb) * cut.parts + j) * (2 * cut.keys * D) + (size_t)x * 4;
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, k = v;
#pragma unroll 4
    for (int c = c0; c < cut.nc; ++c) {
        const float *p = src + ((size_t)cut.span * c * (c + 1) / 2) * (2 * cut.keys * D);
        v += *reinterpret_cast<const f32x4 *>(p);
        k += *reinterpret_cast<const f32x4 *>(p + cut.keys * D);
    }
    const size_t o = ((size_t)token_of(g, box, key) * g.Hkv + kv) * D + 16 * e + 4 * (lane >> 4);
    *reinterpret_cast<uint2 *>(dV + o) = pack_bf16(v);
    *reinterpret_cast<uint2 *>(dK + o) = pack_bf16(k * (1.0f / sqrtf((float)D)));
}

// Wavefronts that share 32 rows in the dQ kernel.
// Two: while the workgroups of 256 rows find a CU each the kernel takes what
// the longest walk takes; shared, a little over half of that.  With more, every CU is busy most of the time and sharing only adds
// its own cost.  A backward pass, us, shared and not, by workgroups of 256 rows: 28/4 heads of 128, 112 146, 157, 252 226, 233, 308 293, 283;
// 6/2 of 128, 102 206, 253, 282 749, 791, 330 980, 966; 8/2 of 64, 160 171, 204, 280 379, 396, 328 514, 493; 4/4 of 64, 280 653, 702,
// 328 860, 839; 32/8 of 128, 256 198, 206, 288 263, 251; 6/2 in cubes of up to 128 clipped to 32, 282 911, 953, 330 1,238, 1,214.
// Eight (attn_bwd_dq_split_kernel): from what each of the two takes (us), fitted to the backward passes of 132 shapes of 500 to 6,000 tokens, heads
// 4/4 .. 32/8 of 64 and 128, cubes of 32 to 256 tokens; but for four the choice is the faster kernel or within 2.5 % of it (10 %: 480 tokens).
//   two    a tile of 64 keys takes 1.28 at head-dim 64 and 1.85 at 128; the longest walk's tiles, or all of them over the CUs
//   eight  a step of 32 keys takes a CU 0.29 and 0.42, half the steps on average; a workgroup 4 to start and to combine its sums
// On both sides of the line: 8/2 heads of 64 in cubes of 256, 2,048 tokens 86 eight, 95 two; 4,096 166, 150.  6/2 of 128 in clipped cubes of
// up to 128, 1,080 tokens 57, 92.  28/4 of 128 in cubes of 256, 512 tokens 65, 66; 1,024 135, 109.
int bwd_dq_waves(const Geom &g)
{
    const long long blocks = (long long)g.Hkv * ((g.S * g.G - 1) / BWD_ROWS + 1);
    if (blocks > DQ_SHARED_BLOCKS) return 1;
    const long long list = (long long)g.N * ((g.Cmax + DqSplit<64>::STEP - 1) / DqSplit<64>::STEP);
    if (list > (g.D == 64 ? DqSplit<64>::LIST_MAX : DqSplit<128>::LIST_MAX) || g.Cmax > 65536 * DqSplit<64>::STEP / 2) return 2;
    const double x = g.Hkv * std::ceil((double)g.S * g.G / DqSplit<64>::ROWS) / 256;
    const double two = (g.D == 64 ? 1.28 : 1.85) * (double)tiles_of_cubes(g, KEY_TILE) *
                       std::max(1.0, 0.64 * g.Hkv * std::ceil((double)g.S * g.G / (BWD_ROWS / 2)) / 256);
    const double eight = 8 + 4 * std::max(0.0, x - 1) +
                         (g.D == 64 ? 0.145 : 0.21) * std::max(0.8, x) * (double)tiles_of_cubes(g, DqSplit<64>::STEP);
    return eight < two ? 8 : 2;
}

bool bwd_dq_half_tiles(const Geom &g) { return g.Cmax <= KEY_TILE / 2 && bwd_dq_waves(g) == 1; }

// Whether two wavefronts share 32 keys in the dK/dV kernel: with cubes of up to 128 tokens half or more of a workgroup's wavefronts
// have no keys of their own.  Few rows do not make up for the sums' exchange: it takes the rows of a KV head, or those of a cube, which a
// workgroup has all of in one piece.  A backward pass, us, shared and not,
// by rows of a KV head: 28/4 heads of 128, cubes of 32, 5,040 135, 135, 8,064 176, 181, 16,128 390, 429; of 128, 3,584 57, 59, 16,128 233, 239;
// 6/2 of 128, cubes of 32, 4,320 175, 167, 6,480 215, 216, 15,984 552, 591; of 64, 5,472 120, 117, 8,064 184, 176, 16,128 303, 319; 8/2 of 64, cubes of
// 32, 5,760 133, 126, 8,064 149, 149; 4/4 of 64, cubes of 64, 2,976 116, 114, 7,968 294, 312.  Between 3,000 and 8,000 rows either is up to 7 % faster.
// By rows of a cube, 480 to 2,000 tokens: 896 (28/4, 14/2 heads of 128) 61, 67 and 71, 76; 448 48, 50 and 65, 70; 512 (32/8 of 128, 8/2 of 64) 107, 112 and 56, 59;
// 384 (6/2 of 128) 67, 71 and 107, 106; 256 69, 67 and 61, 61; 192 73, 71; 128 (4/4 of 64) 92, 82; 96 113, 105.  Between 224 and 384 rows either is
// faster by up to 6 %: 8/2 of 64, 960 tokens, 256 37.7, 39.7, 320 42.3, 45.1, 384 38.6, 39.7, but 1,440, 256 59.2, 58.6; 6/2 of 128, 336, 1,080 tokens 59.9, 62.0,
// 1,920 93.7, 90.8; 384, 1,080 56.6, 58.0, 1,920 88.6, 86.5; 32/8 of 128, 320 113, 107; 28/4 of 128, 224 97.5, 93.5, 336 130, 129.
static bool dkv_shared(const Geom &g)
{
    return g.Cmax <= BWD_ROWS / 2 && ((long long)g.S * g.G >= SHARED_ROWS || g.G * g.Cmax >= SHARED_CUBE_ROWS);
}

template <int D>
static hipError_t launch_bwd_d(const Geom &g, const uint16_t *Q, const uint16_t *K, const uint16_t *V,
                               const uint16_t *O, const float *lse, const uint16_t *dO, const uint32_t *sel_mask,
                               uint16_t *dQ, uint16_t *dK, uint16_t *dV, bool in_place, void *ws, hipStream_t st)
{
    const BwdWorkspace w = bwd_workspace(g, ws, in_place);
    if (in_place) {
        const long long pieces = (long long)g.S * g.Hq * (D / 8);
        hipLaunchKernelGGL(bwd_copy_rows_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, st, pieces,
                           reinterpret_cast<const uint4 *>(Q), reinterpret_cast<const uint4 *>(dO),
                           reinterpret_cast<uint4 *>(w.Q), reinterpret_cast<uint4 *>(w.dO));
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        Q = w.Q;
        dO = w.dO;
    }
    BwdPrep prep{K, V, O, dO, lse, sel_mask, w.Kn, w.Vn, w.Kt, w.csize, w.lse2, w.delta, w.colmask, w.rowtab, w.tpcr, 0, 0};
    prep.mask_blocks = (uint32_t)(((long long)w.tpcr * g.N * g.Hkv + 3) / 4);
    prep.key_blocks = (uint32_t)((long long)g.TPC * g.N * g.Hkv);
    const long long row_blocks = ((long long)g.S * g.Hq + 1 + 256 / (D / 8) - 1) / (256 / (D / 8));
    hipLaunchKernelGGL((bwd_prep_kernel<D>), dim3((unsigned)(prep.mask_blocks + prep.key_blocks + row_blocks)), dim3(256), 0, st, g,
                       prep);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int TILE = 64 * D * 2;

    const int waves = bwd_dq_waves(g), keys = std::min(2, waves), rows_q = BWD_ROWS / keys;
    const dim3 grid_q(bwd_grid(g.Hkv, (g.S * g.G - 1) / rows_q + 1));
    const int lds_q = 2 * 3 * TILE + BWD_ROWS * 16 + ADASPARK_MAX_CUBES / 8 + ADASPARK_MAX_CUBES * 2 + 16;
    const BwdParts &cut = w.cut;
    const dim3 grid_k(bwd_grid(g.Hkv, (int)(cut.nkb * cut.parts)));
    constexpr int lds_k = Dkv<D>::BYTES;
    auto launch_dq = [&](auto masked, auto keys_c, auto small) -> hipError_t {
        constexpr bool MASKED = decltype(masked)::value, SMALL = decltype(small)::value;
        constexpr int KEYS = decltype(keys_c)::value;
        static LdsOptIn opted_q;  // one per kernel instantiation
        const hipError_t err = opted_q.ensure(reinterpret_cast<const void *>(&attn_bwd_dq_kernel<D, MASKED, KEYS, SMALL>), lds_q);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((attn_bwd_dq_kernel<D, MASKED, KEYS, SMALL>), grid_q, dim3(BWD_THREADS), lds_q, st, g, Q, dO, w.Kn, w.Vn,
                           w.Kt, w.csize, w.lse2, w.delta, sel_mask, dQ);
        return hipGetLastError();
    };
    const std::integral_constant<int, 1> one;
    const std::integral_constant<int, 2> two;
    auto launch_split = [&](auto masked) -> hipError_t {
        constexpr bool MASKED = decltype(masked)::value;
        static LdsOptIn opted_s;  // one per kernel instantiation
        const hipError_t err = opted_s.ensure(reinterpret_cast<const void *>(&attn_bwd_dq_split_kernel<D, MASKED>), DqSplit<D>::BYTES);
        if (err != hipSuccess) return err;
        const unsigned blocks = (unsigned)((g.S * g.G - 1) / DqSplit<D>::ROWS + 1) * (unsigned)g.Hkv;
        hipLaunchKernelGGL((attn_bwd_dq_split_kernel<D, MASKED>), dim3(blocks), dim3(BWD_THREADS), DqSplit<D>::BYTES, st, g, Q, dO, w.Kn,
                           w.Vn, w.Kt, w.csize, w.lse2, w.delta, sel_mask, dQ);
        return hipGetLastError();
    };
    if (waves == 8)
        e = sel_mask != nullptr ? launch_split(std::true_type{}) : launch_split(std::false_type{});
    else {
        const std::true_type yes;
        const std::false_type no;
        auto launch_masked = [&](auto masked) -> hipError_t {
            if (keys == 2) return launch_dq(masked, two, no);
            return bwd_dq_half_tiles(g) ? launch_dq(masked, one, yes) : launch_dq(masked, one, no);
        };
        e = sel_mask != nullptr ? launch_masked(yes) : launch_masked(no);
    }
    if (e != hipSuccess) return e;
    auto launch_dkv = [&](auto shared) -> hipError_t {
        constexpr bool SHARED = decltype(shared)::value;
        static LdsOptIn opted_k;  // one per kernel instantiation
        const hipError_t err = opted_k.ensure(reinterpret_cast<const void *>(&attn_bwd_dkv_kernel<D, SHARED>), lds_k);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, SHARED>), grid_k, dim3(BWD_THREADS), lds_k, st, g, K, V, Q, dO, w.lse2, w.delta,
                           w.tpcr, w.colmask, w.rowtab, cut, w.part, dK, dV);
        return hipGetLastError();
    };
    e = dkv_shared(g) ? launch_dkv(std::true_type{}) : launch_dkv(std::false_type{});
    if (e != hipSuccess) return e;
    if (cut.nc > 1)
        hipLaunchKernelGGL((bwd_reduce_kernel<D>), dim3(cut.nkb * (cut.keys * D / 4 / 256), g.N, g.Hkv), dim3(256), 0, st, g,
                           cut, w.part, dK, dV);
    return hipGetLastError();
}

hipError_t launch_attn_bwd(const Geom &g, const uint16_t *Q, const uint16_t *K, const uint16_t *V, const uint16_t *O,
                           const float *lse, const uint16_t *dO, const uint32_t *sel_mask, uint16_t *dQ, uint16_t *dK,
                           uint16_t *dV, bool in_place, void *ws, hipStream_t st)
{
    if (g.D == 64) return launch_bwd_d<64>(g, Q, K, V, O, lse, dO, sel_mask, dQ, dK, dV, in_place, ws, st);
    return launch_bwd_d<128>(g, Q, K, V, O, lse, dO, sel_mask, dQ, dK, dV, in_place, ws, st);
}

}  // namespace adaspark
