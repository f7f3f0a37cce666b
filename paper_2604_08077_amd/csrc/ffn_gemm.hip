// The two matrix products of the token-selective FFN (Sec. 3.3, Eq. 6) on the activated tokens:
//   gated:  H[r][n] = silu(sum_k X[active[r]][k] Wg[n][k]) * (sum_k X[active[r]][k] Wu[n][k])   bf16 out
//   down :  F[r][n] = sum_k H[r][k] Wd[n][k]                                                    fp32 out
// Both are C = A.B^T with A (activations) and B (weights) stored row-major with the reduction index contiguous.
//
// Workgroup = 256 activation rows x 256 weight rows, 64 reduction elements per step, 8 wavefronts (2 along the activation
// rows x 4 along the weight rows; a wavefront has 64 rows of either activation half and 32 of either weight half).  Tiles
// go from global memory straight into LDS (global_load_lds_dwordx4), two stages; the 16-byte chunks of a tile row are
// XOR-swizzled by the choice of which chunk a lane fetches, so that the MFMA operand reads are conflict-free.
// mfma_f32_16x16x32_bf16 with the weights on the M side and the activations on the N side: a lane ends up with four
// consecutive output features of one token, which is what a row-major store wants.  For the gated product a tile's
// weight halves are 128 rows of W_gate and the same 128 rows of W_up, so every wavefront holds matching pairs.
//
// A reduction step is two halves (the activation halves), a half is two slots -- operands into registers, 32 MFMAs --
// with a workgroup barrier between slots, and the two wavefronts of a SIMD are one slot apart: while one multiplies, the
// other reads its operands and starts loads.  A half's place in LDS is free as soon as both sets have read it, so loads run
// a step and a half ahead in two stages.  In slots (set P: wavefronts 0-3, set Q: 4-7, one later), step k is
//   P  4k: read A0 W0 W1, load A1(k+1)   4k+1: multiply   4k+2: read A1, load A0 W0 W1(k+2)   4k+3: multiply
// Q's last read of A0 W0 W1(k) is in slot 4k+1 and of A1(k) in 4k+3, before their loads of step k+2 (same stage) start
// in 4k+2 and 4k+4; those have to have landed (vmcnt, then the barrier) before P's reads in slots 4k+8 and 4k+10.
//
// Bound by power: with random operands the chip clocks 1.75 GHz under this kernel (2.0 without the loads and LDS reads),
// where the matrix pipes then are 73 % busy.  65,536 tokens, 3584/18944, Top-p 0.7: 6.4 + 3.05 ms, 1.3 PFLOP/s; one barrier per
// step, both wavefronts of a SIMD in phase and loads one step ahead: 7.0 + 3.3 ms.  Tried: both in phase with operands
// prefetched across two barriers a step (6.7 + 3.2, loads spread between the MFMAs: 6.5 + 3.1), the barrier ahead of a
// slot's last MFMAs (slower: it holds the other set's reads back).
#include "attn_tile.h"
#include "ffn.h"

namespace adaspark {

constexpr int GT = FFN_ROW_TILE;            // rows of a tile, both operands
constexpr int GK = 64;                      // reduction elements per step: 128 bytes per row
constexpr int GEMM_THREADS = 512;
constexpr int TILE_BYTES = GT * GK * 2;     // 32 KB
constexpr int HALF_BYTES = TILE_BYTES / 2;
constexpr int STAGE_BYTES = 2 * TILE_BYTES;  // activations, weights
constexpr int HALF_STAGE = HALF_BYTES + TILE_BYTES;  // half the activation rows
constexpr int GEMM_LDS = 3 * HALF_STAGE;    // 144 KB (two whole stages: 128)

// Ends a slot: everything this wavefront has loaded but the newest KEEP loads (63: whatever is on the way) has landed and
// its LDS reads are done, then the workgroup barrier.
template <int KEEP>
__device__ __forceinline__ void open_slot()
{
    if (KEEP == 63) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(KEEP) : "memory");
}

template <bool GATED>
__global__ __launch_bounds__(GEMM_THREADS) void ffn_gemm_kernel(const uint16_t *__restrict__ A,
                                                                const int32_t *__restrict__ gather,
                                                                const uint16_t *__restrict__ W0,
                                                                const uint16_t *__restrict__ W1, int K, int n_tiles,
                                                                const int32_t *__restrict__ n_rows_ptr,
                                                                void *__restrict__ out, int ldo)
{
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    const int m_tiles = (*n_rows_ptr + GT - 1) / GT;  // row tiles that hold activated tokens
    if (m_tiles == 0) return;
    int tm, tn, split = 0, splits = 1;
    int half = -1;  // 0, 1: that half of the tile's activation rows only
    if (GATED) {
        // The tiles that fill whole rounds of one per CU, then the last ones: as halves, where all of them find a CU (964 rows of
        // 3584/18944: 592 tiles, the last 80 as 160 halves on 256 CUs: a layer with its selection 383 us, and 405).  A tile is
        // one of m_tiles x n_tiles, in blocks four row tiles high as below; those of a round that share an XCD follow each other.
        const int total = m_tiles * n_tiles, whole = total / 256 * 256, rest = total - whole;
        const int round = blockIdx.x >> 8, xcd = blockIdx.x & 7, idx = (blockIdx.x & 255) >> 3;
        int tile = round * 256 + xcd * 32 + idx;
        if (round * 256 >= whole) {
            if (round * 256 > whole) return;
            const bool halves = 2 * rest <= 256;
            const int n = halves ? 2 * rest : rest, per = (n + 7) / 8, x = xcd * per + idx;
            if (idx >= per || x >= n) return;
            tile = whole + (halves ? x >> 1 : x);
            if (halves) half = x & 1;
        }
        const int group = tile / (4 * n_tiles), high = min(4, m_tiles - 4 * group), in = tile - group * 4 * n_tiles;
        tm = 4 * group + in % high;
        tn = in / high;
        const bool short_tile = *n_rows_ptr - tm * GT <= GT / 2;  // nothing in its second half
        if (short_tile && half == 1) return;
        if (short_tile) half = 0;
    } else {
        splits = ffn_down_splits(m_tiles, n_tiles, K);
        // Workgroup -> tile.  Consecutive workgroups go to different XCDs (each with its own L2), so the 32 tiles of a
        // 4 x 8 block -- four row tiles that share their weights with eight weight tiles that share their rows -- are
        // given to one XCD: block k of 32 goes to XCD k % 8.
        const int total = (m_tiles + 3) / 4 * 4 * n_tiles;
        const int idx = blockIdx.x >> 3;
        const int block = (idx >> 5) * 8 + (blockIdx.x & 7), blocks = (total + 31) >> 5;  // (a split: that many blocks)
        split = block / blocks;
        const int logical = ((block - split * blocks) << 5) + (idx & 31);
        if (split >= splits || logical >= total) return;
        tm = logical / (4 * n_tiles) * 4 + (logical & 3);
        tn = (logical >> 2) % n_tiles;
        if (tm >= m_tiles) return;
    }
    const int half_row = half == 1 ? GT / 2 : 0;
    // this split's reduction steps (at least one: K / GK >= splits)
    const int k_first = (int)((long long)split * (K / GK) / splits);
    const int nk = (int)((long long)(split + 1) * (K / GK) / splits) - k_first;

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int n16 = lane & 15, q4 = lane >> 4;
    const int wm = wave >> 2, wn = wave & 3;

    // Tile loads: of either half of either tile wavefront w fills rows 16 w .. 16 w + 15, two loads.  Physical 16-byte slot
    // x of a tile holds chunk `chunk` of row `row` (vt_tile_coords); a lane's sources stay fixed over the loop.
    uint32_t voffA[2][2], voffW[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int row, chunk;
        vt_tile_coords((wave * 2 + i) * 64 + lane, row, chunk);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const long long arow = gather ? (long long)gather[tm * GT + (half < 0 ? h * 128 : half_row) + row] : (long long)(h * 128 + row);
            voffA[h][i] = (uint32_t)(arow * K * 2 + chunk * 16);
        }
        voffW[i] = (uint32_t)(row * K * 2 + chunk * 16);
    }
    const unsigned char *baseA =
        reinterpret_cast<const unsigned char *>(A) + (gather ? 0 : (size_t)tm * GT * K * 2) + (size_t)k_first * (GK * 2);
    const unsigned char *baseW[2];
#pragma unroll
    for (int h = 0; h < 2; ++h)
        baseW[h] = (GATED ? reinterpret_cast<const unsigned char *>(h == 0 ? W0 : W1) + (size_t)tn * 128 * K * 2
                          : reinterpret_cast<const unsigned char *>(W0) + ((size_t)tn * GT + h * 128) * K * 2) +
                   (size_t)k_first * (GK * 2);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem + (uint32_t)(wave * 2048));
    auto issue_a = [&](int h, int k) __attribute__((always_inline)) {
        const void *src = uniform_ptr(baseA + (size_t)k * (GK * 2));
#pragma unroll
        for (int i = 0; i < 2; ++i)
            dma_1k_s(lds0 + (uint32_t)((k & 1) * STAGE_BYTES + h * HALF_BYTES + i * 1024), src, voffA[h][i]);
    };
    auto issue_w = [&](int h, int k) __attribute__((always_inline)) {
        const void *src = uniform_ptr(baseW[h] + (size_t)k * (GK * 2));
#pragma unroll
        for (int i = 0; i < 2; ++i)
            dma_1k_s(lds0 + (uint32_t)((k & 1) * STAGE_BYTES + TILE_BYTES + h * HALF_BYTES + i * 1024), src, voffW[i]);
    };

    // Operand reads: row rb + n16 (rb a multiple of 16), chunk 4c + q4 -> rb * 128 + lo[c]
    uint32_t ra[2], rw[2];  // of stage 0: + the stage
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const uint32_t lo = (uint32_t)((n16 >> 1) * 256 + (((((n16 & 1) << 3) | (4 * c + q4)) ^ ((n16 >> 1) & 7)) << 4));
        ra[c] = lo + (uint32_t)(wm * 64 * 128);
        rw[c] = lo + (uint32_t)(TILE_BYTES + wn * 32 * 128);
    }

    f32x4 acc[8][4];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int g = 0; g < 4; ++g) acc[s][g] = f32x4{0.f, 0.f, 0.f, 0.f};

    bf16x8 a[8], w[2][4];  // operands: [c * 4 + slab] of one activation half, [weight half][c * 2 + group]
    auto read_a = [&](int h, uint32_t st) __attribute__((always_inline)) {
#pragma unroll
        for (int x = 0; x < 8; ++x)
            a[x] = *reinterpret_cast<const bf16x8 *>(smem + st + ra[x >> 2] + h * HALF_BYTES + (x & 3) * 2048);
    };
    auto read_w = [&](int st) __attribute__((always_inline)) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                w[h][x] = *reinterpret_cast<const bf16x8 *>(smem + (st + (int)rw[x >> 1]) + h * HALF_BYTES + (x & 1) * 2048);
    };
    // 32 MFMAs: activation half h times both weight halves
    auto multiply = [&](int h) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int x = 0; x < 8; ++x)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                acc[4 * h + (x & 3)][g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[g >> 1][2 * (x >> 2) + (g & 1)], a[x],
                                                                                 acc[4 * h + (x & 3)][g], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    auto issue_first = [&](int k) __attribute__((always_inline)) {  // all of a step but the second activation half
        issue_a(0, k);
        issue_w(0, k);
        issue_w(1, k);
    };
    // the barrier before the slot that reads the second activation half of step k; before the one that reads step k's rest
    auto open_second = [&](int k) __attribute__((always_inline)) {
        if (k + 1 < nk) open_slot<8>();
        else open_slot<0>();
    };
    auto open_first = [&](int k) __attribute__((always_inline)) {
        if (k + 1 < nk) open_slot<8>();
        else open_slot<2>();
    };

    if (GATED && half >= 0) {
        // Half the activation rows: a step is two slots, three stages, loads two steps ahead.  In slots (Q one later), step k is
        //   P  2k: read, load(k+2)   2k+1: multiply
        // Q's last read of step k is in slot 2k+1, before the loads of step k+3 (same stage) start in 2k+2; those of step k+1
        // have to have landed before P's read in slot 2k+2.
        auto issue_step = [&](int k) __attribute__((always_inline)) {
            const uint32_t dst = lds0 + (uint32_t)(k % 3 * HALF_STAGE);
            const void *src_a = uniform_ptr(baseA + (size_t)k * (GK * 2));
#pragma unroll
            for (int i = 0; i < 2; ++i) dma_1k_s(dst + (uint32_t)(i * 1024), src_a, voffA[0][i]);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const void *src_w = uniform_ptr(baseW[h] + (size_t)k * (GK * 2));
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    dma_1k_s(dst + (uint32_t)(HALF_BYTES + h * HALF_BYTES + i * 1024), src_w, voffW[i]);
            }
        };
        auto open_step = [&](int k) __attribute__((always_inline)) {  // the barrier before P reads step k
            if (k + 1 < nk) open_slot<6>();
            else open_slot<0>();
        };
        auto read_step = [&](int k) __attribute__((always_inline)) {
            const int st = k % 3 * HALF_STAGE;
            read_a(0, (uint32_t)st);
            read_w(st - (TILE_BYTES - HALF_BYTES));
        };
        issue_step(0);
        if (nk > 1) issue_step(1);
        open_step(0);
        if (wave < 4) {
            for (int k = 0; k < nk; ++k) {
                read_step(k);
                if (k + 2 < nk) issue_step(k + 2);
                open_slot<63>();
                multiply(0);
                open_step(k + 1);
            }
            open_slot<63>();
        } else {
            if (nk > 2) issue_step(2);
            open_slot<63>();
            for (int k = 0; k < nk; ++k) {
                read_step(k);
                open_step(k + 1);
                if (k + 3 < nk) issue_step(k + 3);
                multiply(0);
                open_slot<63>();
            }
        }
    } else {
        issue_first(0);
        issue_a(1, 0);
        if (nk > 1) issue_first(1);
        open_first(0);
        if (wave < 4) {
            for (int k = 0; k < nk; ++k) {
                const uint32_t st = (uint32_t)((k & 1) * STAGE_BYTES);
                read_a(0, st);
                read_w((int)st);
                if (k + 1 < nk) issue_a(1, k + 1);
                open_slot<63>();
                multiply(0);
                open_second(k);
                read_a(1, st);
                if (k + 2 < nk) issue_first(k + 2);
                open_slot<63>();
                multiply(1);
                open_first(k + 1);
            }
            open_slot<63>();
        } else {
            open_slot<63>();
            for (int k = 0; k < nk; ++k) {
                const uint32_t st = (uint32_t)((k & 1) * STAGE_BYTES);
                read_a(0, st);
                read_w((int)st);
                if (k + 1 < nk) issue_a(1, k + 1);
                open_second(k);
                multiply(0);
                open_slot<63>();
                read_a(1, st);
                if (k + 2 < nk) issue_first(k + 2);
                open_first(k + 1);
                multiply(1);
                open_slot<63>();
            }
        }
    }

    // Results: a lane holds output features 4*q4 .. 4*q4+3 of weight group g for the token of row n16 of slab s.
    const size_t row0 = (size_t)tm * GT + half_row + wm * 64 + n16;  // slab s: + 128 (s / 4) + 16 (s % 4)
    if (GATED) {
        uint16_t *H = static_cast<uint16_t *>(out);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            if (s >= 4 && half >= 0) break;
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                bf16x2 p0, p1;
                float h[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float z = acc[s][g][v];
                    h[v] = z / (1.0f + __expf(-z)) * acc[s][g + 2][v];
                }
                p0[0] = (__bf16)h[0]; p0[1] = (__bf16)h[1]; p1[0] = (__bf16)h[2]; p1[1] = (__bf16)h[3];
                uint2 o;
                o.x = *reinterpret_cast<uint32_t *>(&p0);
                o.y = *reinterpret_cast<uint32_t *>(&p1);
                *reinterpret_cast<uint2 *>(H + (row0 + (s >> 2) * 128 + (s & 3) * 16) * ldo + tn * 128 + wn * 32 + g * 16 + 4 * q4) = o;
            }
        }
    } else {
        float *F = static_cast<float *>(out) + (size_t)split * m_tiles * GT * ldo;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f32x4 *>(F + (row0 + (s >> 2) * 128 + (s & 3) * 16) * ldo + tn * GT + (g >> 1) * 128 + wn * 32 +
                                           (g & 1) * 16 + 4 * q4) = acc[s][g];
    }
}

template <bool GATED>
hipError_t launch_gemm(const uint16_t *A, const int32_t *gather, const uint16_t *W0, const uint16_t *W1, int K,
                       int n_tiles, long long blocks, const int32_t *n_rows, void *out, int ldo, hipStream_t st)
{
    static LdsOptIn opted;  // one per instantiation
    const hipError_t e = opted.ensure(reinterpret_cast<const void *>(&ffn_gemm_kernel<GATED>), GEMM_LDS);
    if (e != hipSuccess) return e;
    const long long grid = (blocks + 7) / 8 * 8 * 32;  // whole rounds over the eight XCDs (and so of 256 CUs)
    hipLaunchKernelGGL((ffn_gemm_kernel<GATED>), dim3((unsigned)grid), dim3(GEMM_THREADS), GEMM_LDS, st, A, gather, W0, W1, K,
                       n_tiles, n_rows, out, ldo);
    return hipGetLastError();
}

hipError_t launch_ffn_gemm_gated(const uint16_t *X, const int32_t *active, const uint16_t *Wg, const uint16_t *Wu,
                                 int d_model, int d_ff, int m_tiles, const int32_t *n_rows, uint16_t *H, hipStream_t st)
{
    return launch_gemm<true>(X, active, Wg, Wu, d_model, d_ff / 128, ffn_tile_blocks(m_tiles, d_ff / 128), n_rows, H, d_ff, st);
}

hipError_t launch_ffn_gemm_down(const uint16_t *H, const uint16_t *Wd, int d_ff, int d_model, long long blocks,
                                const int32_t *n_rows, float *F, hipStream_t st)
{
    return launch_gemm<false>(H, nullptr, Wd, nullptr, d_ff, d_model / GT, blocks, n_rows, F, d_model, st);
}

}  // namespace adaspark
