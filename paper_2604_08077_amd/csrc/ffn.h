// Internal interface of the token-selective FFN (Sec. 3.3): ffn.hip (selection, tables, mean compensation) and
// ffn_gemm.hip (the two matrix products on the activated tokens).
#pragma once
#include "kvtile.h"

namespace adaspark {

constexpr int FFN_ROW_TILE = 256;        // activated tokens per workgroup of the matrix products
constexpr int FFN_MAX_CUBE_TOKENS = 4096;

constexpr int FFN_SPLIT_TILES = 1024;    // most (tile, split) pairs of a split W_down product

// How many workgroups share the reduction of one 256 x 256 tile of the W_down product (m_tiles x n_tiles tiles, d_ff
// long), each leaving an fp32 partial result.  One tile per CU and d_ff / 64 steps of 1.4 us each otherwise: few activated
// tokens leave most of the chip idle.  The cost model: the rounds of workgroups over 256 CUs times the steps of one, and 0.1 us
// of the chip's memory time per partial tile (512 KB written and read).  964 activated tokens, 3584/18944 (56 tiles):
// 4 splits, 130 us; unsplit 381 to 444.  2,048 tokens (112 tiles): 2 splits, 251 us, and 18 to add the parts; 4 splits, 263
// and 27; unsplit 425 and 13.
__host__ __device__ inline int ffn_down_splits(int m_tiles, int n_tiles, int d_ff)
{
    const int tiles = m_tiles * n_tiles, steps = d_ff / 64;
    int best = 1;
    long long least = 0;
#pragma unroll
    for (int s = 1; s <= 16; ++s) {
        if (s > 1 && (tiles > FFN_SPLIT_TILES / s || steps < 2 * s)) break;
        const long long cost = (long long)((tiles * s + 255) / 256) * ((steps + s - 1) / s) * 14 + (long long)tiles * s;
        if (s == 1 || cost < least) {
            least = cost;
            best = s;
        }
    }
    return best;
}

// Views into the caller's workspace.
struct FfnWorkspace {
    int32_t *cnt;       // [N]      activated tokens per cube
    int32_t *cube_ptr;  // [N + 1]  exclusive prefix sums of cnt; cube_ptr[N] = number of activated tokens
    int32_t *active;    // [rows]   activated tokens, cube by cube in rank order, padded to a multiple of FFN_ROW_TILE
    int32_t *bypass;    // [S]      the other tokens, cube by cube in rank order
    uint16_t *H;        // [rows][d_ff]     bf16 hidden activations silu(gate) * up
    float *F;           // [splits][rows up to the activated ones'][d_model]  fp32 FFN(x) of the activated tokens, in as
                        //          many parts as the W_down product was split into
    long long rows;     // S rounded up to a multiple of FFN_ROW_TILE
    long long down_blocks;  // blocks of 32 tiles that the W_down product's grid has to cover, however many tokens are activated
    size_t bytes;
};
FfnWorkspace ffn_workspace(const Geom &g, int d_model, int d_ff, void *ws);

hipError_t launch_ffn_select(const Geom &g, int d_model, const uint16_t *X, float top_p, float eps, uint8_t *keep,
                             float *score, int32_t *keep_count, hipStream_t st);
hipError_t launch_ffn_sparse(const Geom &g, int d_model, int d_ff, const uint16_t *X, const uint16_t *Wg,
                             const uint16_t *Wu, const uint16_t *Wd, const uint8_t *keep, uint16_t *Y,
                             const FfnWorkspace &w, hipStream_t st);

// H[r][:] = silu(W_gate . x) * (W_up . x) for x = X[active[r]], r < *n_rows (rows up to the next multiple of half a
// FFN_ROW_TILE, or of a whole one, are computed too, from the padding of `active`; those behind them hold what they held).  m_tiles: upper bound of row tiles (grid size).
hipError_t launch_ffn_gemm_gated(const uint16_t *X, const int32_t *active, const uint16_t *Wg, const uint16_t *Wu,
                                 int d_model, int d_ff, int m_tiles, const int32_t *n_rows, uint16_t *H, hipStream_t st);
// F[split][r][:]: over the splits (ffn_down_splits) summing to W_down . H[r][:], in fp32.  blocks: FfnWorkspace::down_blocks.
hipError_t launch_ffn_gemm_down(const uint16_t *H, const uint16_t *Wd, int d_ff, int d_model, long long blocks,
                                const int32_t *n_rows, float *F, hipStream_t st);
// Blocks of 32 tiles for m_tiles row tiles (a multiple of four of them: a block is four row tiles high).
inline long long ffn_tile_blocks(long long m_tiles, int n_tiles) { return ((m_tiles + 3) / 4 * 4 * n_tiles + 31) / 32; }

}  // namespace adaspark
