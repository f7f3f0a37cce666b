// Adaptive Token-Selective FFN (Sec. 3.3): everything around the two matrix products --
//   ffn_select_kernel   token norms, importance scores, Top-p token selection per cube (Eqs. 4-5)
//   ffn_count_kernel / ffn_fill_kernel   the lists of activated and of other tokens in cube order
//   ffn_finish_kernel   residual sums and mean compensation (Eqs. 6-7)
// One workgroup per cube in all of them (and, in the last, block of columns).
#include <algorithm>

#include "ffn.h"

namespace adaspark {

constexpr int SEL_THREADS = 1024;
constexpr int TAB_THREADS = 256;
constexpr int FINISH_SMALL_TOKENS = 100;  // finish_small

__device__ __forceinline__ float wave_sum(float x)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// Sum of n floats held in LDS, in a fixed order (the same on every run): per-thread strided partial sums, then a
// tree over the wavefronts.  All threads get the result.  `red` holds one float per wavefront.
template <int THREADS>
__device__ float block_sum(const float *vals, int n, float *red)
{
    float acc = 0.f;
    for (int j = threadIdx.x; j < n; j += THREADS) acc += vals[j];
    acc = wave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) tot += red[w];
    return tot;
}

// Eqs. 4-5 for cube blockIdx.x.  INFLIGHT: tokens of a wavefront whose loads are on the way together -- 4, whose sums then
// stay in registers over a token's pieces; 16 where a token is a single piece per lane (d_model <= 512) and a cube has tokens
// for it, so that 256 tokens are one trip to memory and not four.
template <int INFLIGHT>
__global__ __launch_bounds__(SEL_THREADS) void ffn_select_kernel(Geom g, int d_model, const uint16_t *__restrict__ X,
                                                                 float top_p, float eps, uint8_t *__restrict__ keep,
                                                                 float *__restrict__ score, int32_t *__restrict__ keep_count)
{
    extern __shared__ float sm[];
    float *sc = sm;                 // [Cmax] norms, then scores
    float *red = sm + g.Cmax;       // [SEL_THREADS / 64]
    int *cnt = reinterpret_cast<int *>(red + SEL_THREADS / 64);
    const int c = blockIdx.x;
    const CubeBox b = cube_box(g, c);
    const int n = b.size();
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int chunks = d_model / 8;  // 16-byte pieces of a token
    if (threadIdx.x == 0) *cnt = 0;

    // token norms: a wavefront per token, INFLIGHT tokens in flight
    constexpr int NW = SEL_THREADS / 64;
    for (int r0 = wave; r0 < n; r0 += INFLIGHT * NW) {
        const uint16_t *x[INFLIGHT];
        float a[INFLIGHT];
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u) {
            const int r = r0 + u * NW;
            x[u] = X + (size_t)token_of(g, b, r < n ? r : r0) * d_model;
            a[u] = 0.f;
        }
        for (int k = lane; k < chunks; k += 64) {
            u32x4 v[INFLIGHT];
#pragma unroll
            for (int u = 0; u < INFLIGHT; ++u) v[u] = *reinterpret_cast<const u32x4 *>(x[u] + 8 * k);
#pragma unroll
            for (int u = 0; u < INFLIGHT; ++u)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float lo = __uint_as_float(v[u][e] << 16), hi = __uint_as_float(v[u][e] & 0xffff0000u);
                    a[u] = fmaf(lo, lo, a[u]);
                    a[u] = fmaf(hi, hi, a[u]);
                }
        }
#pragma unroll
        for (int u = 0; u < INFLIGHT; ++u) {
            const float tot = wave_sum(a[u]);
            const int r = r0 + u * NW;
            if (lane == 0 && r < n) sc[r] = sqrtf(tot);
        }
    }
    __syncthreads();
    const float total = block_sum<SEL_THREADS>(sc, n, red);
    // a cube of zero-norm tokens with eps = 0: every score is 0 (Eq. 4's epsilon is there for this cube)
    const float inv = (total + eps > 0.f) ? 1.0f / (total + eps) : 0.f;
    __syncthreads();
    for (int j = threadIdx.x; j < n; j += SEL_THREADS) sc[j] = sc[j] * inv;
    __syncthreads();

    const bool text = b.t0 < 0;
    int mine = 0;
    for (int j = threadIdx.x; j < n; j += SEL_THREADS) {
        const float sj = sc[j];
        bool k = true;
        if (!text && top_p < 1.0f) {
            // mass of the tokens ranked before j (larger score, or equal score and lower rank), added in rank order: those below
            // the wavefront's tokens, these, those above
            float before = 0.f;
            const int w0 = __builtin_amdgcn_readfirstlane(j - lane), w1 = min(n, w0 + 64);
#pragma unroll 8
            for (int i = 0; i < w0; ++i) before += sc[i] >= sj ? sc[i] : 0.f;
#pragma unroll 4
            for (int i = w0; i < w1; ++i) {
                const float si = sc[i];
                before += si > sj || (si == sj && i < j) ? si : 0.f;
            }
#pragma unroll 8
            for (int i = w1; i < n; ++i) before += sc[i] > sj ? sc[i] : 0.f;
            k = before < top_p;
        }
        const int tok = token_of(g, b, j);
        keep[tok] = k ? 1 : 0;
        if (score) score[tok] = sj;
        mine += k ? 1 : 0;
    }
    if (keep_count) {
        if (mine) atomicAdd(cnt, mine);
        __syncthreads();
        if (threadIdx.x == 0) keep_count[c] = *cnt;
    }
}

// Activated tokens per cube.
__global__ __launch_bounds__(TAB_THREADS) void ffn_count_kernel(Geom g, const uint8_t *__restrict__ keep,
                                                                int32_t *__restrict__ cnt)
{
    __shared__ int tot;
    const CubeBox b = cube_box(g, blockIdx.x);
    const int n = b.size();
    if (threadIdx.x == 0) tot = 0;
    __syncthreads();
    int mine = 0;
    if (keep == nullptr) {
        if (threadIdx.x == 0) mine = n;
    } else {
        for (int j = threadIdx.x; j < n; j += TAB_THREADS) mine += keep[token_of(g, b, j)] != 0;
    }
    if (mine) atomicAdd(&tot, mine);
    __syncthreads();
    if (threadIdx.x == 0) cnt[blockIdx.x] = tot;
}

// cube_ptr[c] = activated tokens of the cubes before c; active[cube_ptr[c] + k] = k-th activated token of cube c in
// rank order; bypass[tokens of the cubes before c - cube_ptr[c] + k] = k-th of its other tokens.  The last cube also
// writes cube_ptr[N] and pads `active` with token 0 up to a multiple of FFN_ROW_TILE (rows that the matrix products
// compute and nobody reads).
__global__ __launch_bounds__(TAB_THREADS) void ffn_fill_kernel(Geom g, const uint8_t *__restrict__ keep,
                                                               const int32_t *__restrict__ cnt,
                                                               int32_t *__restrict__ cube_ptr, int32_t *__restrict__ active,
                                                               int32_t *__restrict__ bypass)
{
    __shared__ int part[TAB_THREADS], tpart[TAB_THREADS];
    const int c = blockIdx.x;
    const CubeBox b = cube_box(g, c);
    const int n = b.size();
    // offsets of this cube: activated tokens, and tokens, of the cubes before it
    int acc = 0, tacc = 0;
    for (int i = threadIdx.x; i < c; i += TAB_THREADS) {
        acc += cnt[i];
        tacc += cube_box(g, i).size();
    }
    part[threadIdx.x] = acc;
    tpart[threadIdx.x] = tacc;
    __syncthreads();
    for (int d = TAB_THREADS / 2; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) {
            part[threadIdx.x] += part[threadIdx.x + d];
            tpart[threadIdx.x] += tpart[threadIdx.x + d];
        }
        __syncthreads();
    }
    const int base = part[0], tbase = tpart[0];
    __syncthreads();

    // every thread takes a run of consecutive ranks; exclusive scan of the runs' counts
    const int per = (n + TAB_THREADS - 1) / TAB_THREADS;
    const int j0 = min(n, (int)threadIdx.x * per), j1 = min(n, j0 + per);
    int mine = 0;
    for (int j = j0; j < j1; ++j) mine += keep == nullptr || keep[token_of(g, b, j)] != 0;
    part[threadIdx.x] = mine;
    __syncthreads();
    for (int d = 1; d < TAB_THREADS; d <<= 1) {
        const int v = (int)threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    int pos = base + part[threadIdx.x] - mine;
    for (int j = j0; j < j1; ++j) {
        const int tok = token_of(g, b, j);
        if (keep == nullptr || keep[tok] != 0) active[pos++] = tok;
        else bypass[tbase + j - pos] = tok;  // (j - (pos - base) of the cube's tokens before j are bypassed)
    }
    if (threadIdx.x == 0) cube_ptr[c] = base;
    if (c == g.N - 1) {
        const int total = base + part[TAB_THREADS - 1];
        if (threadIdx.x == 0) cube_ptr[g.N] = total;
        const int padded = (total + FFN_ROW_TILE - 1) / FFN_ROW_TILE * FFN_ROW_TILE;
        for (int i = total + threadIdx.x; i < padded; i += TAB_THREADS) active[i] = 0;
    }
}

// Eqs. 6-7 for cube blockIdx.x and columns COLS blockIdx.y ..: F holds FFN(x) of the activated tokens (fp32, row = index in
// the active list), in `splits` parts that are added in order.  A lane owns eight columns of every (WAVES * 512 / COLS)-th
// activated token: y = x + F, and a sum of F; the lanes' sums are combined in a fixed order; then of every so many-th
// bypassed token: x + mean.  Bound by memory (F, X and Y once each) with WAVES = 4, COLS = 512: 65,536 tokens of 3584, 47 %
// activated, 0.27 ms = 5.1 TB/s.  With few cubes by the trips to memory that a wavefront makes one after the other:
// finish_small.
template <int WAVES, int COLS>
__global__ __launch_bounds__(64 * WAVES) void ffn_finish_kernel(Geom g, int d_model, int d_ff, const uint16_t *__restrict__ X,
                                                                const float *__restrict__ F,
                                                                const int32_t *__restrict__ cube_ptr,
                                                                const int32_t *__restrict__ active,
                                                                const int32_t *__restrict__ bypass, uint16_t *__restrict__ Y)
{
    constexpr int THREADS = 64 * WAVES, LANES = COLS / 8, TOKENS = THREADS / LANES;  // lanes of a token, tokens at a time
    __shared__ f32x4 sums[2][WAVES][LANES];
    __shared__ int tpart[WAVES];
    const int c = blockIdx.x;
    const int tid = threadIdx.x;
    // tokens of the cubes before this one: the start of its bypassed tokens (see ffn_fill_kernel)
    int tacc = 0;
    for (int i = tid; i < c; i += THREADS) tacc += cube_box(g, i).size();
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) tacc += __shfl_xor(tacc, d, 64);
    if ((tid & 63) == 0) tpart[tid >> 6] = tacc;
    __syncthreads();
    int tbase = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) tbase += tpart[w];
    const int n = cube_box(g, c).size();
    const int first = cube_ptr[c], count = cube_ptr[c + 1] - first;
    const float inv = count > 0 ? 1.0f / (float)count : 0.f;
    const int m_tiles = (cube_ptr[g.N] + FFN_ROW_TILE - 1) / FFN_ROW_TILE;
    const int splits = count > 0 ? ffn_down_splits(m_tiles, d_model / FFN_ROW_TILE, d_ff) : 1;
    const size_t part = (size_t)m_tiles * FFN_ROW_TILE * d_model;
    const int slot = LANES == 64 ? __builtin_amdgcn_readfirstlane(tid / 64) : tid / LANES;  // (scalar addresses)
    const int col = COLS * blockIdx.y + 8 * (tid % LANES);
    const bool on = col < d_model;

    auto add_store = [&](int tok, const u32x4 &xv, const f32x4 &f0, const f32x4 &f1) __attribute__((always_inline)) {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float lo = __uint_as_float(xv[e] << 16) + (e < 2 ? f0[2 * e] : f1[2 * e - 4]);
            const float hi = __uint_as_float(xv[e] & 0xffff0000u) + (e < 2 ? f0[2 * e + 1] : f1[2 * e - 3]);
            o[e] = (uint32_t)float_to_bf16_bits(lo) | ((uint32_t)float_to_bf16_bits(hi) << 16);
        }
        *reinterpret_cast<u32x4 *>(Y + (size_t)tok * d_model + col) = o;
    };
    constexpr int U = WAVES == 4 ? 4 : 1, PARTS = 8 / U;  // tokens, and parts, in flight
    f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
    if (on) {
        for (int r0 = slot; r0 < count; r0 += U * TOKENS) {
            f32x4 v0[U], v1[U];
            u32x4 xv[U];
            int tok[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int r = min(r0 + u * TOKENS, count - 1);  // (past the end: loaded, not used)
                const float *f = F + (size_t)(first + r) * d_model + col;
                v0[u] = *reinterpret_cast<const f32x4 *>(f);
                v1[u] = *reinterpret_cast<const f32x4 *>(f + 4);
                tok[u] = active[first + r];
                xv[u] = *reinterpret_cast<const u32x4 *>(X + (size_t)tok[u] * d_model + col);
            }
#pragma unroll PARTS
            for (int p = 1; p < splits; ++p)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const float *f = F + p * part + (size_t)(first + min(r0 + u * TOKENS, count - 1)) * d_model + col;
                    v0[u] += *reinterpret_cast<const f32x4 *>(f);
                    v1[u] += *reinterpret_cast<const f32x4 *>(f + 4);
                }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (r0 + u * TOKENS < count) {
                    acc0 += v0[u];
                    acc1 += v1[u];
                    add_store(tok[u], xv[u], v0[u], v1[u]);
                }
        }
    }
    // the tokens of a wavefront, then the wavefronts
#pragma unroll
    for (int d = LANES; d < 64; d <<= 1)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc0[e] += __shfl_xor(acc0[e], d, 64);
            acc1[e] += __shfl_xor(acc1[e], d, 64);
        }
    if ((tid & 63) < LANES) {
        sums[0][tid >> 6][tid % LANES] = acc0;
        sums[1][tid >> 6][tid % LANES] = acc1;
    }
    __syncthreads();
    f32x4 mean0 = sums[0][0][tid % LANES], mean1 = sums[1][0][tid % LANES];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
        mean0 += sums[0][w][tid % LANES];
        mean1 += sums[1][w][tid % LANES];
    }
    mean0 *= inv;
    mean1 *= inv;
    if (!on) return;
    const int32_t *others = bypass + (tbase - first);
    for (int r0 = slot; r0 < n - count; r0 += U * TOKENS) {
        u32x4 xv[U];
        int tok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            tok[u] = others[min(r0 + u * TOKENS, n - count - 1)];
            xv[u] = *reinterpret_cast<const u32x4 *>(X + (size_t)tok[u] * d_model + col);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (r0 + u * TOKENS < n - count) add_store(tok[u], xv[u], mean0, mean1);
    }
}

hipError_t launch_ffn_select(const Geom &g, int d_model, const uint16_t *X, float top_p, float eps, uint8_t *keep,
                             float *score, int32_t *keep_count, hipStream_t st)
{
    const size_t lds = (size_t)(g.Cmax + SEL_THREADS / 64 + 4) * sizeof(float);
    if (d_model <= 512 && g.Cmax >= 128)
        hipLaunchKernelGGL(ffn_select_kernel<16>, dim3(g.N), dim3(SEL_THREADS), lds, st, g, d_model, X, top_p, eps, keep,
                           score, keep_count);
    else
        hipLaunchKernelGGL(ffn_select_kernel<4>, dim3(g.N), dim3(SEL_THREADS), lds, st, g, d_model, X, top_p, eps, keep,
                           score, keep_count);
    return hipGetLastError();
}

FfnWorkspace ffn_workspace(const Geom &g, int d_model, int d_ff, void *ws)
{
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t rows = ((size_t)g.S + FFN_ROW_TILE - 1) / FFN_ROW_TILE * FFN_ROW_TILE;
    FfnWorkspace w;
    unsigned char *p = static_cast<unsigned char *>(ws);
    size_t off = 0;
    w.cnt = reinterpret_cast<int32_t *>(p + off); off = up(off + (size_t)g.N * 4);
    w.cube_ptr = reinterpret_cast<int32_t *>(p + off); off = up(off + (size_t)(g.N + 1) * 4);
    w.active = reinterpret_cast<int32_t *>(p + off); off = up(off + rows * 4);
    w.bypass = reinterpret_cast<int32_t *>(p + off); off = up(off + (size_t)g.S * 4);
    w.H = reinterpret_cast<uint16_t *>(p + off); off = up(off + rows * (size_t)d_ff * 2);
    // F: one part for all rows, or several for few of them (ffn_down_splits).  How many rows there are is known on the
    // device: room, and a grid, for the row-tile count that takes most.
    const int m_tiles = (int)(rows / FFN_ROW_TILE), n_tiles = d_model / FFN_ROW_TILE;
    size_t f_tiles = (size_t)m_tiles * n_tiles;
    w.down_blocks = ffn_tile_blocks(m_tiles, n_tiles);
    for (int m = 1; m <= m_tiles && m * n_tiles <= FFN_SPLIT_TILES / 2; ++m) {  // (with more tiles there is one part)
        const int splits = ffn_down_splits(m, n_tiles, d_ff);
        f_tiles = std::max(f_tiles, (size_t)splits * m * n_tiles);
        w.down_blocks = std::max(w.down_blocks, splits * ffn_tile_blocks(m, n_tiles));
    }
    w.F = reinterpret_cast<float *>(p + off); off = up(off + f_tiles * FFN_ROW_TILE * FFN_ROW_TILE * 4);
    w.bytes = off;
    w.rows = (long long)rows;
    return w;
}

// Whether a cube's rows are shared out among sixteen wavefronts, 64 columns each, by the residual kernel: where the workgroups
// of four wavefronts and 512 columns leave CUs idle, and the largest cube, which is then the kernel's time, has rows for all.  A
// layer with its selection of d_model 512 and d_ff 2,560, us, so and with four wavefronts, by such workgroups: cubes of 36 tokens, 50 74, 73; of 120,
// 50 90, 97, 85 118, 117; of 128, 48 91, 98, 88 117, 117, 120 148, 141; of 256, 48 122, 142, 120 203, 206, 152 260, 253; of 512, 140 455, 478.
// The same lines with cubes that the grid clips to a few tokens beside these, and at d_model 1,024 to 3,584.
static bool finish_small(const Geom &g, int d_model)
{
    const int largest = std::max(min(g.ct, g.T) * min(g.ch, g.H) * min(g.cw, g.W), min(g.Cmax, std::max(g.Sp, g.St)));
    const long long blocks = (long long)g.N * ((d_model + 511) / 512);
    return largest >= FINISH_SMALL_TOKENS && blocks <= 45 + 3LL * largest / 8;
}

hipError_t launch_ffn_sparse(const Geom &g, int d_model, int d_ff, const uint16_t *X, const uint16_t *Wg,
                             const uint16_t *Wu, const uint16_t *Wd, const uint8_t *keep, uint16_t *Y,
                             const FfnWorkspace &w, hipStream_t st)
{
    hipLaunchKernelGGL(ffn_count_kernel, dim3(g.N), dim3(TAB_THREADS), 0, st, g, keep, w.cnt);
    hipLaunchKernelGGL(ffn_fill_kernel, dim3(g.N), dim3(TAB_THREADS), 0, st, g, keep, w.cnt, w.cube_ptr, w.active,
                       w.bypass);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int m_tiles = (int)(w.rows / FFN_ROW_TILE);
    // hidden activations of the activated tokens, then the layer's output for them
    e = launch_ffn_gemm_gated(X, w.active, Wg, Wu, d_model, d_ff, m_tiles, w.cube_ptr + g.N, w.H, st);
    if (e != hipSuccess) return e;
    e = launch_ffn_gemm_down(w.H, Wd, d_ff, d_model, w.down_blocks, w.cube_ptr + g.N, w.F, st);
    if (e != hipSuccess) return e;
    if (finish_small(g, d_model))
        hipLaunchKernelGGL((ffn_finish_kernel<16, 64>), dim3(g.N, d_model / 64), dim3(1024), 0, st, g, d_model, d_ff, X, w.F,
                           w.cube_ptr, w.active, w.bypass, Y);
    else
        hipLaunchKernelGGL((ffn_finish_kernel<4, 512>), dim3(g.N, (d_model + 511) / 512), dim3(256), 0, st, g, d_model, d_ff, X,
                           w.F, w.cube_ptr, w.active, w.bypass, Y);
    return hipGetLastError();
}

}  // namespace adaspark
