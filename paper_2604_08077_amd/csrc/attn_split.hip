// Attention for short sequences (dense, or sparse with the selection as a mask): the wavefronts of a workgroup share
// the KEYS of one small block of rows instead of the rows of a big one.
//
// The walk kernel (attn_walk.hip) gives a workgroup 256 rows of a KV head and one walk over all keys, tile by tile with a
// barrier each.  On a short sequence that leaves most of the chip idle -- 2,048 tokens of 4 heads are 32 workgroups, and the
// time is the latency of the longest walk -- so here a workgroup takes 32 rows, and its eight wavefronts take every eighth 32-key step of their walk,
// operands straight from memory (the packed copy is in operand order, and nobody else on the CU wants the same tile).
// The eight partial results (running reference, sum, unnormalised O, all fp32) are combined through LDS at the end.
// Cubes in which no row of the block takes part (selection) are left out of the walk.
//
// Bound by the latency of a step at the smallest sizes and by L2 above (every wavefront fetches 16 KB at head-dim 128
// for 34 MFMAs: 12 to 15 TB/s over the chip), which is why the walk kernel takes over as soon as it fills the chip
// (attn_split_pays).  2,048 tokens, 4/4 heads of 64, cubes of 32: 18.1 us, the walk kernel 98 us; 1,080 tokens, 6/2 heads
// of 128, clipped cubes of up to 128: 19.1 against 48 us.
#include <type_traits>

#include "attn_tile.h"

namespace adaspark {

template <int D>
struct Split {
    static constexpr int WAVES = 8;
    static constexpr int THREADS = 64 * WAVES;
    static constexpr int NS = FWD_NS;
    static constexpr int ROWS = 16 * NS;
    static constexpr int STEP = 32;  // keys per step
    static constexpr int DT = D / 16;
    static constexpr int OFF_ML = WAVES * NS * DT * 1024;     // after the wavefronts' O: m and l of their rows
    static constexpr int OFF_UNION = OFF_ML + WAVES * ROWS * 8;
    static constexpr int OFF_N = OFF_UNION + ADASPARK_MAX_CUBES / 8;
    static constexpr int BYTES = OFF_N + 16;
    // the list of steps lies where the wavefronts' O goes at the end
    static constexpr int LIST_MAX = OFF_ML / 4;
};

bool attn_split_fits(const Geom &g)
{
    const long long steps = (long long)g.N * ((g.Cmax + Split<64>::STEP - 1) / Split<64>::STEP);
    return steps <= (g.D == 64 ? Split<64>::LIST_MAX : Split<128>::LIST_MAX) && g.Cmax <= 65536 * Split<64>::STEP / 2;
}

template <int D, bool MASKED>
__global__ __launch_bounds__(512) void attn_split_kernel(Geom g, const uint16_t *__restrict__ Q,
                                                         const uint16_t *__restrict__ Kp, const uint16_t *__restrict__ Vt,
                                                         const int32_t *__restrict__ csize,
                                                         const uint32_t *__restrict__ sel_mask,
                                                         const int *__restrict__ mode_flag, int my_mode,
                                                         uint16_t *__restrict__ O, float *__restrict__ lse)
{
    if (MASKED && mode_flag != nullptr && mode_flag[FLAG_MODE] != my_mode) return;
    using C = Split<D>;
    constexpr int NS = C::NS, KSTEPS = D / 32, DT = C::DT;
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];
    uint32_t *list = reinterpret_cast<uint32_t *>(smem);  // steps of the walk: cube << 16 | step of the cube
    uint32_t *uni = reinterpret_cast<uint32_t *>(smem + C::OFF_UNION);
    int *nsteps_s = reinterpret_cast<int *>(smem + C::OFF_N);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, q4 = lane >> 4;

    // workgroup -> (KV head, block of 32 rows), late rows (long walks) first.  A KV head's rows are numbered as in the walk
    // kernel, cube by cube and in a cube head by head, and cut into blocks across the cubes' borders: a block per cube leaves
    // most of its rows empty where cubes are clipped to a few tokens.  Consecutive workgroups are of different heads, so that
    // an XCD's L2 sees the tiles of few of them.
    const int kv = blockIdx.x % g.Hkv;
    const int row1 = g.S * g.G - (int)(blockIdx.x / g.Hkv) * C::ROWS, row0 = max(0, row1 - C::ROWS), last = row1 - 1;
    // Lane l works out row l % 32 (rows past the last one repeat it), and the lanes that hold a row's column fetch its place.
    const RowAt at = row_at(g, kv, min(row0 + (lane & 31), last));
    int rank[NS], own[NS];
    size_t rowid[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        rank[s] = __shfl(at.rank, 16 * s + n16, 64);
        own[s] = __shfl(at.cube, 16 * s + n16, 64);
        rowid[s] = (size_t)__shfl(at.id, 16 * s + n16, 64);
    }
    // the last cube with rows here, and the first
    const int i = __builtin_amdgcn_readlane(at.cube, 31), i_first = __builtin_amdgcn_readfirstlane(at.cube);
    const int max_rank = __builtin_amdgcn_readlane(block_max_rank(at, row1 - row0), 31);  // of the block's rows in cube i
    const float c2 = 1.44269504088896340736f / sqrtf((float)D);  // softmax scale in base 2, folded into Q
    bf16x8 qf[NS][KSTEPS];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
            qf[s][c] = score_operand(*reinterpret_cast<const bf16x8 *>(Q + rowid[s] * D + 32 * c + 8 * q4), c2);

    // ---- the steps of the walk: the rows' own cubes, the last one up to the block's largest rank, and of the others those
    // that a row selected
    const int ncubes = g.causal ? i + 1 : g.N;
    if (MASKED) {
        // wavefront w takes mask words w, w + 8, ...; its lanes are the block's rows, twice over
        for (int w = wave; 32 * w < ncubes; w += C::WAVES) {
            uint32_t m = sel_mask[rowid[(lane >> 4) & 1] * g.words + w];
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) m |= __shfl_xor(m, d, 64);
            if (lane == 0) uni[w] = m;
        }
        __syncthreads();
    }
    if (wave == 0) {
        int n = 0;
        for (int c0 = 0; c0 < ncubes; c0 += 64) {
            const int c = c0 + lane;
            int steps = 0;
            if (c < ncubes) {
                const int size = c == i && g.causal ? max_rank + 1 : g.ragged ? csize[c] : g.Cmax;
                if ((c >= i_first && c <= i) || !MASKED || ((uni[c >> 5] >> (c & 31)) & 1u)) steps = (size + C::STEP - 1) / C::STEP;
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

    // ---- this wavefront's steps: wave, wave + 8, ...  The K operands of the next step are loaded when this one's scores
    // are done, its V^T operands when this one's P.V is done.
    const size_t head = (size_t)kv * g.N * g.TPC * (KEY_TILE * D);
    bf16x8 kf[KSTEPS][2], vf[DT];
    uint32_t word[NS], word_next[NS];
    auto entry = [&](int p) -> uint32_t {  // (past the end the last step's operands are loaded, and not used)
        return __builtin_amdgcn_readfirstlane(list[min(p, nsteps - 1)]);
    };
    auto load_k = [&](uint32_t e) __attribute__((always_inline)) {
        const int j = (int)(e >> 16), k = (int)(e & 0xffffu);
        const unsigned char *kt = reinterpret_cast<const unsigned char *>(Kp + head + ((size_t)j * g.TPC + (k >> 1)) * (KEY_TILE * D));
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2) {
                const int krow = 32 * (k & 1) + 8 * (n16 >> 2) + 4 * k2 + (n16 & 3);
                kf[c][k2] = *reinterpret_cast<const bf16x8 *>(kt + k_tile_off<D>(krow, 4 * c + q4));
            }
        if (MASKED) {
#pragma unroll
            for (int s = 0; s < NS; ++s) word_next[s] = sel_mask[rowid[s] * g.words + (j >> 5)];
        }
    };
    auto load_v = [&](uint32_t e) __attribute__((always_inline)) {
        const int j = (int)(e >> 16), k = (int)(e & 0xffffu);
        const unsigned char *vt = reinterpret_cast<const unsigned char *>(Vt + head + ((size_t)j * g.TPC + (k >> 1)) * (KEY_TILE * D));
#pragma unroll
        for (int e2 = 0; e2 < DT; ++e2)
            vf[e2] = *reinterpret_cast<const bf16x8 *>(vt + vt_tile_off(16 * e2 + n16, 4 * (k & 1) + q4));
    };
    float m_run[NS];
    bool fresh[NS];
    f32x4 l_run[NS], oacc[NS][DT];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        m_run[s] = 0.f;
        fresh[s] = true;
        l_run[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < DT; ++e) oacc[s][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // The step e0; e1 is the next one.  BEHIND: of a cube behind some rows' own.  These rows' probabilities are zero there, but V
    // need not be finite (0 * inf): they keep their O.
    auto work = [&](uint32_t e0, uint32_t e1, auto behind) __attribute__((always_inline)) {
        constexpr bool BEHIND = decltype(behind)::value;
        const int j = (int)(e0 >> 16);
        const bool edge = j >= i_first;  // some row's own cube, or (causal) behind it
        const int jsize = g.ragged ? csize[j] : g.Cmax;
        const int key0 = C::STEP * (int)(e0 & 0xffffu);
#pragma unroll
        for (int s = 0; s < NS; ++s) word[s] = MASKED ? word_next[s] : 0u;
        f32x4 sa[NS][2];
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c)
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    // (from minus the reference point of the row's exponentials, -inf for a row that takes no part)
                    bool in = !MASKED || ((word[s] >> (j & 31)) & 1u);
                    if (MASKED && edge) in = j == own[s] || (in && (!g.causal || j < own[s]));
                    const float b = in ? -m_run[s] : -INFINITY;
                    sa[s][k2] = score_mfma(kf[c][k2], qf[s][c], c == 0 ? f32x4{b, b, b, b} : sa[s][k2]);
                }
        load_k(e1);
        if (key0 + C::STEP > jsize || (edge && g.causal)) {
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const int lim = !g.causal || j < own[s] ? jsize - 1 : j == own[s] ? min(rank[s], jsize - 1) : -1;
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (key0 + 8 * q4 + 4 * k2 + v > lim) sa[s][k2][v] = -INFINITY;
            }
        }
        float mx[NS];
        bool grow[NS], any = false;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            mx[s] = vmax3(vmax3(sa[s][0][0], sa[s][0][1], sa[s][0][2]), vmax3(sa[s][0][3], sa[s][1][0], sa[s][1][1]),
                          vmax(sa[s][1][2], sa[s][1][3]));
            mx[s] = quad_max(mx[s]);
            grow[s] = (mx[s] >= SOFTMAX_LAZY) | (fresh[s] & (mx[s] > -INFINITY));
            any = any || grow[s];
        }
        if (__ballot(any) != 0ull) {  // (as in softmax_tile_folded)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const float d = grow[s] ? mx[s] + SOFTMAX_HEADROOM : 0.f;
                const float alpha = (grow[s] && !fresh[s]) ? __builtin_amdgcn_exp2f(-d) : 1.f;
                m_run[s] += d;
                fresh[s] = fresh[s] && !grow[s];
#pragma unroll
                for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sa[s][k2][v] -= d;
#pragma unroll
                for (int e = 0; e < DT; ++e) oacc[s][e] *= alpha;
                l_run[s] *= alpha;
            }
        }
        bf16x8 pf[NS];
        const bf16x8 ones = ones_operand();
#pragma unroll
        for (int s = 0; s < NS; ++s) {
#pragma unroll
            for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
                for (int v = 0; v < 4; ++v) pf[s][4 * k2 + v] = (__bf16)__builtin_amdgcn_exp2f(sa[s][k2][v]);
            l_run[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[s], l_run[s], 0, 0, 0);
        }
#pragma unroll
        for (int e = 0; e < DT; ++e)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const f32x4 sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[e], pf[s], oacc[s][e], 0, 0, 0);
                oacc[s][e] = BEHIND && j > own[s] ? oacc[s][e] : sum;
            }
        load_v(e1);
    };
    if (wave < nsteps) {
        uint32_t e0 = entry(wave);
        load_k(e0);
        load_v(e0);
        int p = wave;
        const uint32_t behind = g.causal ? (uint32_t)(i_first + 1) << 16 : ~0u;  // the first such step
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

    // ---- combine the wavefronts' parts: O = sum_w 2^(m_w - M) O_w / sum_w 2^(m_w - M) l_w
    f32x4 *part = reinterpret_cast<f32x4 *>(smem);  // [wave][s][e][lane]
    float2 *ml = reinterpret_cast<float2 *>(smem + C::OFF_ML);  // [wave][row]
#pragma unroll
    for (int s = 0; s < NS; ++s) {
#pragma unroll
        for (int e = 0; e < DT; ++e) part[((wave * NS + s) * DT + e) * 64 + lane] = oacc[s][e];
        if (q4 == 0) ml[wave * C::ROWS + 16 * s + n16] = make_float2(fresh[s] ? -INFINITY : m_run[s], l_run[s][0]);
    }
    __syncthreads();
    // (thread -> lane as above, one s and e per wavefront and turn)
#pragma unroll
    for (int x = wave; x < NS * DT; x += C::WAVES) {
        const int s = x / DT, e = x % DT;
        const int rho = row0 + 16 * s + n16;
        float M = -INFINITY, L = 0.f, f[C::WAVES];
#pragma unroll
        for (int w = 0; w < C::WAVES; ++w) M = fmaxf(M, ml[w * C::ROWS + 16 * s + n16].x);
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < C::WAVES; ++w) {
            const float2 v = ml[w * C::ROWS + 16 * s + n16];
            f[w] = __builtin_amdgcn_exp2f(v.x - M);
            L = fmaf(f[w], v.y, L);
            o += f[w] * part[((w * NS + s) * DT + e) * 64 + lane];
        }
        if (rho > last) continue;
        const float inv = 1.0f / L;
        const size_t rid = s == 0 ? rowid[0] : rowid[1];
        *reinterpret_cast<uint2 *>(O + rid * D + 16 * e + 4 * q4) = pack_bf16(o * inv);
        if (lse != nullptr && e == 0 && q4 == 0) lse[rid] = (M + log2f(L)) * 0.69314718055994530942f;
    }
}

template <int D, bool MASKED>
static hipError_t launch_split(const Geom &g, const uint16_t *Q, const void *packed, const uint32_t *sel_mask,
                               const int *mode_flag, int my_mode, uint16_t *O, float *lse, hipStream_t st)
{
    using C = Split<D>;
    const uint16_t *Kp = reinterpret_cast<const uint16_t *>(packed);
    const size_t half_elems = (size_t)g.Hkv * g.N * g.TPC * KEY_TILE * D;
    const uint16_t *Vt = Kp + half_elems;
    const int32_t *csize = reinterpret_cast<const int32_t *>(Vt + half_elems);
    static LdsOptIn opted;  // one per kernel instantiation
    const hipError_t e = opted.ensure(reinterpret_cast<const void *>(&attn_split_kernel<D, MASKED>), C::BYTES);
    if (e != hipSuccess) return e;
    const unsigned blocks = (unsigned)((g.S * g.G - 1) / C::ROWS + 1) * (unsigned)g.Hkv;
    hipLaunchKernelGGL((attn_split_kernel<D, MASKED>), dim3(blocks), dim3(C::THREADS), C::BYTES, st, g, Q, Kp, Vt, csize,
                       sel_mask, mode_flag, my_mode, O, lse);
    return hipGetLastError();
}

hipError_t launch_attn_split(const Geom &g, const uint16_t *Q, const void *packed, const uint32_t *sel_mask,
                             const int *mode_flag, int my_mode, uint16_t *O, float *lse, hipStream_t st)
{
    if (g.D == 64)
        return sel_mask ? launch_split<64, true>(g, Q, packed, sel_mask, mode_flag, my_mode, O, lse, st)
                        : launch_split<64, false>(g, Q, packed, sel_mask, mode_flag, my_mode, O, lse, st);
    return sel_mask ? launch_split<128, true>(g, Q, packed, sel_mask, mode_flag, my_mode, O, lse, st)
                    : launch_split<128, false>(g, Q, packed, sel_mask, mode_flag, my_mode, O, lse, st);
}

}  // namespace adaspark
