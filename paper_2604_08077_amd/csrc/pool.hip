// Cube mean keys (Eq. 1: k-bar_j = Mean(k in K_j)).
//
// A token's KV heads are contiguous in memory (Hkv*D bf16); a workgroup has one cube and
// all of a token's row, or a part of it of 128 bytes or more: thread = (token slot,
// 16-byte chunk); slots stride over the cube's tokens, the partial
// sums of the slots are combined through LDS in the slots' order.
// The order of the additions is a function of the shape alone: as many slots as fit POOL_THREADS beside the whole row (or
// POOL_THREADS chunks of it), whatever part of it a workgroup has.  A selection at the edge of its nucleus hangs on the last bits of a
// mean key: another order selects other cubes in a few rows of a million.
// HBM-bound: K is read exactly once.
#include "geom.h"

namespace adaspark {

constexpr int POOL_THREADS = 1024;  // of a whole row: 16 wavefronts
// Rows are cut while there are fewer workgroups than this, each part with its share of the threads, so that a CU holds several: cubes by
// themselves leave CUs empty, and a little above 256 of them, the second half of the time.  (Mean keys, us, parts up to 256 workgroups and up to
// this many: 16,384 tokens of 4 KV heads of 128 in cubes of 256 6.2, 6.4; 65,536 15.9, 12.9; 262,144 47.5, 41.5; 30,000 of 8, 14.9, 13.0;
// 69,630 of 2 in 318 cubes 11.0, 7.5; uncut rows took 11.1, 16.5, 47.2, 19.3 and 11.9.)
constexpr int POOL_WORKGROUPS = 2048;
// Places of a cube's tokens that a workgroup works out at a time, each once.  A row of many heads leaves few slots, and their chains are then the
// time: 8,192 tokens of 32 heads of 128 20.7 us, one cube of 64 heads 31.5, and 31.4 and 56.5 with every thread working out its own; 16,384 of 4
// heads 5.3, 6.4.
constexpr int POOL_TOKENS = 2048;

__global__ __launch_bounds__(POOL_THREADS) void cube_pool_kernel(Geom g, const uint16_t *__restrict__ K,
                                                                 float *__restrict__ kbar)
{
    extern __shared__ float part[];  // [slot][chunk][8]: as many as threads
    __shared__ int token[POOL_TOKENS];
    const int c = blockIdx.x;
    const CubeBox box = cube_box(g, c);
    const int size = box.size();
    const int row_elems = g.Hkv * g.D;  // elements per token row
    const int chunks = row_elems / 8;   // 16-byte chunks per row
    const int begin = chunks / gridDim.y * blockIdx.y, end = begin + chunks / gridDim.y;  // this workgroup's

    for (int sweep = begin / POOL_THREADS * POOL_THREADS; sweep < end; sweep += POOL_THREADS) {  // of as many chunks as threads
        const int chunk0 = max(sweep, begin), lanes = min(end, sweep + POOL_THREADS) - chunk0;  // handled here
        const int slots = POOL_THREADS / min(chunks - sweep, POOL_THREADS);                     // token slots working in parallel
        const int slot = threadIdx.x / lanes, col = threadIdx.x % lanes;
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        const int span = POOL_TOKENS / slots * slots;
        for (int base = 0; base < size; base += span) {
            const int n = min(span, size - base);
            __syncthreads();  // (the tokens before are done with)
            for (int r = threadIdx.x; r < n; r += blockDim.x) token[r] = token_in_cube(g, box, base + r);
            __syncthreads();
            if (slot >= slots) continue;
            // eight independent 16-byte loads in flight per thread: a cube is read by few workgroups, so the
            // memory-level parallelism has to come from inside them
            constexpr int UNROLL = 8;
            for (int r0 = slot; r0 < n; r0 += slots * UNROLL) {
                uint4 v[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    const int r = r0 + u * slots;
                    v[u] = make_uint4(0, 0, 0, 0);
                    if (r < n)
                        v[u] = *reinterpret_cast<const uint4 *>(K + (size_t)token[r] * row_elems + (size_t)(chunk0 + col) * 8);
                }
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        acc[2 * e] += __uint_as_float(w[e] << 16);
                        acc[2 * e + 1] += __uint_as_float(w[e] & 0xffff0000u);
                    }
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) part[threadIdx.x * 8 + e] = acc[e];
        __syncthreads();
        for (int x = threadIdx.x; x < lanes * 8; x += blockDim.x) {
            float sum = 0.f;
#pragma unroll 8
            for (int s2 = 0; s2 < slots; ++s2) sum += part[s2 * (lanes * 8) + x];
            kbar[(size_t)c * row_elems + (size_t)chunk0 * 8 + x] = sum / (float)size;
        }
        __syncthreads();
    }
}

hipError_t launch_cube_pool(const Geom &g, const uint16_t *K, float *kbar, hipStream_t st)
{
    const int chunks = g.Hkv * g.D / 8;
    int parts = 1;
    while (g.N * parts < POOL_WORKGROUPS && chunks % (16 * parts) == 0) parts *= 2;
    const int threads = chunks <= POOL_THREADS ? max(64, POOL_THREADS / parts) : POOL_THREADS;
    hipLaunchKernelGGL(cube_pool_kernel, dim3(g.N, parts), dim3(threads), threads * 32, st, g, K, kbar);
    return hipGetLastError();
}

}  // namespace adaspark
