// Cube mean keys (Eq. 1: k-bar_j = Mean(k in K_j)).
//
// A token's KV heads are contiguous in memory (Hkv*D bf16); a workgroup has one cube and
// all of a token's row, or, with fewer cubes than CUs, a part of it of 128 bytes or more: thread = (token slot,
// 16-byte chunk); slots stride over the cube's tokens, the partial
// sums of the slots are combined through LDS in a fixed order (the result does
// not depend on scheduling).  HBM-bound: K is read exactly once.
#include "geom.h"

namespace adaspark {

constexpr int POOL_THREADS = 1024;  // 16 wavefronts: one workgroup (one cube) per CU has to keep that CU's share of HBM busy

__global__ __launch_bounds__(POOL_THREADS) void cube_pool_kernel(Geom g, const uint16_t *__restrict__ K,
                                                                 float *__restrict__ kbar)
{
    __shared__ float part[POOL_THREADS * 8];
    const int c = blockIdx.x;
    const CubeBox box = cube_box(g, c);
    const int size = box.size();
    const int row_elems = g.Hkv * g.D;  // elements per token row
    const int chunks = row_elems / 8 / gridDim.y;  // 16-byte chunks of a row that are this workgroup's
    const int begin = chunks * blockIdx.y, end = begin + chunks;

    for (int chunk0 = begin; chunk0 < end; chunk0 += POOL_THREADS) {
        const int lanes = min(end - chunk0, POOL_THREADS);  // chunks handled in this sweep
        const int slots = POOL_THREADS / lanes;                // token slots working in parallel
        const int slot = threadIdx.x / lanes, col = threadIdx.x % lanes;
        float acc[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
        if (slot < slots) {
            // eight independent 16-byte loads in flight per thread: a cube is read by one workgroup, so the
            // memory-level parallelism has to come from inside it
            constexpr int UNROLL = 8;
            for (int r0 = slot; r0 < size; r0 += slots * UNROLL) {
                uint4 v[UNROLL];
#pragma unroll
                for (int u = 0; u < UNROLL; ++u) {
                    const int r = r0 + u * slots;
                    v[u] = make_uint4(0, 0, 0, 0);
                    if (r < size) {
                        const int n = token_in_cube(g, box, r);
                        v[u] = *reinterpret_cast<const uint4 *>(K + (size_t)n * row_elems + (size_t)(chunk0 + col) * 8);
                    }
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
        // the slots' sums: `groups` threads an element, each over every groups-th slot, then these
        const int elems = lanes * 8, groups = max(1, POOL_THREADS / elems);
        const int x = threadIdx.x % elems, group = threadIdx.x / elems;
        float sum = 0.f;
        if (groups > 1) {
            if (group < groups)
                for (int s2 = group; s2 < slots; s2 += groups) sum += part[s2 * elems + x];
            __syncthreads();
            if (group < groups) part[threadIdx.x] = sum;
            __syncthreads();
        }
        const int left = groups > 1 ? groups : slots;
        for (int y = threadIdx.x; y < elems; y += POOL_THREADS) {
            float total = 0.f;
            for (int s2 = 0; s2 < left; ++s2) total += part[s2 * elems + y];
            kbar[(size_t)c * row_elems + (size_t)chunk0 * 8 + y] = total / (float)size;
        }
        __syncthreads();
    }
}

hipError_t launch_cube_pool(const Geom &g, const uint16_t *K, float *kbar, hipStream_t st)
{
    // Parts of a row while the workgroups do not fill the CUs.
    const int chunks = g.Hkv * g.D / 8;
    int parts = 1;
    while (g.N * parts < 256 && chunks % (16 * parts) == 0) parts *= 2;
    hipLaunchKernelGGL(cube_pool_kernel, dim3(g.N, parts), dim3(POOL_THREADS), 0, st, g, K, kbar);
    return hipGetLastError();
}

}  // namespace adaspark
