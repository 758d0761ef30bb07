// Column sums of the bf16 layer's dO over every expert's rows, split into kColsumSplit row ranges per expert (the first pass of
// db2; f32 partial sums, added over the row lanes in LDS, no atomics: reproducible bit for bit).
#include "ffn_internal.h"

namespace evomoe {

// A block streams whole row segments: CL column lanes x 16 bytes are contiguous in a row (up to 4 KB), RL = 256/CL
// row lanes take alternate rows, four rows of loads in flight per thread.
// Blocks: column block fastest, then expert, then row range.
__global__ __launch_bounds__(256) void colsum_kernel(
    const bf16_t* __restrict__ Mx, int N, int E, const int32_t* __restrict__ expert_offsets, int64_t P_cap,
    int CL, int gx, float* __restrict__ part)
{
    constexpr int KV = Elem<bf16_t>::kVec;           // elements per 16-byte load
    extern __shared__ float red[];               // [RL][CL*KV]
    const int RL = 256 / CL;
    const int g = (blockIdx.x / gx) % E, split = blockIdx.x / (gx * E);
    const int cl = threadIdx.x % CL, rl = threadIdx.x / CL;
    const int n = (blockIdx.x % gx * CL + cl) * KV;
    const int r0 = clamp_pairs(expert_offsets[g], P_cap), r1 = clamp_pairs(expert_offsets[g + 1], P_cap);
    const int per = (r1 - r0 + kColsumSplit - 1) / kColsumSplit;
    const int rb = r0 + split * per, re = min(r1, rb + per);
    float acc[KV];
#pragma unroll
    for (int q = 0; q < KV; ++q) acc[q] = 0.f;
    if (n < N && rl < RL) {
        int r = rb + rl;
        for (; r + 3 * RL < re; r += 4 * RL) {
            float v[4][KV];
#pragma unroll
            for (int u = 0; u < 4; ++u) Elem<bf16_t>::load_vec(Mx + (size_t)(r + u * RL) * N + n, v[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int q = 0; q < KV; ++q) acc[q] += v[u][q];
        }
        for (; r < re; r += RL) {
            float v[KV];
            Elem<bf16_t>::load_vec(Mx + (size_t)r * N + n, v);
#pragma unroll
            for (int q = 0; q < KV; ++q) acc[q] += v[q];
        }
    }
    if (rl < RL) {
#pragma unroll
        for (int q = 0; q < KV; ++q) red[(size_t)rl * CL * KV + cl * KV + q] = acc[q];
    }
    __syncthreads();
    // row lanes added in order by the threads of lane 0
    if (rl == 0 && n < N) {
#pragma unroll
        for (int q = 0; q < KV; ++q) {
            float sum = 0.f;
            for (int l = 0; l < RL; ++l) sum += red[(size_t)l * CL * KV + cl * KV + q];
            part[((size_t)split * E + g) * N + n + q] = sum;
        }
    }
}

size_t colsum_scratch_bytes(const evomoe_shape& s) {
    if (s.dtype != EVOMOE_BF16) return ((size_t)kF32ColsumSplit * s.E * (s.d + s.F) * sizeof(float) + 255) & ~(size_t)255;
    return (((size_t)kColsumSplit * s.E * s.d * sizeof(float) + 255) & ~(size_t)255) + dh_colpart_bytes(s);
}

hipError_t launch_colsum(const Ctx& c, const evomoe_shape& s, const void* Mx, int N, const int32_t* expert_offsets,
                         float* scratch) {
    constexpr int KV = Elem<bf16_t>::kVec;
    const int vecs = (N + KV - 1) / KV;                       // 16-byte vectors per row
    int CL = vecs >= 256 ? 256 : vecs;                        // column lanes (contiguous in a row)
    if (CL > 128) CL = 256;                                   // 129..255 vectors: two column blocks of 256 lanes
    const int RL = 256 / CL, gx = (vecs + CL - 1) / CL;
    hipLaunchKernelGGL(colsum_kernel, dim3(gx * s.E * kColsumSplit), dim3(256), (size_t)RL * CL * KV * sizeof(float),
                       c.stream, (const bf16_t*)Mx, N, s.E, expert_offsets, s.P_cap, CL, gx, scratch);
    return hipGetLastError();
}

}  // namespace evomoe
