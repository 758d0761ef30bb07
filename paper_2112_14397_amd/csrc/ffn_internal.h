// Launchers shared between the expert-FFN translation units.  Internal to the library.
#pragma once
#include "kernels.h"

namespace evomoe {

// Which tile (rows, columns, waves) an expert-FFN launch takes on c.num_cu compute units for c.pair_hint announced pairs; the
// weight-gradient launch (EVOMOE_K_FFN_BWD_DW2) with both gradients wanted.  Host only: the launchers ask the same rule.
struct FfnTile { int rows, cols, waves; };
FfnTile mfma_ffn_tile(const Ctx& c, const evomoe_shape& s, int kernel);
FfnTile f32_ffn_tile(const Ctx& c, const evomoe_shape& s, int kernel);

// float32 matrix-core path (ffn_f32.hip)
hipError_t f32_ffn_fwd(const Ctx& c, const evomoe_shape& s, const void* x, const int32_t* pair_token,
                       const int32_t* expert_offsets, const void* W1, const float* b1, const void* W2,
                       const float* b2, void* H, void* A, void* O);
hipError_t f32_ffn_bwd(const Ctx& c, const evomoe_shape& s, const void* dO, const void* H, const void* A,
                       const void* x, const int32_t* pair_token, const int32_t* expert_offsets, const void* W1,
                       const void* W2, void* dW1, float* db1, void* dW2, float* db2, void* dXp, int accumulate,
                       void* dH);
// the float32 layer's column sums: row ranges per expert (at most)
constexpr int kF32ColsumSplit = 16;
// the bf16 layer's column sums of dO: row ranges per expert (at most), part[range][g][n], added in order
constexpr int kColsumSplit = 32;
// bf16 layer: [partial column sums of dO][column sums of dH for each 64 rows]; float32 layer: [partial column sums of dO][of
// dH]; a multiple of 256
size_t colsum_scratch_bytes(const evomoe_shape& s);
size_t dh_colpart_bytes(const evomoe_shape& s);       // the second part alone (0 for a float32 layer)
// the backward workspace is [dH : P_cap x F elements, rounded up to 256 B][bias-gradient partial sums]
inline size_t dh_bytes(const evomoe_shape& s) {
    const size_t esz = s.dtype == EVOMOE_BF16 ? 2 : 4;
    return ((size_t)s.P_cap * s.F * esz + 255) & ~(size_t)255;
}

// bf16 matrix-core path (ffn_mfma.hip)
hipError_t mfma_ffn_fwd(const Ctx& c, const evomoe_shape& s, const void* x, const int32_t* pair_token,
                        const int32_t* expert_offsets, const void* W1, const float* b1, const void* W2,
                        const float* b2, void* H, void* A, void* O);
hipError_t mfma_ffn_bwd(const Ctx& c, const evomoe_shape& s, const void* dO, const void* H, const void* A,
                        const void* x, const int32_t* pair_token, const int32_t* expert_offsets,
                        const void* W1, const void* W2, const void* dy, const float* pair_gate, void* dW1,
                        float* db1, void* dW2, float* db2, void* dXp, int accumulate, void* dH);

}  // namespace evomoe
