// Expert FFNs: choice of kernel family per storage type.
#include "ffn_internal.h"

namespace evomoe {

size_t ffn_bwd_workspace_bytes(const evomoe_shape& s) {
    return dh_bytes(s) + colsum_scratch_bytes(s);          // [dH][bias-gradient partials]
}

hipError_t launch_expert_ffn(const Ctx& c, const evomoe_shape& s, const void* x,
                             const int32_t* pair_token, const int32_t* expert_offsets, const void* W1,
                             const float* b1, const void* W2, const float* b2, void* H, void* A, void* O) {
    if (s.dtype == EVOMOE_BF16)
        return mfma_ffn_fwd(c, s, x, pair_token, expert_offsets, W1, b1, W2, b2, H, A, O);
    return f32_ffn_fwd(c, s, x, pair_token, expert_offsets, W1, b1, W2, b2, H, A, O);
}

hipError_t launch_expert_ffn_bwd(const Ctx& c, const evomoe_shape& s, const void* dO, const void* H,
                                 const void* A, const void* x, const int32_t* pair_token,
                                 const int32_t* expert_offsets, const void* W1, const void* W2,
                                 const void* dy, const float* pair_gate,
                                 void* dW1, float* db1, void* dW2, float* db2, void* dXp,
                                 int accumulate, void* workspace) {
    if (s.dtype == EVOMOE_BF16)
        return mfma_ffn_bwd(c, s, dO, H, A, x, pair_token, expert_offsets, W1, W2, dy, pair_gate, dW1, db1,
                            dW2, db2, dXp, accumulate, workspace);
    return f32_ffn_bwd(c, s, dO, H, A, x, pair_token, expert_offsets, W1, W2, dW1, db1, dW2,
                                 db2, dXp, accumulate, workspace);
}

// Recompute variant: workspace = [H : P_cap x F][A : P_cap x F][the plain backward's workspace].
static size_t act_bytes(const evomoe_shape& s) { return dh_bytes(s); }
size_t ffn_bwd_recompute_workspace_bytes(const evomoe_shape& s) {
    return 2 * act_bytes(s) + ffn_bwd_workspace_bytes(s);
}
hipError_t launch_expert_ffn_bwd_recompute(const Ctx& c, const evomoe_shape& s, const void* dO, const void* x,
                                           const int32_t* pair_token, const int32_t* expert_offsets,
                                           const void* W1, const float* b1, const void* W2, const void* dy,
                                           const float* pair_gate, void* dW1,
                                           float* db1, void* dW2, float* db2, void* dXp, int accumulate,
                                           void* workspace) {
    char* w = static_cast<char*>(workspace);
    void* H = w;
    void* A = w + act_bytes(s);
    void* rest = w + 2 * act_bytes(s);
    hipError_t err = launch_expert_ffn(c, s, x, pair_token, expert_offsets, W1, b1, W2, nullptr, H, A, nullptr);
    if (err != hipSuccess) return err;
    return launch_expert_ffn_bwd(c, s, dO, H, A, x, pair_token, expert_offsets, W1, W2, dy, pair_gate, dW1, db1,
                                 dW2, db2, dXp, accumulate, rest);
}

}  // namespace evomoe

// Not part of the ABI: lets the tests see on the host which kernel a call reaches.  tile: rows, columns, waves.
extern "C" int evomoe_test_ffn_tile(const evomoe_shape* shape, int num_cu, int64_t announced_pairs, int kernel, int* tile) {
    evomoe::Ctx c{};
    c.num_cu = num_cu;
    c.pair_hint = announced_pairs;
    const evomoe::FfnTile t = shape->dtype == EVOMOE_BF16 ? evomoe::mfma_ffn_tile(c, *shape, kernel)
                                                          : evomoe::f32_ffn_tile(c, *shape, kernel);
    tile[0] = t.rows; tile[1] = t.cols; tile[2] = t.waves;
    return t.rows > 0;
}
