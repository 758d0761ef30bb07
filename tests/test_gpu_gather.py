"""The rows of x that dispatch gathers: fewer vectors than threads, a ragged last round, several rounds of the grid."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402


@pytest.mark.parametrize("T,d,E,dtype", [(1, 4, 1, "f32"), (33, 72, 3, "bf16"), (3001, 1032, 2, "bf16"), (9001, 1028, 2, "f32")])
def test_gathered_rows_are_the_tokens_rows(T, d, E, dtype):
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("gather", T=T, d=d, E=E, F=64, act="gelu", dtype=dtype, taus=(1.0,), threshold=0.1, seed=613,
                            bias_std=0.02)
    gl = h.GpuLayer(synth.make_layer_inputs(cfg), backward=False)
    b, B = gl.buf, h.B
    B.evomoe_dts_gate(gl.ctx, gl.shape, gl.x, gl.params.Wg, gl.params.bg, gl.noise, 1.0, 0.1, b.gprime, b.gate_w, b.mask_bits,
                      b.counts, b.k, b.block_hist)
    rows = torch.full((gl.shape.P_cap + 1, d), -7.0, dtype=gl.x.dtype, device="cuda")
    B.evomoe_dispatch(gl.ctx, gl.shape, b.mask_bits, b.gprime, b.expert_offsets, b.pair_token, b.pair_gate, b.tok_off,
                      b.tok_rows, b.num_pairs, gl.x, rows)
    P = B.evomoe_num_pairs(gl.ctx, b.num_pairs)
    assert torch.equal(rows[:P], gl.x[b.pair_token[:P].long()])
    assert (rows[P:] == -7.0).all()
