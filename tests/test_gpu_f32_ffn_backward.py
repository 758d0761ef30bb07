"""The float32 expert FFN's backward with some of its outputs left out, accumulating into the others."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402


def _layer(T, d, E, F, threshold=0.1):
    import gpu_harness as h
    cfg = synth.LayerConfig("f32-bwd", T=T, d=d, E=E, F=F, act="gelu", dtype="f32", taus=(1.0,), threshold=threshold,
                            seed=523, bias_std=0.02)
    return h, h.GpuLayer(synth.make_layer_inputs(cfg))


@pytest.mark.parametrize("keep", [("db1",), ("db2",), ("db1", "db2"), ("dW1", "db1", "db2"), ("dW2", "db1", "db2"),
                                  ("dW1", "db1", "dW2", "db2")], ids="-".join)
def test_f32_gradients_accumulate_with_others_left_out(keep):
    """g + g is exact: two accumulating calls onto zeros give twice the gradient of the full call, bit for bit."""
    import torch
    h, gl = _layer(300, 68, 3, 132)            # several experts, several tiles of every matrix
    gl.forward(1.0, 0.1)
    gl.backward(1.0)
    b, p, B = gl.buf, gl.params, h.B
    got = {n: torch.zeros_like(getattr(b, n)) for n in keep}
    for _ in range(2):
        B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, b.dO, b.H, b.A, gl.x, b.pair_token, b.expert_offsets, p.W1, p.W2, gl.dy,
                                b.pair_gate, got.get("dW1"), got.get("db1"), got.get("dW2"), got.get("db2"), b.dXp, True,
                                b.workspace)
    torch.cuda.synchronize()
    for n in keep:
        assert torch.equal(got[n], 2 * getattr(b, n)), n
