"""The announced pair count picks tiles and nothing else: every output of the expert FFN, forward and backward, keeps its bits
whatever was announced."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402

# T, d, E, F, P_cap, announced pair counts (0: none, the tiles are picked for P_cap).  The first case of each type reaches
# every tile of every forward launch, dH and dXp.
CASES = {
    "f32": [(1900, 508, 3, 508, 1900, (0, 1, 900)),
            (300, 68, 4, 132, 300, (0, 1))],
    "bf16": [(700, 392, 3, 392, 200000, (0, 1, 2400, 7500, 8250, 17800, 42000, 195700)),
             (700, 136, 5, 264, 50000, (0, 1, 700, 9000))],
}


@pytest.mark.parametrize("dtype,case", [(t, c) for t in CASES for c in CASES[t]])
def test_results_do_not_depend_on_the_announced_pair_count(dtype, case):
    import torch
    import gpu_harness as h
    T, d, E, F, P_cap, hints = case
    cfg = synth.LayerConfig("hint", T=T, d=d, E=E, F=F, act="gelu", dtype=dtype, taus=(1.0,), threshold=0.9, seed=419,
                            bias_std=0.02)
    gl = h.GpuLayer(synth.make_layer_inputs(cfg), P_cap=P_cap)
    first = None
    for hint in hints:
        h.B.evomoe_hint_pairs(gl.ctx, hint)
        P = gl.forward(1.0, 0.9)
        gl.backward(1.0)
        assert P == T                      # (Top-1 through c = 0.9)
        b = gl.buf
        got = {n: getattr(b, n)[:P].clone() for n in ("H", "A", "O", "dXp")}
        got.update({n: getattr(b, n).clone() for n in ("dW1", "db1", "dW2", "db2")})
        first = first or got
        for n in got:
            assert torch.equal(got[n].view(torch.uint8), first[n].view(torch.uint8)), (n, hint)
