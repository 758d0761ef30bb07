"""The bf16 expert FFN at the edges of its tiles (64x64 to 256x256), against the oracle.  The launch
picks a tile from the sizes, so each case names those it reaches: (GEMM1, GEMM2, dH, dXp; weight gradients)."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402

# name, T, d, E, F: Top-1 through c = 0.9, so the single expert of an E = 1 layer owns exactly T rows
CASES = [
    ("64-few-rows", 9, 64, 1, 64),               # 64x64 throughout, here and below the weight gradients' too
    ("64-below", 63, 72, 1, 136),                # 64x64 throughout; one vector past a slab of 64 and past two tiles
    ("64-above", 65, 64, 1, 192),                # 64x64 throughout; one row past a tile
    ("64x128-long", 2497, 392, 1, 264),          # 64x64, 64x128, 64x64, 64x128
    ("64x128-short", 1900, 776, 16, 1544),       # 64x128, 64x64, 64x128, 64x64; 256x256
    ("128-below", 4095, 512, 4, 1032),           # 128x128 throughout, the long contractions with 64-wide slabs
    ("128x256-above", 4100, 1032, 1, 1032),      # 128x128, 128x256 with four waves, 128x128, 128x256 with eight; 128x128
    ("256-above", 16900, 1032, 1, 520),          # 256x256 with eight waves, with four, 128x256, 256x256 with four; 64x64
    # the tile is picked for the buffers' capacity where no pair count is announced: 256x256 for dH as well
    ("256-dh-one", 299, 1032, 1, 264, 200000),   # one full row tile and a ragged one
    ("256-dh-three", 700, 1032, 3, 264, 200000),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bf16_ffn_at_tile_edges(case):
    import gpu_harness as h
    name, T, d, E, F = case[:5]
    cfg = synth.LayerConfig(name, T=T, d=d, E=E, F=F, act="gelu", dtype="bf16", taus=(1.0,), threshold=0.9, seed=311,
                            bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    # the pair buffers hold a row for each token (Top-1): the launch picks its tiles for that many pairs
    gl = h.GpuLayer(inp, P_cap=case[5] if len(case) > 5 else T)
    fwd, P, _, _ = h.compare_forward(gl, inp, 1.0, 0.9)
    gl.backward(1.0)
    # the FFN's own gradients (the gate's are sums over tokens of terms of either sign: a small one carries the rounding
    # of the large terms that cancelled in it, whatever the tile)
    ref = h.orc.moe_layer_backward(fwd, inp.dy, inp.x, inp.Wg, 1.0, inp.W1, inp.W2, cfg.act).ffn
    b = gl.buf
    for what, got, want in (("dXp", h.np_of(b.dXp)[:P], ref.dXp), ("dW1", h.np_of(b.dW1), ref.dW1),
                            ("db1", h.np_of(b.db1), ref.db1), ("dW2", h.np_of(b.dW2), ref.dW2),
                            ("db2", h.np_of(b.db2), ref.db2)):
        worst, above = h.tol_stats(got, want, h.RTOL["bf16"])
        assert above == 0, f"{what}: worst err/bound {worst:.3g}, {above} elements above it"


@pytest.mark.parametrize("which", ["dW1", "dW2"])
def test_one_weight_gradient_alone_accumulates_once(which):
    """With the other weight gradient left out, accumulation adds the micro-batch's gradient once."""
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("alone", T=300, d=72, E=3, F=136, act="gelu", dtype="bf16", taus=(1.0,), threshold=0.1, seed=5,
                            bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    gl = h.GpuLayer(inp)
    gl.forward(1.0, 0.1)
    gl.backward(1.0)
    b, p, s, B = gl.buf, gl.params, gl.shape, h.B
    want, got = getattr(b, which).float(), torch.zeros_like(getattr(b, which))
    for _ in range(2):
        B.evomoe_expert_ffn_bwd(gl.ctx, s, b.dO, b.H, b.A, gl.x, b.pair_token, b.expert_offsets, p.W1, p.W2, gl.dy,
                                b.pair_gate, got if which == "dW1" else None, None, got if which == "dW2" else None, None,
                                b.dXp, True, b.workspace)
    torch.cuda.synchronize()
    assert torch.equal(got.float(), 2 * want)         # g + g is exact
