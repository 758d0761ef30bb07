"""The bf16 expert FFN at the edges of its tiles (64x64 to 256x256), against the oracle.  The launch picks a tile from the
sizes; each case names those it reaches, and the test asks the library whether it does."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402
from helpers import ffn_tiles  # noqa: E402

TINY = ("64x64/4",) * 5
# name, T, d, E, F, rows of the pair buffers, tiles of GEMM1, GEMM2, dH, dXp and the weight gradients.
# Top-1 through c = 0.9, so the single expert of an E = 1 layer owns exactly T rows.  Where no pair count is announced the
# tiles are picked for the buffers' rows.
CASES = [
    ("64-few-rows", 9, 64, 1, 64, 9, TINY),
    ("64-below", 63, 72, 1, 136, 63, TINY),      # one vector past a slab of 64 and past two tiles
    ("64-above", 65, 64, 1, 192, 65, TINY),      # one row past a tile
    ("64x128-long", 2497, 392, 1, 264, 2497, ("64x64/4", "64x128/4", "64x64/4", "64x128/4", "64x64/4")),
    ("64x128-short", 1900, 776, 16, 1544, 1900, ("64x128/4", "64x64/4", "64x128/4", "64x64/4", "256x256/8")),
    ("128-below", 4095, 512, 4, 1032, 4095, ("128x128/4",) * 5),
    ("128x256-above", 4100, 1032, 1, 1032, 4100, ("128x128/4", "128x256/4", "128x128/4", "128x256/8", "128x128/4")),
    ("256-above", 16900, 1032, 1, 520, 16900, ("256x256/8", "256x256/4", "128x256/4", "256x256/4", "64x64/4")),
    ("128x256-gemm1", 300, 72, 1, 504, 40000, ("128x256/4", "256x256/4", "128x256/4", "256x256/4", "64x64/4")),
    # one full row tile and a ragged one, one expert and three
    ("256-dh-one", 299, 1032, 1, 504, 200000, ("256x256/8", "256x256/4", "256x256/8", "256x256/4", "64x64/4")),
    ("256-dh-three", 700, 1032, 3, 504, 200000, ("256x256/8", "256x256/4", "256x256/8", "256x256/4", "128x128/4")),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_bf16_ffn_at_tile_edges(case):
    import gpu_harness as h
    name, T, d, E, F, rows, tiles = case
    cfg = synth.LayerConfig(name, T=T, d=d, E=E, F=F, act="gelu", dtype="bf16", taus=(1.0,), threshold=0.9, seed=311,
                            bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    gl = h.GpuLayer(inp, P_cap=rows)
    assert ffn_tiles(gl.shape, num_cu=h.torch.cuda.get_device_properties(0).multi_processor_count) == tiles
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


@pytest.mark.parametrize("T,d,E,F,rows", [(45, 96, 1, 160, 45), (45, 72, 1, 264, 45), (45, 96, 1, 160, 100000), (300, 1056, 3, 544, 100000)])
def test_infinite_operands_stay_infinite_in_partial_slabs(T, d, E, F, rows):
    """No contraction length is a multiple of a slab of 64 here, some are of 32.  An infinity in the last element of a
    contraction must reach the result as in plain arithmetic: a slab's padding must not turn it into 0 * Inf."""
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("inf", T=T, d=d, E=E, F=F, act="gelu", dtype="bf16", taus=(1.0,), threshold=0.9, seed=523,
                            bias_std=0.02)
    gl = h.GpuLayer(synth.make_layer_inputs(cfg), P_cap=rows)
    P = gl.forward(1.0, 0.9)
    assert P == T
    b, p, B, inf = gl.buf, gl.params, h.B, float("inf")
    n = int(b.expert_offsets[1])                   # rows of expert 0
    assert n % 64
    f64 = lambda t: t.double().cpu()

    def same(got, want, what):
        got, want = f64(got), want.cpu()
        assert not torch.isnan(want).any() and torch.isinf(want).any(), what
        assert torch.equal(torch.isinf(got), torch.isinf(want)) and not torch.isnan(got).any(), what
        assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), what

    tok = b.pair_token[:n].long()
    A = b.A.clone()
    A[A == 0] = 1.0
    W1, W2 = p.W1.clone(), p.W2.clone()
    W1[0, 7, d - 1] = inf
    W2[0, 9, F - 1] = inf
    H, A2, O = torch.zeros_like(b.H), torch.zeros_like(b.A), torch.zeros_like(b.O)
    B.evomoe_expert_ffn(gl.ctx, gl.shape, gl.x, b.pair_token, b.expert_offsets, W1, p.b1, p.W2, p.b2, H, A2, O)
    same(H[:n], f64(gl.x[tok]) @ f64(W1[0]).T, "H")
    B.evomoe_expert_ffn(gl.ctx, gl.shape, gl.x, b.pair_token, b.expert_offsets, p.W1, p.b1, W2, p.b2, H, A2, O)
    same(O[:n], f64(A2[:n]) @ f64(W2[0]).T, "O")

    dO = torch.randn(gl.shape.P_cap, d, generator=torch.Generator("cuda").manual_seed(6), device="cuda").bfloat16()
    dW1, dW2, H0 = torch.zeros_like(p.W1), torch.zeros_like(p.W2), torch.zeros_like(b.H)

    def backward(A=A, x=gl.x, W1=p.W1, W2=p.W2):
        B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, dO, H0, A, x, b.pair_token, b.expert_offsets, W1, W2, None, None, dW1, None,
                                dW2, None, b.dXp, False, b.workspace)
        torch.cuda.synchronize()

    W2 = p.W2.clone()
    W2[0, d - 1, 5] = inf                          # dH = (dO W2) * act'(0), act'(0) = 1/2
    backward(W2=W2)
    dH = b.workspace[:n * F * 2].view(torch.bfloat16).view(n, F)         # the workspace begins with dH
    same(dH, f64(dO[:n]) @ f64(W2[0]) * 0.5, "dH")
    W1 = p.W1.clone()
    W1[0, F - 1, 5] = inf
    backward(W1=W1)
    same(b.dXp[:n], f64(dH) @ f64(W1[0]), "dXp")
    Ai, x = A.clone(), gl.x.clone()
    Ai[n - 1, 3] = inf
    x[tok[n - 1], 4] = inf
    backward(A=Ai, x=x)
    same(dW2[0], f64(dO[:n]).T @ f64(Ai[:n]), "dW2")
    same(dW1[0], f64(dH).T @ f64(x[tok]), "dW1")


# rows of the first expert (the others have none), d, E, F, capacity, tile of dH: a tile's last rows repeat the last one there is
@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("P,d,E,F,rows,tile", [(45, 96, 1, 160, 45, "64x64/4"), (1900, 776, 16, 1544, 1900, "64x128/4"),
                                               (4095, 512, 1, 4104, 4095, "128x128/4"), (300, 72, 1, 504, 40000, "128x256/4"),
                                               (45, 96, 1, 160, 100000, "256x256/8")])
def test_infinite_last_row_does_not_become_nan_in_the_bias_gradient(P, d, E, F, rows, tile, scaled):
    import torch
    import gpu_harness as h
    B, inf = h.B, float("inf")
    shape = B.make_shape(rows, d, E, F, "bf16", "gelu", rows)
    assert ffn_tiles(shape, num_cu=torch.cuda.get_device_properties(0).multi_processor_count)[2] == tile
    g = torch.Generator("cuda").manual_seed(P)
    rnd = lambda *s: torch.rand(*s, generator=g, device="cuda").bfloat16() + 0.5
    offs = torch.tensor([0] + [P] * E, dtype=torch.int32, device="cuda")
    dO, x, W1, W2 = rnd(rows, d), rnd(rows, d), rnd(E, F, d), rnd(E, d, F)
    H = torch.zeros(rows, F, dtype=torch.bfloat16, device="cuda")          # act'(0) = 1/2
    tok = torch.arange(rows, dtype=torch.int32, device="cuda")
    gate = torch.full((rows,), 0.25, device="cuda")
    dO[P - 1, 3] = inf
    db1 = torch.empty(E, F, device="cuda")
    dXp = torch.empty(rows, d, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(B.evomoe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ctx = B.Context()
    B.evomoe_expert_ffn_bwd(ctx, shape, dO, H, H, x, tok, offs, W1, W2, dO if scaled else None, gate if scaled else None, None, db1,
                            None, None, dXp, False, ws)
    torch.cuda.synchronize()
    assert torch.equal(db1[0], torch.full_like(db1[0], inf)) and not db1[1:].any()
    ctx.close()
