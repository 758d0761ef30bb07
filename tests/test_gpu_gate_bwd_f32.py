"""The float32 gate backward at each number of columns a thread owns (it follows d and E), against the oracle."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402

# T, d, E: 1, 2 and 4 columns for up to 16 experts, 1 and 2 for up to 32, with a last block that is not full
CASES = [(70, 64, 4), (33, 508, 16), (70, 512, 5), (70, 1020, 16), (70, 1024, 16), (70, 508, 24), (70, 516, 32)]


@pytest.mark.parametrize("T,d,E", CASES)
def test_gate_backward_columns(T, d, E):
    import gpu_harness as h
    cfg = synth.LayerConfig("gate-bwd", T=T, d=d, E=E, F=64, act="gelu", dtype="f32", taus=(1.0,), threshold=0.05, seed=41,
                            bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    gl = h.GpuLayer(inp)
    fwd, P, _, _ = h.compare_forward(gl, inp, 1.0, 0.05)
    gl.backward(1.0)
    # The gate's own share: dx starts from zero, and the oracle takes the dG and g' that the layer computed (dz is a small
    # difference of them where one expert has nearly all the weight, which magnifies their own errors).  What is left is
    # rounding: 4 * 2^-24 / (1 - g') for dz, 2.4e-6 at g' = 0.9, and E 2^-24, 1.9e-6, for a sum over 32 experts.
    b, B, dp = gl.buf, h.B, fwd.disp
    b.dx.zero_()
    B.evomoe_dts_gate_bwd(gl.ctx, gl.shape, b.dG_pairs, b.tok_off, b.tok_rows, b.gprime, b.mask_bits, 1.0, gl.x,
                          gl.params.Wg, b.dWg, b.dbg, b.dx, b.workspace)
    _, dWg, dbg, dx = h.orc.dts_gate_bwd(h.np_of(b.dG_pairs)[:P], dp.pair_token, dp.pair_expert,
                                         h.np_of(b.gprime), 1.0, inp.x, inp.Wg)
    for what, got, want in (("dWg", b.dWg, dWg), ("dbg", b.dbg, dbg), ("dx", b.dx, dx)):
        worst, above = h.tol_stats(h.np_of(got), want, h.RTOL["f32"])
        assert above == 0, f"{what}: worst err/bound {worst:.3g}, {above} elements above it"
