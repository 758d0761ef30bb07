"""The gate of the smallest calls runs in one block that writes the counts outright; the next size takes one block for
every 16 tokens, counts cleared and added to by atomics.  Both sides of the line between them, against the oracle."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402

# T, d, E, dtype; the one block holds T <= 256 tokens, E <= 16 experts and d <= 256, at 16, 32 or 64 tokens per wave group, in
# float32 with T (d + 4 E) <= 39 * 1024
CASES = [
    (1, 64, 1, "bf16"), (15, 72, 16, "bf16"), (64, 256, 16, "bf16"), (65, 200, 7, "bf16"), (128, 256, 15, "bf16"),
    (129, 136, 4, "bf16"), (256, 256, 16, "bf16"),
    (48, 256, 17, "bf16"), (86, 264, 16, "bf16"), (257, 64, 4, "bf16"),
    (17, 64, 16, "f32"), (100, 68, 5, "f32"), (146, 256, 4, "f32"), (156, 192, 16, "f32"), (256, 64, 16, "f32"),
    (147, 256, 4, "f32"), (157, 192, 16, "f32"), (256, 256, 4, "f32"), (256, 260, 4, "f32"), (257, 64, 4, "f32"),
]


@pytest.mark.parametrize("T,d,E,dtype", CASES)
def test_gate_counts_and_histogram(T, d, E, dtype):
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("one-block", T=T, d=d, E=E, F=64, act="gelu", dtype=dtype, taus=(1.0,), threshold=0.1,
                            seed=977, bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    gl = h.GpuLayer(inp)
    gl.buf.counts.fill_(-7)              # whatever an earlier call left there
    gl.buf.block_hist.fill_(-7)
    fwd, P, _, _ = h.compare_forward(gl, inp, 1.0, 0.1)
    b = gl.buf
    bits = h.np_of(b.mask_bits).astype("uint64")
    sel = (bits[:, None] >> torch.arange(E).numpy().astype("uint64")) & 1
    assert (h.np_of(b.counts) == sel.sum(0)).all()
    hist = h.np_of(b.block_hist)
    for r in range(hist.shape[0]):
        assert (hist[r] == sel[256 * r:256 * (r + 1)].sum(0)).all(), r
