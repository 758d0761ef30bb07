"""The float32 expert FFN at the edges of its tiles (64x64, and 32x32 with the contraction split over four waves), against
the oracle.  `few` tiles leave the chip mostly idle (32x32), `many` fill it (64x64); each case names the tiles it reaches, and
the test asks the library whether it does."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402
from helpers import ffn_tiles  # noqa: E402

# name, T, d, E, F, tile sizes of GEMM1, GEMM2, dH, dXp and the weight gradients: Top-1 through c = 0.9, so the single
# expert of an E = 1 layer owns exactly T rows
CASES = [
    ("few-one-row", 1, 4, 1, 4, (32, 32, 32, 32, 32)),
    ("few-below", 31, 60, 1, 124, (32, 32, 32, 32, 32)),           # one short of a tile in every dimension
    ("few-exact", 32, 64, 1, 128, (32, 32, 32, 32, 32)),
    ("few-above", 33, 68, 1, 132, (32, 32, 32, 32, 32)),           # one vector past a tile and past a slab
    # (two experts would make a row of dWg two opposite numbers: nothing bounds its relative error when they cancel)
    ("many-below", 2047, 188, 4, 1020, (64, 64, 64, 64, 32)),
    ("many-above", 2049, 196, 4, 1028, (64, 32, 64, 32, 32)),
    ("many-dw-below", 1500, 252, 8, 1020, (64, 64, 64, 64, 64)),
    ("many-dw-above", 1500, 316, 8, 1028, (64, 64, 64, 64, 64)),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_f32_ffn_at_tile_edges(case):
    import gpu_harness as h
    name, T, d, E, F, sizes = case
    cfg = synth.LayerConfig(name, T=T, d=d, E=E, F=F, act="gelu", dtype="f32", taus=(1.0,), threshold=0.9, seed=301,
                            bias_std=0.02)
    inp = synth.make_layer_inputs(cfg)
    gl = h.GpuLayer(inp)
    assert ffn_tiles(gl.shape, num_cu=h.torch.cuda.get_device_properties(0).multi_processor_count) == \
        tuple(f"{n}x{n}/4" for n in sizes)
    fwd, P, _, _ = h.compare_forward(gl, inp, 1.0, 0.9)
    h.compare_backward(gl, inp, fwd, 1.0)
