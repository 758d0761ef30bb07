"""CPU-only: the sizes at which the GPU tests compare the expert FFN with the oracle reach the kernels they are there for."""
import pytest

from helpers import ffn_tiles
from paper_2112_14397_amd import binding as B
import test_gpu_bf16_tiles as bf16
import test_gpu_f32_tiles as f32
import test_gpu_ffn_pair_hint as hint

# every tile each launch can take: GEMM1, GEMM2, dH, dXp, weight gradients
BF16 = [{"256x256/8", "128x256/4", "128x128/4", "64x128/4", "64x64/4"}, {"256x256/4", "128x256/4", "128x128/4", "64x128/4", "64x64/4"},
        {"256x256/8", "128x256/4", "128x128/4", "64x128/4", "64x64/4"}, {"256x256/4", "128x256/8", "128x128/4", "64x128/4", "64x64/4"},
        {"256x256/8", "128x128/4", "64x64/4"}]
F32 = [{"64x64/4", "32x32/4"}] * 5


def test_bf16_cases_reach_the_tiles_they_name_and_all_there_are():
    seen = [set() for _ in BF16]
    for name, T, d, E, F, rows, tiles in bf16.CASES:
        assert ffn_tiles(B.make_shape(T, d, E, F, "bf16", "gelu", rows)) == tiles, name
        for s, t in zip(seen, tiles):
            s.add(t)
    assert seen == BF16


def test_f32_cases_reach_the_tiles_they_name_and_all_there_are():
    seen = [set() for _ in F32]
    for name, T, d, E, F, sizes in f32.CASES:
        tiles = ffn_tiles(B.make_shape(T, d, E, F, "f32", "gelu", T * E))
        assert tiles == tuple(f"{n}x{n}/4" for n in sizes), name
        for s, t in zip(seen, tiles):
            s.add(t)
    assert seen == F32


@pytest.mark.parametrize("dtype,every", [("f32", F32), ("bf16", BF16)])
def test_announced_pair_counts_reach_every_tile(dtype, every):
    T, d, E, F, P_cap, hints = hint.CASES[dtype][0]
    shape = B.make_shape(T, d, E, F, dtype, "gelu", P_cap)
    seen = [set(t) for t in zip(*(ffn_tiles(shape, h) for h in hints))]
    # (weight-gradient tiles follow the matrices, not the pairs: they add an expert's rows in one order)
    assert seen[:4] == every[:4]
