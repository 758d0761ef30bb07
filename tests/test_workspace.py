"""CPU-only: the workspace that the FFN backward asks for.  Programs size buffers once; what was enough stays enough."""
import pytest

from paper_2112_14397_amd import binding as B

up = lambda n: (n + 255) // 256 * 256

SHAPES = [(777, 136, 7, 264, 2000), (8192, 768, 16, 3072, 58330), (8192, 512, 64, 2048, 22073), (64, 1024, 2, 1024, 128),
          (700, 264, 5, 64, 3500), (100, 64, 64, 64, 6400), (48, 768, 16, 3072, 48), (16384, 64, 1, 256, 16384)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,d,E,F,P", SHAPES)
def test_workspace_does_not_outgrow_its_stated_parts(dtype, T, d, E, F, P):
    esz = 2 if dtype == "bf16" else 4
    s = B.make_shape(T, d, E, F, dtype, "gelu", P)
    dH = up(P * F * esz)
    # bias gradients: 32 partial sums of the wider matrix for each expert, for bf16 also two rows of F for each 128 rows
    partials = up(32 * E * max(d, F) * 4)
    if dtype == "bf16":
        partials += up(2 * ((P + 127) // 128 + E) * F * 4) + P * d * 2
    # the gate backward shares the buffer: dz [T,E] and up to 256 partial tables (bf16: blocks of its own choice)
    gate = up(4 * (T * E + 256 * (d * E + E)))
    assert B.evomoe_workspace_bytes(s) <= max(up(dH + partials), gate)
    assert B.evomoe_workspace_bytes_recompute(s) <= max(up(3 * dH + partials), gate)
    if dtype == "f32":      # nothing is asked for that nothing uses: dH, and 16 partial sums of both matrices
        assert B.evomoe_workspace_bytes(s) <= max(up(dH + up(16 * E * (d + F) * 4)), gate)
