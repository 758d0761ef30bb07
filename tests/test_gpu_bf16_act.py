"""The bf16 expert FFN's activation functions in both epilogues (256x256 tiles of eight waves, small tiles)."""
import pytest

pytestmark = pytest.mark.gpu

from helpers import ffn_tiles  # noqa: E402

# pairs, experts, F, tile of GEMM1 and dH
SIZES = [(192, 64, 4096, "64x128/4"), (60000, 5, 1032, "256x256/8")]


class Layer:
    """Every row has the pre-activations b1 of its expert: W1 is zero."""
    def __init__(self, P, E, F, tile, act, b1):
        import torch
        import gpu_harness as h
        self.B, d = h.B, 64
        self.shape = self.B.make_shape(P, d, E, F, "bf16", act, P)
        tiles = ffn_tiles(self.shape, num_cu=torch.cuda.get_device_properties(0).multi_processor_count)
        assert tiles[0] == tiles[2] == tile
        g = torch.Generator("cuda").manual_seed(E)
        rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
        self.offs = torch.tensor([P * e // E for e in range(E + 1)], dtype=torch.int32, device="cuda")
        self.x, self.dO, self.W1, self.W2 = rnd(P, d), rnd(P, d), rnd(E, F, d) * 0, rnd(E, d, F)
        self.H, self.A = (torch.empty(P, F, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        self.O, self.dXp = (torch.empty(P, d, dtype=torch.bfloat16, device="cuda") for _ in range(2))
        self.ctx = self.B.Context()
        self.B.evomoe_expert_ffn(self.ctx, self.shape, self.x, None, self.offs, self.W1, b1, self.W2, None, self.H, self.A, self.O)
        torch.cuda.synchronize()


@pytest.mark.parametrize("P,E,F,tile", SIZES)
def test_gelu_is_off_by_no_more_than_its_polynomial(P, E, F, tile):
    """|2^p(z) - Q(z)| z is below 9.6e-7 for every z = |h|, float32 evaluation included, and the sum of that and the positive part
    is rounded once to float32 (2.4e-7 below 8): 1.2e-6 beside the rounding to bf16."""
    import torch
    g = torch.Generator("cuda").manual_seed(3)
    h = torch.rand(E, F, generator=g, device="cuda") * 16 - 8
    h[:, ::3] = torch.exp(h[:, ::3]) * torch.sign(torch.rand(E, F, generator=g, device="cuda") - 0.5)[:, ::3]     # 3e-4 .. 3e3
    h.clamp_(-8, 8)
    layer = Layer(P, E, F, tile, "gelu", h)
    want = h.double() * torch.special.ndtr(h.double())
    half = torch.exp2(torch.floor(torch.log2(want.abs())) - 8)          # half a unit of bf16's last place
    for row in (0, -1):
        at = layer.offs[:-1].long() if row == 0 else layer.offs[1:].long() - 1
        more = (layer.A[at].double() - want).abs() - half
        assert (more <= 1.2e-6).all(), (row, more.max().item(), h.flatten()[more.argmax()].item())
    layer.ctx.close()
