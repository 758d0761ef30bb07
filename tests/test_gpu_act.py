"""The expert FFN's activation functions, bf16 in both epilogues (256x256 tiles of eight waves, small tiles)."""
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
    """Phi is off by less than 1.2e-5, gelu by |h| times that, for small |h| by 3.6e-5 h^2 (Phi's polynomial is odd about 1/2; its first
    coefficient is off by 3.5e-5), float32 evaluation 1e-7 |h|: beside the rounding to bf16."""
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
        bound = torch.minimum(1.2e-5 * h.abs(), 3.6e-5 * h * h) + 1e-7 * h.abs()
        assert (more <= bound).all(), (row, (more / bound).max().item(), h.flatten()[(more / bound).argmax()].item())
    layer.ctx.close()


@pytest.mark.parametrize("act", ["gelu", "relu"])
@pytest.mark.parametrize("P,E,F,tile", SIZES)
def test_nan_stays_nan(P, E, F, tile, act):
    """A NaN in one bias: A has one exactly where H has; dH of gelu too (the derivative of ReLU is taken as 0 there)."""
    import torch
    b1 = torch.randn(E, F, generator=torch.Generator("cuda").manual_seed(4), device="cuda")
    b1[E - 2, 9] = float("nan")
    layer = Layer(P, E, F, tile, act, b1)
    B, nan = layer.B, torch.zeros(P, F, dtype=torch.bool, device="cuda")
    nan[int(layer.offs[E - 2]):int(layer.offs[E - 1]), 9] = True
    assert torch.equal(layer.H.isnan(), nan)
    assert torch.equal(layer.A.isnan(), nan)
    db1 = torch.empty(E, F, device="cuda")
    ws = torch.empty(B.evomoe_workspace_bytes(layer.shape), dtype=torch.uint8, device="cuda")
    B.evomoe_expert_ffn_bwd(layer.ctx, layer.shape, layer.dO, layer.H, layer.A, layer.x, None, layer.offs, layer.W1, layer.W2, None,
                            None, None, db1, None, None, layer.dXp, False, ws)
    torch.cuda.synchronize()
    if act == "gelu":
        assert torch.equal(ws[:P * F * 2].view(torch.bfloat16).view(P, F).isnan(), nan)
        assert torch.equal(db1.isnan(), b1.isnan())
    layer.ctx.close()


@pytest.mark.parametrize("act", ["gelu", "relu"])
def test_nan_stays_nan_in_float32(act):
    import torch
    import gpu_harness as h
    B, P, d, E, F = h.B, 100, 64, 2, 64
    b1 = torch.zeros(E, F, device="cuda")
    b1[1, 9] = float("nan")
    x, W1, W2 = torch.ones(P, d, device="cuda"), torch.ones(E, F, d, device="cuda"), torch.ones(E, d, F, device="cuda")
    H, A, O = torch.empty(P, F, device="cuda"), torch.empty(P, F, device="cuda"), torch.empty(P, d, device="cuda")
    ctx = B.Context()
    B.evomoe_expert_ffn(ctx, B.make_shape(P, d, E, F, "f32", act, P), x, None, torch.tensor([0, 33, P], dtype=torch.int32, device="cuda"),
                        W1, b1, W2, None, H, A, O)
    torch.cuda.synchronize()
    want = torch.zeros_like(H, dtype=torch.bool)
    want[33:, 9] = True
    assert torch.equal(H.isnan(), want) and torch.equal(A.isnan(), want)
    ctx.close()
