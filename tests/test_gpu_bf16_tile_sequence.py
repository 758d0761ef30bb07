"""The 256x256 tiles of GEMM1 and dH when a block works through several of them: the next tile's first slab is fetched under a
tile's epilogue, into the stage that the parity of the slab count leaves free.  Against float32 products on the GPU."""
import pytest

pytestmark = pytest.mark.gpu

from helpers import ffn_tiles  # noqa: E402


# rows, d (slabs of GEMM1 and dH: 1, 2 with a tail, 3 with a tail, 4 with a tail), act
@pytest.mark.parametrize("P,d,act", [(60000, 64, "gelu"), (33000, 72, "relu"), (120000, 136, "gelu"), (120000, 248, "relu")])
def test_blocks_with_several_256_row_tiles(P, d, act):
    import torch
    import gpu_harness as h
    B = h.B
    T, E, F = 5000, 5, 1032                                  # 1032: the last column tile has eight columns
    offs = torch.tensor([0, P // 2 + 3, P // 2 + 3, P // 2 + 4, P - 300, P], dtype=torch.int32, device="cuda")   # an empty expert, one row
    shape = B.make_shape(T, d, E, F, "bf16", act, P)
    tiles = ffn_tiles(shape, num_cu=torch.cuda.get_device_properties(0).multi_processor_count)
    assert tiles[0] == tiles[2] == "256x256/8"
    g = torch.Generator("cuda").manual_seed(d)
    rnd = lambda *s, std=1.0: (torch.randn(*s, generator=g, device="cuda") * std).bfloat16()
    x, dy, W1, W2 = rnd(T, d), rnd(T, d), rnd(E, F, d, std=0.1), rnd(E, d, F, std=0.1)
    b1 = torch.randn(E, F, generator=g, device="cuda") * 0.1
    tok = torch.randint(0, T, (P,), generator=g, device="cuda", dtype=torch.int32)
    gate = torch.rand(P, generator=g, device="cuda")
    buf = lambda n: torch.full((P, n), 7.0, dtype=torch.bfloat16, device="cuda")
    H, A, O, dXp = buf(F), buf(F), buf(d), buf(d)
    ctx = B.Context()
    B.evomoe_expert_ffn(ctx, shape, x, tok, offs, W1, b1, W2, None, H, A, O)
    dO = (gate[:, None] * dy[tok.long()].float()).bfloat16()
    db1 = torch.zeros(E, F, device="cuda")
    ws = torch.empty(B.evomoe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    B.evomoe_expert_ffn_bwd(ctx, shape, dO, H, A, x, tok, offs, W1, W2, dy, gate, None, db1, None, None, dXp, False, ws)
    torch.cuda.synchronize()
    dH = ws[:P * F * 2].view(torch.bfloat16).view(P, F)
    o = offs.tolist()

    def near(got, want, what, more=0.0):
        # one rounding to bf16 of a float32 value (2^-9, twice that for the decision at a tie), float32 sums of 248 products and
        # the gelu's own error (2.2e-5) below 2e-4
        err = (got.float() - want).abs()
        assert (err <= 2 ** -8 * want.abs() + 2e-4 + more).all(), (what, err.max().item())

    for e in range(E):
        r = slice(o[e], o[e + 1])
        if r.start == r.stop:
            assert (db1[e] == 0).all()
            continue
        t = tok[r].long()
        Href = x[t].float() @ W1[e].float().T + b1[e]
        near(H[r], Href, ("H", e))
        near(A[r], torch.nn.functional.gelu(Href) if act == "gelu" else Href.clamp(min=0), ("A", e))
        hb = H[r].float()
        slope = 0.5 * (1 + torch.erf(hb / 2 ** 0.5)) + hb * torch.exp(-hb * hb / 2) / (2 * torch.pi) ** 0.5 \
            if act == "gelu" else (hb > 0).float()
        dA = gate[r, None] * (dy[t].float() @ W2[e].float())
        want = dA * slope
        near(dH[r], want, ("dH", e), 2.5e-4 * dA.abs())       # gelu' is taken as 0 or 1 beyond 4.2: up to 2.4e-4 off
        # the same per row, and float32 sums of up to 60000 rows
        bound = (2.5e-4 * dA.abs() + 1e-5 * want.abs()).sum(0) + 1e-6
        assert ((db1[e] - want.double().sum(0)).abs() <= bound).all(), ("db1", e)
    ctx.close()
