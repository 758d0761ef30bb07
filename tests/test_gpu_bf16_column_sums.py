"""db2 of a bf16 layer: dO's column sums behind dXp's tiles, on blocks that are idle in the last round and on the others, with
the tiles in one sequence or an eighth of it per XCD, and in a launch of their own."""
import pytest

pytestmark = pytest.mark.gpu


# few tiles, an eighth per XCD; the same with more than one tile per block of some XCDs; one sequence; 64 experts; own launch
@pytest.mark.parametrize("P,d,E,F", [(200, 768, 16, 3072), (8192, 768, 16, 3072), (5626, 136, 7, 264), (20000, 512, 64, 2048),
                                     (30000, 768, 5, 256), (1, 64, 1, 64)])
def test_column_sums(P, d, E, F):
    import torch
    import gpu_harness as h
    B = h.B
    T = P
    g = torch.Generator("cuda").manual_seed(P)
    cuts = torch.randint(0, P + 1, (E - 1,), generator=g, device="cuda").sort().values
    if E > 2:
        cuts[1] = cuts[0]                                    # an empty expert
    offs = torch.cat([cuts.new_zeros(1), cuts, cuts.new_full((1,), P)]).int()
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").bfloat16()
    shape = B.make_shape(T, d, E, F, "bf16", "relu", P)
    dO, x, H, W1, W2 = rnd(P, d), rnd(T, d), rnd(P, F), rnd(E, F, d), rnd(E, d, F)
    A = H.clamp(min=0)
    db2 = torch.full((E, d), 3.0, device="cuda")
    dXp = torch.empty(P, d, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((B.evomoe_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")     # NaN: a sum left out shows
    ctx = B.Context()
    B.evomoe_expert_ffn_bwd(ctx, shape, dO, H, A, x, None, offs, W1, W2, None, None, None, None, None, db2, dXp, False, ws)
    torch.cuda.synchronize()
    o = offs.tolist()
    for e in range(E):
        rows = dO[o[e]:o[e + 1]].double()
        # up to 330 float32 additions behind one another (a row lane's rows, the lanes, the ranges), 2^-24 of the sum of magnitudes each
        assert ((db2[e] - rows.sum(0)).abs() <= 330 * 2 ** -24 * rows.abs().sum(0)).all(), e
    ctx.close()
