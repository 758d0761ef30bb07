"""db2 of a bf16 layer: dO's column sums behind dXp's tiles, on blocks that are idle in the last round and on the others, with
the tiles in one sequence or an eighth of it per XCD, and in a launch of their own."""
import pytest

pytestmark = pytest.mark.gpu

from helpers import ffn_tiles  # noqa: E402

BLOCKS_PER_CU = {"64x64/4": 2, "64x128/4": 2, "128x128/4": 1, "128x256/8": 1, "256x256/4": 1}      # of dXp's tiles


# pairs, d, E, F, announced pairs (0: none), dXp's tile, whether every XCD walks an eighth of its own, rounds of tiles; with few pairs
# announced a larger number takes several rounds
@pytest.mark.parametrize("P,d,E,F,hint,tile,eighths,rounds", [
    (200, 768, 16, 3072, 0, "64x64/4", True, 1), (8192, 768, 16, 3072, 0, "128x256/8", True, 1),
    (20000, 768, 16, 3072, 8192, "128x256/8", True, 2), (6000, 768, 16, 3072, 200, "64x64/4", True, 3),
    (9000, 768, 16, 3072, 2500, "128x128/4", True, 2), (5626, 136, 7, 264, 0, "64x128/4", False, 1),
    (20000, 512, 64, 2048, 0, "256x256/4", False, 1), (20000, 512, 64, 2048, 5000, "64x128/4", False, 3),
    (1, 64, 1, 64, 0, "64x64/4", False, 1),
    (30000, 768, 5, 256, 0, "256x256/4", False, 2)])         # (from 32 MB of dO on in a launch of its own)
def test_column_sums(P, d, E, F, hint, tile, eighths, rounds):
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
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    bm, bn = (int(n) for n in tile.split("/")[0].split("x"))
    columns = -(-d // bn)
    group = columns if bm * F * 2 >= 1 << 20 else int(2.4 * 2 ** 20) // (bn * F * 2)     # column tiles that an XCD's L2 holds
    tiles = sum(-(-n // bm) for n in offs.diff().tolist()) * columns
    walk = (-(-tiles // 8), cu * BLOCKS_PER_CU[tile] // 8) if eighths else (tiles, cu * BLOCKS_PER_CU[tile])
    assert ffn_tiles(shape, hint, cu)[3] == tile and (max(1, group) < columns) == eighths and -(-walk[0] // walk[1]) == rounds
    dO, x, H, W1, W2 = rnd(P, d), rnd(T, d), rnd(P, F), rnd(E, F, d), rnd(E, d, F)
    A = H.clamp(min=0)
    db2 = torch.full((E, d), 3.0, device="cuda")
    dXp = torch.empty(P, d, dtype=torch.bfloat16, device="cuda")
    ws = torch.full((B.evomoe_workspace_bytes(shape),), 255, dtype=torch.uint8, device="cuda")     # NaN: a sum left out shows
    ctx = B.Context()
    B.evomoe_hint_pairs(ctx, hint)
    B.evomoe_expert_ffn_bwd(ctx, shape, dO, H, A, x, None, offs, W1, W2, None, None, None, None, None, db2, dXp, False, ws)
    torch.cuda.synchronize()
    o = offs.tolist()
    for e in range(E):
        rows = dO[o[e]:o[e + 1]].double()
        # up to 330 float32 additions behind one another (a row lane's rows, the lanes, the ranges), 2^-24 of the sum of magnitudes each
        assert ((db2[e] - rows.sum(0)).abs() <= 330 * 2 ** -24 * rows.abs().sum(0)).all(), e
    ctx.close()
