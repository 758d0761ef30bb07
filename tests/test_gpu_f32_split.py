"""The float32 expert FFN takes its operands apart into bf16 terms: accuracy over contraction lengths and magnitudes."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402


@pytest.mark.parametrize("T,d,E,F,scale", [(300, 64, 2, 64, 1.0), (500, 4, 1, 4, 1.0), (260, 256, 4, 516, 1.0),
                                           (700, 516, 2, 1024, 1.0), (260, 256, 4, 516, 1e18), (260, 256, 4, 516, 1e-18)])
def test_f32_contractions_are_as_exact_as_float32_sums(T, d, E, F, scale):
    """Float32 products added one k at a time in four partial sums have a relative rms error of about 2.6e-8 sqrt(K / 8), the
    additions of the partial sums and the bias a few roundings more: sqrt(K / 8 + 6) in all.  Nothing may be above that."""
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("split", T=T, d=d, E=E, F=F, act="relu", dtype="f32", taus=(1.0,), threshold=0.9, seed=77,
                            bias_std=0.0)
    gl = h.GpuLayer(synth.make_layer_inputs(cfg))
    P = gl.forward(1.0, 0.9)
    assert P == T
    b, p, B = gl.buf, gl.params, h.B
    x, dO = gl.x * scale, torch.randn(gl.shape.P_cap, d, generator=torch.Generator("cuda").manual_seed(5), device="cuda") * scale
    H, A, O = torch.zeros_like(b.H), torch.zeros_like(b.A), torch.zeros_like(b.O)
    B.evomoe_expert_ffn(gl.ctx, gl.shape, x, b.pair_token, b.expert_offsets, p.W1, None, p.W2, None, H, A, O)
    B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, dO, H, A, x, b.pair_token, b.expert_offsets, p.W1, p.W2, None, None, b.dW1, None,
                            b.dW2, None, b.dXp, False, b.workspace)
    dH = b.workspace[:P * F * 4].view(torch.float32).view(P, F)
    off = b.expert_offsets.tolist()
    err = {}
    for e in range(E):
        r = slice(off[e], off[e + 1])
        xr, W1, W2 = x[b.pair_token[r].long()].double(), p.W1[e].double(), p.W2[e].double()
        for what, k, got, want in (("H", d, H[r], xr @ W1.T), ("O", F, O[r], A[r].double() @ W2.T),
                                   ("dH", d, dH[r], (dO[r].double() @ W2) * (H[r] > 0)), ("dXp", F, b.dXp[r], dH[r].double() @ W1),
                                   ("dW1", r.stop - r.start, b.dW1[e], dH[r].double().T @ xr),
                                   ("dW2", r.stop - r.start, b.dW2[e], dO[r].double().T @ A[r].double())):
            unit = want.abs().max()                          # (squares of 1e36 leave float32, not float64)
            rel = (((got.double() - want) / unit).square().sum() / (want / unit).square().sum()).sqrt().item()
            assert rel <= 2.6e-8 * (k / 8 + 6) ** 0.5, (what, e, rel)
            err[what] = max(rel, err.get(what, 0.0))
    print(T, d, E, F, scale, {k: f"{v:.2g}" for k, v in err.items()})


def test_f32_largest_values_stay_finite():
    """3.4e38 is above the largest bf16 value: its first term must not become infinite."""
    import torch
    import gpu_harness as h
    cfg = synth.LayerConfig("large", T=40, d=64, E=1, F=64, act="relu", dtype="f32", taus=(1.0,), threshold=0.9, seed=78,
                            bias_std=0.0)
    gl = h.GpuLayer(synth.make_layer_inputs(cfg))
    P = gl.forward(1.0, 0.9)
    b, p, B = gl.buf, gl.params, h.B
    x = torch.zeros_like(gl.x)
    x[b.pair_token[3].long(), 17] = 3.4e38
    H = torch.zeros_like(b.H)
    B.evomoe_expert_ffn(gl.ctx, gl.shape, x, b.pair_token, b.expert_offsets, p.W1, None, p.W2, None, H, b.A, b.O)
    want = x[b.pair_token[:P].long()].double() @ p.W1[0].double().T
    assert torch.isfinite(H).all()
    assert ((H[:P].double() - want).abs() <= 2e-7 * want.abs()).all()


@pytest.mark.parametrize("d,F,tile", [(64, 128, "32x32/4"), (516, 1028, "64x64/4")])
def test_f32_weight_gradients_of_a_few_rows(d, F, tile):
    """Experts with 1 to 49 rows.  n float32 products added one behind the other in chains of eight have a relative rms error of
    2.52e-8 sqrt((n + 1) / 2), n <= 8, of sqrt((8 + 1) / 2 + 1) above and more beyond 32: nothing may be above that (8 % for the
    samples: the mantissas of a row of dO and one of A are behind all products of a single row)."""
    import torch
    import gpu_harness as h
    from helpers import ffn_tiles
    B, counts = h.B, [1, 2, 3, 0, 5, 8, 16, 17, 48, 49]
    E, P = len(counts), sum(counts)
    offs = [sum(counts[:e]) for e in range(E + 1)]
    shape = B.make_shape(P, d, E, F, "f32", "relu", P)
    assert ffn_tiles(shape, num_cu=torch.cuda.get_device_properties(0).multi_processor_count)[4] == tile
    g = torch.Generator("cuda").manual_seed(d)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    dO, x, A, W1, W2 = rnd(P, d), rnd(P, d), rnd(P, F), rnd(E, F, d), rnd(E, d, F)
    dW1, dW2, dXp = torch.empty(E, F, d, device="cuda"), torch.empty(E, d, F, device="cuda"), torch.empty(P, d, device="cuda")
    ws = torch.empty(B.evomoe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    tok = torch.randperm(P, generator=g, device="cuda").int()
    ctx = B.Context()
    B.evomoe_expert_ffn_bwd(ctx, shape, dO, torch.ones_like(A), A, x, tok, torch.tensor(offs, dtype=torch.int32, device="cuda"), W1, W2,
                            None, None, dW1, None, dW2, None, dXp, False, ws)
    torch.cuda.synchronize()
    dH = ws[:P * F * 4].view(torch.float32).view(P, F).double()
    for e, n in enumerate(counts):
        r = slice(offs[e], offs[e + 1])
        for what, got, want in (("dW2", dW2[e], dO[r].double().T @ A[r].double()), ("dW1", dW1[e], dH[r].T @ x[tok[r].long()].double())):
            err = ((got.double() - want).square().sum() / want.square().sum().clamp(min=1e-300)).sqrt().item()
            print(what, n, f"{err:.3g}")
            assert err <= 1.08 * 2.52e-8 * (((min(n, 8) + 1) / 2 + (n > 8)) ** 0.5), (what, n, err)
    ctx.close()


def _ffn(offsets, d, F, x, W1):
    """H of a float32 layer without biases."""
    import torch
    import gpu_harness as h
    B, E, P = h.B, len(offsets) - 1, offsets[-1]
    shape = B.make_shape(P, d, E, F, "f32", "relu", P)
    offs = torch.tensor(offsets, dtype=torch.int32, device="cuda")
    H, A, O = torch.empty(P, F, device="cuda"), torch.empty(P, F, device="cuda"), torch.empty(P, d, device="cuda")
    ctx = B.Context()
    B.evomoe_expert_ffn(ctx, shape, x, None, offs, W1, None, torch.zeros(E, d, F, device="cuda"), None, H, A, O)
    torch.cuda.synchronize()
    ctx.close()
    return H


@pytest.mark.parametrize("d,F", [(64, 64), (256, 2048)])
def test_f32_sums_overflow_where_float32_does(d, F):
    """Products on either side of the largest float32 value, 2^128 - 2^104, by less than the smaller terms of the operands."""
    import torch
    x, W1 = torch.zeros(40, d, device="cuda"), torch.zeros(1, F, d, device="cuda")
    x[:20, 17], x[20:, 17] = 1.99 * 2.0 ** 63, -1.99 * 2.0 ** 63
    W1[0, :, 17] = torch.linspace(1.0, 1.02, F, device="cuda") * 2.0 ** 64
    H = _ffn([0, 40], d, F, x, W1)
    want = (x.double() @ W1[0].double().T).float()
    assert want.isinf().any() and want.isfinite().any()
    assert torch.equal(H.isinf(), want.isinf()) and torch.equal(H.sign(), want.sign())
    ok = want.isfinite()
    assert ((H - want).abs()[ok] <= 2e-7 * want.abs()[ok]).all()


@pytest.mark.parametrize("bits", [0x7f800001, 0x7f80ffff, 0x7fc00000, 0xff800100 - 2 ** 32, 0x7fffffff])
@pytest.mark.parametrize("d,F", [(64, 64), (256, 2048)])
def test_f32_nans_stay_nans(bits, d, F):
    """Also those whose payload a bf16 value does not have."""
    import torch
    rnd = lambda *s: torch.randn(*s, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    x, W1 = rnd(40, d), rnd(1, F, d)
    x.view(torch.int32)[7, d - 1] = bits
    W1.view(torch.int32)[0, 5, 3] = bits
    H = _ffn([0, 40], d, F, x, W1)
    want = torch.zeros_like(H, dtype=torch.bool)
    want[7], want[:, 5] = True, True
    assert torch.equal(H.isnan(), want) and H[~want].isfinite().all()


@pytest.mark.parametrize("d,F", [(64, 64), (256, 2048)])
@pytest.mark.parametrize("exponent", [-108, -110, -114, -118, -126])
def test_f32_small_values_lose_no_more_than_the_last_terms_range(exponent, d, F):
    """The smallest bf16 subnormal is 2^-133: an x is off by up to half of it, times the weights, beside the error of ordinary values,
    2.6e-8 sqrt(K / 8 + 6) of the root of the products' sum of squares, rms, as above; no output is further off than five times that
    (82 000 normal errors stay within 4.5)."""
    import torch
    g = torch.Generator("cuda").manual_seed(1)
    rnd = lambda *s: torch.rand(*s, generator=g, device="cuda")
    x = (rnd(40, d) + 1) * torch.sign(rnd(40, d) - 0.5) * 2.0 ** exponent
    W1 = torch.randn(1, F, d, generator=g, device="cuda") * 64          # (so that the results are no subnormals)
    H = _ffn([0, 40], d, F, x, W1).double()
    xd, Wd = x.double(), W1[0].double()
    size = (xd.square() @ Wd.square().T).sqrt()
    bound = 2.0 ** -134 * Wd.abs().sum(1) + 5 * 2.6e-8 * (d / 8 + 6) ** 0.5 * size
    assert ((H - xd @ Wd.T).abs() <= bound).all()


@pytest.mark.parametrize("gathered,accumulate,which", [(True, False, "both"), (False, True, "both"), (True, True, "dW1"),
                                                       (False, False, "dW2")])
def test_f32_weight_gradients_of_a_few_rows_are_those_of_tiles(gathered, accumulate, which):
    """Up to 48 rows of an expert, waves work without the LDS (32 rows by 64 columns of a gradient each) where the launch has two such
    pieces for every block: the same bits as in 64x64 tiles, which the expert alone is worked in.  No side is a multiple of a piece's."""
    import torch
    import gpu_harness as h
    from helpers import ffn_tiles
    B, d, F, counts = h.B, 516, 1028, [1, 0, 15, 16, 17, 31, 33, 47, 48, 49, 63, 65, 130, 0]
    E, P = len(counts), sum(counts)
    offs = [sum(counts[:e]) for e in range(E + 1)]
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert ffn_tiles(B.make_shape(P, d, E, F, "f32", "relu", P), num_cu=cu)[4] == "64x64/4"
    tiles = 2 * -(-d // 64) * -(-F // 64)
    pieces = -(-d // 32) * -(-F // 64) + -(-F // 32) * -(-d // 64)
    if which != "both":
        tiles, pieces = tiles // 2, pieces // 2              # (either problem has about half of the pieces)
    assert pieces + 8 < 2 * min(tiles, 2 * cu) and (pieces - 8) * sum(n <= 48 for n in counts) >= 2 * 2 * cu
    g = torch.Generator("cuda").manual_seed(8)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    dO, x, A, W1, W2, start1, start2 = rnd(P, d), rnd(P, d), rnd(P, F), rnd(E, F, d), rnd(E, d, F), rnd(E, F, d), rnd(E, d, F)
    tok = torch.randperm(P, generator=g, device="cuda").int() if gathered else None
    dXp, ctx = torch.empty(P, d, device="cuda"), B.Context()

    def gradients(experts):
        first, last = offs[experts[0]], offs[experts[-1] + 1]
        e = slice(experts[0], experts[-1] + 1)
        shape = B.make_shape(P, d, len(experts), F, "f32", "relu", max(1, last - first))
        r = slice(first, max(last, first + 1))
        dW1, dW2 = start1[e].clone(), start2[e].clone()
        ws = torch.empty(B.evomoe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
        part = torch.tensor([offs[i] - first for i in range(experts[0], experts[-1] + 2)], dtype=torch.int32, device="cuda")
        B.evomoe_expert_ffn_bwd(ctx, shape, dO[r].clone(), torch.ones_like(A[r]), A[r].clone(), x if gathered else x[r].clone(),
                                tok[r].clone() if gathered else None, part, W1[e].clone(), W2[e].clone(), None, None,
                                dW1 if which != "dW2" else None, None, dW2 if which != "dW1" else None, None, dXp, accumulate, ws)
        torch.cuda.synchronize()
        return {"both": (dW1, dW2), "dW1": (dW1,), "dW2": (dW2,)}[which]

    together = gradients(range(E))
    for e in range(E):
        if offs[e] == P:
            continue                                         # (no row to hand over for the last, empty one)
        for got, want in zip(together, gradients([e])):
            assert torch.equal(got[e], want[0]), (e, counts[e])
    first = start2 if which == "dW2" else start1
    assert torch.equal(together[0][-1], first[-1] if accumulate else torch.zeros_like(first[-1]))
    ctx.close()


# (single waves, tiles of 64x64 and of 32x32)
@pytest.mark.parametrize("d,F,E,n", [(64, 64, 1, 40), (516, 1028, 8, 40), (516, 1028, 8, 200)])
@pytest.mark.parametrize("bits", [0x7f800001, 0xff80ffff - 2 ** 32, 0x7fc00000])
def test_f32_nans_stay_nans_in_the_backward(d, F, E, n, bits):
    """One NaN in an operand: every output that it is multiplied into is one, no other."""
    import torch
    import gpu_harness as h
    B, P, e = h.B, E * n, E - 1                              # the last expert's
    shape = B.make_shape(P, d, E, F, "f32", "relu", P)
    g = torch.Generator("cuda").manual_seed(1)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    base = {"dO": rnd(P, d), "A": rnd(P, F), "x": rnd(P, d), "W1": rnd(E, F, d), "W2": rnd(E, d, F)}
    offs = torch.arange(0, P + 1, n, dtype=torch.int32, device="cuda")
    tok = torch.arange(P, dtype=torch.int32, device="cuda")
    dW1, dW2, dXp = torch.empty(E, F, d, device="cuda"), torch.empty(E, d, F, device="cuda"), torch.empty(P, d, device="cuda")
    ws = torch.empty(B.evomoe_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    ctx, r, i, j = B.Context(), P - 2, d - 3, F - 5
    rows = slice(e * n, P)
    for what, at in (("dO", (r, i)), ("A", (r, j)), ("x", (r, i)), ("W1", (e, j, i)), ("W2", (e, i, j))):
        t = dict(base)
        t[what] = base[what].clone()
        t[what].view(torch.int32)[at] = bits
        B.evomoe_expert_ffn_bwd(ctx, shape, t["dO"], torch.ones_like(base["A"]), t["A"], t["x"], tok, offs, t["W1"], t["W2"], None, None,
                                dW1, None, dW2, None, dXp, False, ws)
        torch.cuda.synchronize()
        dH = ws[:P * F * 4].view(torch.float32).view(P, F)
        want = {k: torch.zeros_like(v, dtype=torch.bool) for k, v in (("dH", dH), ("dXp", dXp), ("dW1", dW1), ("dW2", dW2))}
        if what == "dO":
            want["dH"][r], want["dXp"][r], want["dW1"][e], want["dW2"][e, i] = True, True, True, True
        if what == "W2":
            want["dH"][rows, j], want["dXp"][rows], want["dW1"][e, j] = True, True, True
        if what == "A":
            want["dW2"][e, :, j] = True
        if what == "x":
            want["dW1"][e, :, i] = True
        if what == "W1":
            want["dXp"][rows, i] = True
        for k, v in (("dH", dH), ("dXp", dXp), ("dW1", dW1), ("dW2", dW2)):
            assert torch.equal(v.isnan(), want[k]) and v[~want[k]].isfinite().all(), (what, k)
    ctx.close()

