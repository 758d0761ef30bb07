"""The float32 expert FFN: backward with some outputs left out, the bias gradients' error, infinities in partial slabs."""
import pytest

pytestmark = pytest.mark.gpu

import synth_inputs as synth  # noqa: E402


def _layer(T, d, E, F, threshold=0.1):
    import gpu_harness as h
    cfg = synth.LayerConfig("f32-bwd", T=T, d=d, E=E, F=F, act="gelu", dtype="f32", taus=(1.0,), threshold=threshold,
                            seed=523, bias_std=0.02)
    return h, h.GpuLayer(synth.make_layer_inputs(cfg))


@pytest.mark.parametrize("keep", [("db1",), ("db2",), ("db1", "db2"), ("dW1", "db1", "db2"), ("dW2", "db1", "db2"),
                                  ("dW1", "db1", "dW2", "db2")], ids="-".join)
def test_f32_gradients_accumulate_with_others_left_out(keep):
    """g + g is exact: two accumulating calls onto zeros give twice the gradient of the full call, bit for bit."""
    import torch
    h, gl = _layer(300, 68, 3, 132)            # several experts, several tiles of every matrix
    gl.forward(1.0, 0.1)
    gl.backward(1.0)
    b, p, B = gl.buf, gl.params, h.B
    got = {n: torch.zeros_like(getattr(b, n)) for n in keep}
    for _ in range(2):
        B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, b.dO, b.H, b.A, gl.x, b.pair_token, b.expert_offsets, p.W1, p.W2, gl.dy,
                                b.pair_gate, got.get("dW1"), got.get("db1"), got.get("dW2"), got.get("db2"), b.dXp, True,
                                b.workspace)
    torch.cuda.synchronize()
    for n in keep:
        assert torch.equal(got[n], 2 * getattr(b, n)), n


@pytest.mark.parametrize("T,d,F", [(16384, 64, 64), (700, 64, 64), (16384, 256, 1024)])
def test_f32_bias_gradients_are_summed_in_short_chains(T, d, F):
    """A chain of n additions of N(0,1) values has a relative error of about 2.5e-8 sqrt(n / 2) (rounding errors of 0.42 * 2^-24
    of the running sum each); levels of chains add up under the root.  Chains of 8, 16, 16 and 16 terms, what one expert's
    16384 rows take at most, make 1.3e-7; twice that is the bound.  One chain of 4096 terms would be at 1.1e-6."""
    import torch
    h, gl = _layer(T, d, 1, F, threshold=0.9)
    assert gl.forward(1.0, 0.9) == T
    gl.backward(1.0)
    b, p, B = gl.buf, gl.params, h.B
    dO = torch.randn(T, d, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, dO, b.H, b.A, gl.x, b.pair_token, b.expert_offsets, p.W1, p.W2, None, None,
                            b.dW1, b.db1, b.dW2, b.db2, b.dXp, False, b.workspace)
    dH = b.workspace[:T * F * 4].view(torch.float32).view(T, F)        # the workspace begins with dH
    for what, got, rows in (("db2", b.db2, dO), ("db1", b.db1, dH)):
        want = rows.double().sum(0)
        scale = (rows.double() ** 2).sum(0).sqrt()                     # what the sum is worth if its terms are independent
        err = (((got[0].double() - want) / scale) ** 2).mean().sqrt().item()
        print(what, T, d, F, f"{err:.3g}")
        assert err <= 2.7e-7, (what, err)


def test_f32_infinite_operands_stay_infinite_in_partial_slabs():
    """No contraction length is a multiple of a slab here.  An infinity in the last element of a contraction must reach the
    result as in plain arithmetic: a slab's padding must not turn it into 0 * Inf."""
    import torch
    h, gl = _layer(45, 60, 1, 124, threshold=0.9)
    P = gl.forward(1.0, 0.9)
    assert P == 45
    b, p, B, inf = gl.buf, gl.params, h.B, float("inf")

    def same(got, want, what):
        got, want = got.double().cpu(), want.cpu()
        assert not torch.isnan(want).any() and torch.isinf(want).any(), what
        assert torch.equal(torch.isinf(got), torch.isinf(want)) and not torch.isnan(got).any(), what
        assert torch.equal(got[torch.isinf(want)], want[torch.isinf(want)]), what

    x = gl.x[b.pair_token[:P].long()].double().cpu()
    W1, W2 = p.W1.clone(), p.W2.clone()
    W1[0, 7, 59] = inf
    W2[0, 9, 123] = inf
    A0 = b.A[:P].double().cpu()
    H, A, O = torch.zeros_like(b.H), torch.zeros_like(b.A), torch.zeros_like(b.O)
    B.evomoe_expert_ffn(gl.ctx, gl.shape, gl.x, b.pair_token, b.expert_offsets, W1, p.b1, p.W2, p.b2, H, A, O)
    same(H[:P], x @ W1[0].double().cpu().T, "H")
    B.evomoe_expert_ffn(gl.ctx, gl.shape, gl.x, b.pair_token, b.expert_offsets, p.W1, p.b1, W2, p.b2, H, A, O)
    same(O[:P], A0 @ W2[0].double().cpu().T, "O")

    dO = torch.randn(gl.shape.P_cap, 60, generator=torch.Generator("cuda").manual_seed(6), device="cuda")
    dW1, dW2 = torch.zeros_like(p.W1), torch.zeros_like(p.W2)

    def backward(A=b.A, x=gl.x, W1=p.W1, W2=p.W2):
        B.evomoe_expert_ffn_bwd(gl.ctx, gl.shape, dO, torch.zeros_like(b.H), A, x, b.pair_token, b.expert_offsets, W1, W2,
                                None, None, dW1, None, dW2, None, b.dXp, False, b.workspace)
        torch.cuda.synchronize()

    W2 = p.W2.clone()
    W2[0, 59, 5] = inf                                     # dH = (dO W2) * act'(0), act'(0) = 1/2
    backward(W2=W2)
    dH = b.workspace[:P * 124 * 4].view(torch.float32).view(P, 124)
    same(dH, dO[:P].double().cpu() @ W2[0].double().cpu() * 0.5, "dH")
    W1 = p.W1.clone()
    W1[0, 123, 5] = inf
    backward(W1=W1)
    same(b.dXp[:P], dH.double().cpu() @ W1[0].double().cpu(), "dXp")
    A = b.A.clone()
    A[P - 1, 3] = inf
    x = gl.x.clone()
    x[b.pair_token[P - 1], 4] = inf
    backward(A=A, x=x)
    same(dW2[0], dO[:P].double().cpu().T @ A[:P].double().cpu(), "dW2")
    same(dW1[0], dH.double().cpu().T @ x[b.pair_token[:P].long()].double().cpu(), "dW1")
