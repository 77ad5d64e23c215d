"""Layers whose weight matrices are past 2^31 bytes: the four-wavefront GEMM kernels address their
operands with 32-bit offsets, so the register-staged kernels run here (and nowhere else with
128 x 256 tiles).  Reference: the layer and its gradients in fp32 on the device, expert by expert."""
import math

import pytest
import torch

import paper_2210_17223_amd as moe
from gpu_util import DEV

pytestmark = pytest.mark.gpu

# as for the small shapes: forward one 16-bit operand rounding on the path, gradients two
TOL_Y, TOL_GRAD = 2e-2, 3e-2


def rms(t):
    return float(t.square().mean().sqrt())


def worst(got, want):
    """Largest difference, in multiples of the reference's RMS."""
    return float((got - want).abs_().max()) / rms(want)


def worst_beyond_rounding(got, want):
    """The same beyond 2^-7 of each element: sums of a few outer products of rounded factors."""
    bound = want.abs().mul_(2.0 ** -7)
    return float((got - want).abs_().sub_(bound).max()) / rms(want)


@pytest.mark.parametrize("d,h", [(32768, 32768), (32776, 32840)], ids=["whole_stages", "ragged"])
def test_layer_and_gradients_past_32_bit_offsets(d, h):
    T, E, k = 300, 2, 1
    assert d * h * 2 >= 2 ** 31 - 64
    s = moe.Shape.make(T, d, E, h, k, T, dtype="bf16", act="gelu")
    for which in (0, 1):
        assert moe.moe_expert_gemm_kernel(s, which) == "grouped_gemm_staged_kernel 128x256"
    g = torch.Generator(device=DEV)
    g.manual_seed(17)

    def normal(*shape, std=1.0, dtype=torch.bfloat16):
        return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=g)

    x, Wg = normal(T, d), normal(d, E, std=1.0 / math.sqrt(d))
    W1, W2 = normal(E, d, h, std=1.0 / math.sqrt(d)), normal(E, h, d, std=1.0 / math.sqrt(h))
    b = moe.alloc_buffers(s, 1, DEV)
    moe.moe_pack_gate(s, Wg, b["Wgp"])
    moe.moe_pack_weights(s, W1, W2, b["W1p"], b["W2p"])
    pre = torch.empty(T * h, dtype=torch.float16, device=DEV)
    hid = torch.empty_like(pre)
    moe.moe_layer_forward_keep(s, x, b["Wgp"], None, 0, b["W1p"], None, b["W2p"], None, b["expert_idx"],
                               b["gate"], b["counts"], b["offsets"], b["slot_of"], b["src_of"], b["xe"],
                               b["ye"], pre, hid, b["y"], b["workspace"])
    kept_y = b["y"].clone()
    moe.moe_layer_chunked(s, 1, x, b["Wgp"], None, 0, b["W1p"], None, b["W2p"], None, b["expert_idx"],
                          b["gate"], b["counts"], b["offsets"], b["slot_of"], b["src_of"], b["xe"], b["ye"],
                          b["y"], None, b["workspace"])
    torch.cuda.synchronize()
    assert torch.equal(kept_y.view(torch.int32), b["y"].view(torch.int32))
    print("forward done", d, h, flush=True)

    dy = normal(T, d, dtype=torch.float32)
    f32 = dict(dtype=torch.float32, device=DEV)
    ws = torch.empty(moe.moe_backward_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    grads = []
    for kept in (True, False):                           # with kept activations, and computed again
        out = dict(dx=torch.empty((T, d), **f32), dWg=torch.empty((d, E), **f32), dW1=torch.empty((E, d, h), **f32),
                   dW2=torch.empty((E, h, d), **f32), dgate=torch.empty(T * k, **f32))
        moe.moe_layer_backward(s, x, b["Wgp"], None, 0, W1, W2, b["W1p"], b["expert_idx"], b["gate"], b["offsets"],
                               b["slot_of"], b["src_of"], b["xe"], b["ye"], pre if kept else None,
                               hid if kept else None, dy, out["dx"], out["dWg"], out["dW1"], out["dW2"],
                               out["dgate"], ws)
        torch.cuda.synchronize()
        print("backward done", kept, flush=True)
        grads.append(out)
    del ws, pre, hid

    # the reference, from the library's own routing (integers are compared by the other tests)
    off = b["offsets"].tolist()
    assert off[-1] == T and min(off[1], T - off[1]) > 64
    src = b["src_of"][:T].long()
    p = torch.softmax(x.float() @ Wg.float(), dim=1)
    gate = b["gate"]
    y, dx = torch.zeros((T, d), **f32), torch.zeros((T, d), **f32)
    dgate = torch.zeros(T, **f32)
    for e in range(E):
        t = src[off[e]:off[e + 1]]                       # k = 1: an assignment is its token
        assert bool((b["expert_idx"].view(-1)[t] == e).all())
        xe = x[t].float()
        W = W1[e].float()
        P = xe @ W
        phi = 0.5 * (1.0 + torch.erf(P / math.sqrt(2.0)))
        H = P * phi
        slope = phi + P * torch.exp(-0.5 * P * P) / math.sqrt(2.0 * math.pi)
        V = W2[e].float()
        ye = H @ V
        y[t] = gate[t, None] * ye
        dgate[t] = (ye * dy[t]).sum(1)
        dye = gate[t, None] * dy[t]
        dP = (dye @ V.t()) * slope
        del V
        dx[t] += dP @ W.t()
        del W
        for got in grads:
            assert worst_beyond_rounding(got["dW2"][e], H.t() @ dye) <= TOL_GRAD
            assert worst_beyond_rounding(got["dW1"][e], xe.t() @ dP) <= TOL_GRAD
    dg = torch.zeros((T, E), **f32).scatter_(1, b["expert_idx"].view(T, 1).long(), dgate[:, None])
    dz = p * (dg - (p * dg).sum(1, keepdim=True))
    dx += dz @ Wg.float().t()
    assert worst(b["y"].view(T, d), y) <= TOL_Y
    for got in grads:
        assert worst(got["dx"], dx) <= TOL_GRAD
        assert worst(got["dgate"], dgate) <= 5e-3
        assert worst(got["dWg"], x.float().t() @ dz) <= TOL_GRAD
