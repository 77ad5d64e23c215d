"""Parity of the layer's backward pass with the backward oracle: every gradient within
3e-2 of the oracle gradient's RMS (max-abs); dgate much tighter (it is an fp32 dot product
of fp32 rows).  The forward's bound is 2e-2 with ONE 16-bit operand rounding on the path
(the hidden activation); the input and first-layer weight gradients pass through TWO
chained bf16 operand roundings (dye, then dP), each of relative RMS 2^-9/sqrt(3): the
expected error grows by sqrt(2), and so does the bound (2.8e-2, rounded to 3e-2)."""
import math
import threading

import numpy as np
import pytest
import torch

import paper_2210_17223_amd as moe
import workloads as wl
from gpu_util import DEV, DeviceLayer, rel_rms_err, shape_of, upload
from oracle import bwd_oracle as bo

pytestmark = pytest.mark.gpu
BESIDE = 0            # moe_path_calls: weight gradients on a side stream
TOL = 3e-2

CASES = {
    "small": wl.scaled("gpt2s_moe", T=1000, d=256, h=512),
    "ragged_dims": wl.scaled("gpt2s_moe", T=333, d=72, h=200, E=5, k=2, cf=0.8),
    "k1_e6": wl.scaled("gpt2s_moe", T=700, d=192, h=320, E=6, k=1, cf=1.0),
    "k3": wl.scaled("gpt2s_moe", T=512, d=128, h=264, E=8, k=3, cf=1.1),
    "skewed": wl.scaled("skewed", T=2048, d=256, h=384),
    "stack_layer": wl.scaled("infer_stack", T=256, d=256, h=512),
}


def run_backward(li, act="gelu", keep=False, n_chunks=1, with_oracle=True):
    """keep: the forward is moe_layer_forward_keep and hands its pre-activations to the
    backward pass; else the plain layer call, and the backward pass computes them again."""
    s = shape_of(li, act=act)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    pre = hid = None
    if keep:
        plain = {n: b[n].clone() for n in ("expert_idx", "gate", "counts", "offsets", "slot_of", "y")}
        A = int(b["offsets"][-1])
        plain["src_of"], plain["ye"] = b["src_of"][:A].clone(), b["ye"][:A * li.d].clone()
        for n in ("expert_idx", "gate", "counts", "offsets", "slot_of", "src_of", "y", "ye"):
            b[n].fill_(-3)
        pre = torch.full((moe.moe_max_rows(s) * li.h,), 9.0, dtype=torch.float16, device=DEV)
        hid = torch.full_like(pre, 5.0)
        moe.moe_layer_forward_keep(s, L.x, b["Wgp"], L.bias, L.bias_stride, b["W1p"], None, b["W2p"], None,
                                   b["expert_idx"], b["gate"], b["counts"], b["offsets"], b["slot_of"],
                                   b["src_of"], b["xe"], b["ye"], pre, hid, b["y"], b["workspace"])
        torch.cuda.synchronize()
        # same outputs as the plain layer call, bit for bit
        for n, want in plain.items():
            got = b[n][:want.numel()]
            assert torch.equal(got.view(torch.int32), want.view(torch.int32)), n
        # kept pre-activations: fp16 roundings of xe W1 (bf16 products, fp32 accumulation)
        o_pre = _oracle_pre(li, b, A)
        got_pre = pre[:A * li.h].float().cpu().numpy().reshape(A, li.h)
        rms = float(np.sqrt(np.mean(o_pre ** 2)))
        assert np.abs(got_pre - o_pre).max() <= 2.0 ** -10 * np.abs(o_pre).max() + 1e-4 * rms
        assert (pre[A * li.h:] == 9.0).all()              # rows beyond offsets[E] untouched
        # kept hidden activations: act of the fp32 accumulator, rounded to fp16
        from oracle import bwd_oracle as _bo
        o_hid = _bo.act_and_derivative(o_pre, act)[0]
        got_hid = hid[:A * li.h].float().cpu().numpy().reshape(A, li.h)
        assert np.abs(got_hid - o_hid).max() <= 2.0 ** -10 * np.abs(o_hid).max() + 1e-4 * rms
        assert (hid[A * li.h:] == 5.0).all()
    prng = np.random.Generator(np.random.PCG64(77))
    dy = prng.standard_normal((li.T, li.d)).astype(np.float32)
    W1, W2 = upload(li.W1, "bf16"), upload(li.W2, "bf16")
    f32 = lambda *shape: torch.full(shape, 7.0, dtype=torch.float32, device=DEV)
    g = dict(dx=f32(li.T * li.d), dWg=f32(li.d * li.E), dW1=f32(li.E * li.d * li.h),
             dW2=f32(li.E * li.d * li.h), dgate=f32(li.T * li.k))
    ws = torch.empty(moe.moe_backward_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    moe.moe_layer_backward(s, L.x, b["Wgp"], L.bias, L.bias_stride, W1, W2, b["W1p"], b["expert_idx"],
                           b["gate"], b["offsets"], b["slot_of"], b["src_of"], b["xe"], b["ye"], pre, hid,
                           torch.from_numpy(dy).to(DEV), g["dx"], g["dWg"], g["dW1"], g["dW2"],
                           g["dgate"], ws, n_chunks=n_chunks)
    torch.cuda.synchronize()
    if not with_oracle:
        return {n: t.cpu().numpy() for n, t in g.items()}, None
    o = bo.moe_layer_backward(li.x, li.Wg, li.W1, li.W2, dy, k=li.k, capacity=li.C, act=act,
                              bias=li.gate_bias, bias_stride=li.bias_token_stride)
    assert np.array_equal(b["slot_of"].cpu().numpy(), o.fwd.slot_of)
    return {n: t.cpu().numpy() for n, t in g.items()}, o


def _oracle_pre(li, b, A):
    """xe W1 per expert in fp64 from the host inputs and the (already checked) plan."""
    off = b["offsets"].cpu().numpy()
    tok = b["src_of"][:A].cpu().numpy() // li.k
    xe = li.x.astype(np.float64)[tok]
    P = np.empty((A, li.h))
    for e in range(li.E):
        P[off[e]:off[e + 1]] = xe[off[e]:off[e + 1]] @ li.W1[e].astype(np.float64)
    return P


@pytest.mark.parametrize("keep", [False, True], ids=["recompute", "keep"])
@pytest.mark.parametrize("name", list(CASES))
def test_backward_matches_the_oracle(name, keep):
    li = wl.make_layer(CASES[name], seed=0)
    got, o = run_backward(li, keep=keep)
    T, d, E, h, k = li.T, li.d, li.E, li.h, li.k
    assert rel_rms_err(got["dgate"].reshape(T, k), o.dgate) <= 5e-3
    assert rel_rms_err(got["dx"].reshape(T, d), o.dx) <= TOL
    assert rel_rms_err(got["dWg"].reshape(d, E), o.dWg) <= TOL
    assert rel_rms_err(got["dW1"].reshape(E, d, h), o.dW1) <= TOL
    assert rel_rms_err(got["dW2"].reshape(E, h, d), o.dW2) <= TOL
    # per expert too: a wrong row range would hide in the layer-wide RMS
    for e in range(E):
        if o.fwd.count[e] == 0:
            assert not got["dW1"].reshape(E, d, h)[e].any() and not got["dW2"].reshape(E, h, d)[e].any()
        else:
            # An expert with a handful of rows has gradients that are (sums of few) outer
            # products of two bf16-rounded factors: the error of an element is relative to
            # that element (up to 2 x 2^-9 per product), and the largest elements of an
            # outer product are ~20 x its RMS.  Hence relative plus absolute bound here.
            for got_e, ref_e in ((got["dW1"].reshape(E, d, h)[e], o.dW1[e]),
                                 (got["dW2"].reshape(E, h, d)[e], o.dW2[e])):
                rms = float(np.sqrt(np.mean(ref_e ** 2)))
                assert (np.abs(got_e - ref_e) <= 2.0 ** -7 * np.abs(ref_e) + TOL * rms).all(), e
    # a fully dropped token has a zero input gradient
    dropped = (o.fwd.slot_of.reshape(T, k) < 0).all(1)
    assert not got["dx"].reshape(T, d)[dropped].any()


# dP's GEMM over d: one, two and three stages of 64 and a tail, on 256 x 256 (many tiles) and 128 x 128 tiles, and long
# contractions, whole stages and a tail, on 256 x 256 and 128 x 256, with rows and columns that end inside a tile; dxe's over h on
# all three and on 128 x 128 with five stages on their way.  The last shape's weight gradients are 256 x 256 tiles of 66 stages, one to
# a share.  keep: the forward's first GEMM takes dP's tiles, the shape of d = 1928 with five stages on their way.
@pytest.mark.parametrize("keep", [False, True], ids=["recompute", "keep"])
@pytest.mark.parametrize("T,h,d,dp,dxe", [
    (6000, 8712, 40, "256x256", "128x128 deep"), (6000, 8712, 64, "256x256", "128x128 deep"),
    (6000, 8712, 136, "256x256", "128x128 deep"), (6000, 8712, 192, "256x256", "128x128 deep"),
    (600, 264, 8, "128x128", "128x128"), (600, 264, 64, "128x128", "128x128"), (600, 264, 72, "128x128", "128x128"),
    (600, 264, 128, "128x128", "128x128"), (600, 264, 200, "128x128", "128x128"),
    (4000, 1608, 3080, "256x256", "256x256"), (700, 2008, 264, "128x128", "128x128 deep"),
    (300, 1920, 72, "128x128", "128x128 deep"), (4000, 1608, 3072, "128x256", "256x256"),
    (7500, 2152, 3080, "128x256", "256x256"), (6000, 3072, 1032, "256x256", "128x256"),
    (700, 264, 1928, "128x128", "128x128"), (4200, 8192, 4096, "256x256", "256x256")])
def test_backward_of_few_stages(T, h, d, dp, dxe, keep):
    s = moe.Shape.make(T, d, 1, h, 1, T, dtype="bf16", act="gelu")
    assert [moe.moe_backward_gemm_kernel(s, which) for which in (0, 1)] == [f"bwd_gemm_w4_kernel {t}" for t in (dp, dxe)]
    assert moe.moe_expert_gemm_kernel(s, 0).endswith(" deep" if (T, h, d) == (700, 264, 1928) else f" {dp}")
    # one expert with every token: gate weight 1, no gradient through the gate, dx = dP W1^T
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=T, d=d, h=h, E=1, k=1, cf=1.0), seed=5)
    got, _ = run_backward(li, keep=keep, with_oracle=False)
    f64 = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV).double()
    x, W1, W2 = f64(li.x), f64(li.W1[0]), f64(li.W2[0])
    dy = f64(np.random.Generator(np.random.PCG64(77)).standard_normal((T, d)).astype(np.float32))
    P = x @ W1
    cdf = 0.5 * (1.0 + torch.erf(P / math.sqrt(2.0)))
    dP = (dy @ W2.T) * (cdf + P * torch.exp(-0.5 * P * P) / math.sqrt(2.0 * math.pi))
    for name, ref in (("dx", dP @ W1.T), ("dW1", x.T @ dP), ("dW2", (P * cdf).T @ dy)):
        assert rel_rms_err(got[name].reshape(ref.shape), ref.cpu().numpy()) <= TOL, name


def test_backward_is_bitwise_reproducible():
    # fixed-order sums everywhere (no floating-point atomics): two runs, the same bits
    li = wl.make_layer(CASES[list(CASES)[0]], seed=3)
    a, _ = run_backward(li, keep=True)
    b, _ = run_backward(li, keep=True)
    for name in a:
        assert np.array_equal(a[name].view(np.uint32), b[name].view(np.uint32)), name


@pytest.mark.parametrize("keep", [False, True], ids=["recompute", "keep"])
@pytest.mark.parametrize("name", ["skewed", "k3"])
def test_chunked_backward_changes_no_bit(name, keep):
    """moe_layer_backward_chunked: every gradient is the same bits for every n_chunks, with one
    group of GEMMs per chunk (all side streams and events in use), with a few chunks per group,
    and with the default grouping (one group at these sizes)."""
    li = wl.make_layer(CASES[name], seed=2)
    ref, _ = run_backward(li, keep=keep, with_oracle=False)
    for group_rows, chunks in ((1, (2, 3, 8, 64)), (64, (4, 8)), (0, (4,))):
        before = moe.moe_tune_ffn_group_rows(group_rows)
        try:
            for n_chunks in chunks:
                got, _ = run_backward(li, keep=keep, n_chunks=n_chunks, with_oracle=False)
                for n in ref:
                    assert np.array_equal(got[n].view(np.uint32), ref[n].view(np.uint32)), (n, n_chunks, group_rows)
        finally:
            moe.moe_tune_ffn_group_rows(before)


@pytest.mark.parametrize("act", ["relu", "gelu_tanh", "identity"])
def test_backward_other_activations(act):
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=400, d=128, h=256, E=4), seed=3)
    got, o = run_backward(li, act=act, keep=act != "relu")
    for n, shape in (("dx", (li.T, li.d)), ("dWg", (li.d, li.E)), ("dW1", li.W1.shape), ("dW2", li.W2.shape)):
        assert rel_rms_err(got[n].reshape(shape), getattr(o, n)) <= TOL, n


@pytest.mark.parametrize("d,h,E,T,C", [(128, 256, 8, 600, 400), (768, 1024, 64, 700, 300)],
                         ids=["small", "weight_gradient_in_256_tiles"])
def test_backward_with_empty_experts_and_gate_bias(d, h, E, T, C):
    """Two experts take every token, up to their capacity; the others stay empty and get zero
    weight gradients.  The second shape has enough 256 x 256 weight-gradient tiles (64 experts) for
    the four-wavefront kernel: experts without rows, and a contraction that ends inside a stage."""
    cfg = wl.scaled("gpt2s_moe", T=T, d=d, h=h, E=E, k=2, cf=None)
    li = wl.make_layer(cfg, seed=5)
    bias = np.zeros(li.E, np.float32)
    bias[[1, 6]] = 30.0                                  # every token picks experts 1 and 6
    li.gate_bias, li.bias_token_stride, li.C = bias, 0, C
    got, o = run_backward(li)
    assert set(np.nonzero(o.fwd.count)[0]) == {1, 6}
    for n, shape in (("dx", (li.T, li.d)), ("dWg", (li.d, li.E))):
        assert rel_rms_err(got[n].reshape(shape), getattr(o, n)) <= TOL, n
    for e in (1, 6):          # against the expert's own RMS: the empty experts' zeros tell nothing
        assert rel_rms_err(got["dW1"].reshape(li.W1.shape)[e], o.dW1[e]) <= TOL
        assert rel_rms_err(got["dW2"].reshape(li.W2.shape)[e], o.dW2[e]) <= TOL
    for e in range(E):
        if e not in (1, 6):
            assert not got["dW1"].reshape(li.W1.shape)[e].any() and not got["dW2"].reshape(li.W2.shape)[e].any()


def test_kept_activations_through_the_large_weight_gradient_tiles():
    """dW2 from the kept fp16 activations, rounded to bf16 between the LDS read and the multiply, on
    256 x 256 tiles (64 experts x 3 x 4 tiles): against the oracle, expert by expert.  An element sums
    at most 66 products of two factors rounded to bf16 (relative error up to 2 x 2^-9 each): few enough
    that the largest elements carry an error of their own size, so the bound has a part relative to
    the element (2^-7, twice one product's) beside TOL of the expert's RMS, as for the small experts
    above."""
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=2100, d=768, h=1024, E=64, k=2, cf=1.0), seed=9)
    got, o = run_backward(li, keep=True)
    for n, shape in (("dW1", li.W1.shape), ("dW2", li.W2.shape)):
        for e in range(li.E):
            ref, err = getattr(o, n)[e], np.abs(got[n].reshape(shape)[e] - getattr(o, n)[e])
            assert (err <= 2.0 ** -7 * np.abs(ref) + TOL * np.sqrt(np.mean(ref ** 2))).all(), (n, e)


@pytest.mark.parametrize("keep", [False, True], ids=["recompute", "keep"])
def test_weight_gradients_beside_the_other_gemms(keep):
    """Rows x d x h above 2.7e9: the weight gradients run on a side stream, and in launch order while
    stages are timed.  The same bits either way, and the oracle's gradients, on 5 x 6 tiles of 256 x 256
    (squares of four that end inside a band)."""
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=700, d=1280, h=1536, E=18, k=2, cf=1.0), seed=4)
    assert moe.moe_max_rows(shape_of(li)) * li.d * li.h >= 2.7e9
    calls = moe.moe_path_calls(BESIDE)
    got, o = run_backward(li, keep=keep)
    assert moe.moe_path_calls(BESIDE) == calls + 1
    for n, shape in (("dW1", li.W1.shape), ("dW2", li.W2.shape)):
        for e in range(li.E):
            ref, err = getattr(o, n)[e], np.abs(got[n].reshape(shape)[e] - getattr(o, n)[e])
            assert (err <= 2.0 ** -7 * np.abs(ref) + TOL * np.sqrt(np.mean(ref ** 2))).all(), (n, e)
    moe.moe_profile_enable(1, 64)
    try:
        ordered, _ = run_backward(li, keep=keep, with_oracle=False)
    finally:
        moe.moe_profile_enable(0, 0)
    assert moe.moe_path_calls(BESIDE) == calls + 1
    for n in got:
        assert np.array_equal(got[n].view(np.uint32), ordered[n].view(np.uint32)), n


def test_gelu_over_all_16_bit_arguments():
    """Hidden activations for every bf16 value of 2^-13 to 12, both signs, as the pre-activation (token rows
    with a single one): half a unit of fp16 beside the fp32 evaluation's error, which is 6.5e-7 (the fit's
    5.4e-7, and half a unit of its argument's size at 4) and falls with v: |v| (4e-5 |v| + 3e-7), since the
    fitted slope at zero is off by 3.8e-5."""
    bits = np.arange(0x3900, 0x4141, dtype=np.uint32)
    v = (np.concatenate([bits, bits | 0x8000]) << 16).view(np.float32)
    v = np.concatenate([v, np.ones(-len(v) % 8, np.float32)])
    T, d, h = 8, 64, len(v)
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=T, d=d, h=h, E=1, k=1, cf=None), seed=0)
    li.x[:], li.W1[:] = 0.0, 0.0
    li.x[:, 0], li.W1[0, 0] = 1.0, v
    b = PreparedBackward(li, keep=True)
    torch.cuda.synchronize()
    v = v.astype(np.float64)
    exact = v * np.array([0.5 * math.erfc(-t / math.sqrt(2.0)) for t in v])
    unit = np.spacing(np.abs(exact).astype(np.float16)).astype(np.float64)
    bound = unit / 2 + np.minimum(6.5e-7, np.abs(v) * (4e-5 * np.abs(v) + 3e-7)) + 2.0 ** -23 * np.abs(exact)
    pre = b.pre[:T * h].double().cpu().numpy().reshape(T, h)
    hid = b.hid[:T * h].double().cpu().numpy().reshape(T, h)
    assert (pre == v.astype(np.float16)).all()
    assert (np.abs(hid - exact) <= bound).all()


class PreparedBackward:
    """A layer's backward pass ready to be called: everything it reads, its gradients, a workspace."""

    def __init__(self, li, keep=False, ws=None):
        self.s = s = shape_of(li)
        self.L = L = DeviceLayer(li, s)
        b, self.pre, self.hid = L.b, None, None
        if keep:
            self.pre = torch.zeros(moe.moe_max_rows(s) * li.h, dtype=torch.float16, device=DEV)
            self.hid = torch.zeros_like(self.pre)
            moe.moe_layer_forward_keep(s, L.x, b["Wgp"], L.bias, L.bias_stride, b["W1p"], None, b["W2p"], None,
                                       b["expert_idx"], b["gate"], b["counts"], b["offsets"], b["slot_of"],
                                       b["src_of"], b["xe"], b["ye"], self.pre, self.hid, b["y"], b["workspace"])
        else:
            L.layer(1)
        self.W1, self.W2 = upload(li.W1, "bf16"), upload(li.W2, "bf16")
        f32 = lambda n: torch.zeros(n, dtype=torch.float32, device=DEV)
        self.g = dict(dx=f32(li.T * li.d), dWg=f32(li.d * li.E), dW1=f32(li.W1.size), dW2=f32(li.W2.size),
                      dgate=f32(li.T * li.k))
        self.ws = torch.zeros(moe.moe_backward_workspace_bytes(s), dtype=torch.uint8, device=DEV) if ws is None else ws
        g = torch.Generator(device=DEV)
        g.manual_seed(li.T)
        self.dy = torch.empty((li.T, li.d), device=DEV).normal_(generator=g)
        torch.cuda.synchronize()

    def __call__(self, dy=None, n_chunks=1):
        b, g = self.L.b, self.g
        moe.moe_layer_backward(self.s, self.L.x, b["Wgp"], self.L.bias, self.L.bias_stride, self.W1, self.W2,
                               b["W1p"], b["expert_idx"], b["gate"], b["offsets"], b["slot_of"], b["src_of"],
                               b["xe"], b["ye"], self.pre, self.hid, self.dy if dy is None else dy, g["dx"],
                               g["dWg"], g["dW1"], g["dW2"], g["dgate"], self.ws, n_chunks=n_chunks)

    def ordered(self, dy=None):
        """The same call with its launches in order on one stream (stages timed)."""
        moe.moe_profile_enable(1, 64)
        try:
            self(dy)
            torch.cuda.synchronize()
        finally:
            moe.moe_profile_enable(0, 0)
        return self.copy()

    def copy(self):
        return {n: t.clone() for n, t in self.g.items()}

    def spoil(self):
        for t in self.g.values():
            t.fill_(7.0)

    def check(self, want, what):
        for n, t in self.g.items():
            assert torch.equal(t.view(torch.int32), want[n].view(torch.int32)), (n, what)


def medium_layer(seed=4):
    return wl.make_layer(wl.scaled("gpt2s_moe", T=700, d=1280, h=1536, E=18, k=2, cf=1.0), seed=seed)


@pytest.mark.parametrize("keep", [False, True], ids=["recompute", "keep"])
def test_eager_backward_beside_the_capture_of_a_chunked_one(keep):
    """While a backward pass of four groups is being captured on one stream, a medium layer's runs on
    another: the call works, the capture holds, both give the bits of the calls alone."""
    medium = PreparedBackward(medium_layer(), keep)
    chunked = PreparedBackward(wl.make_layer(CASES["skewed"], seed=2), keep)
    before = moe.moe_tune_ffn_group_rows(1)
    try:
        chunked(n_chunks=4)
        medium()                       # (also: every kernel has been launched once)
        torch.cuda.synchronize()
        want_chunked, want = chunked.copy(), medium.ordered()
        other, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        medium.spoil()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            chunked(n_chunks=4)
            calls = moe.moe_path_calls(BESIDE)
            with torch.cuda.stream(other):
                medium()
            assert moe.moe_path_calls(BESIDE) == calls + 1
    finally:
        moe.moe_tune_ffn_group_rows(before)
    torch.cuda.synchronize()
    medium.check(want, "during the capture")
    for rep in range(3):
        chunked.spoil()
        medium.spoil()
        torch.cuda.synchronize()
        graph.replay()
        medium()
        torch.cuda.synchronize()
        chunked.check(want_chunked, rep)
        medium.check(want, rep)


def test_captured_backward_of_a_medium_layer():
    """Under capture the launches stay in order: replays give the eager bits, with eager calls of the same
    layer between them."""
    b = PreparedBackward(medium_layer(), keep=True)
    b()
    torch.cuda.synchronize()
    want, graph = b.ordered(), torch.cuda.CUDAGraph()
    calls = moe.moe_path_calls(BESIDE)
    with torch.cuda.graph(graph):
        b()
    assert moe.moe_path_calls(BESIDE) == calls
    for rep in range(3):
        b.spoil()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        b.check(want, rep)
        b.spoil()
        b()
        torch.cuda.synchronize()
        b.check(want, ("eager", rep))


def test_backward_calls_in_a_row_and_on_several_streams():
    """Medium layers, nothing waited for in between: one call after another with other inputs on the same
    workspace; then six streams, more than the library has side streams, each its own layer's calls, from
    one thread and from a thread each."""
    a = PreparedBackward(medium_layer(), keep=True)
    others = [a.dy * f for f in (0.5, -3.0, 0.25)]
    want = [a.ordered(dy) for dy in others]
    got = []
    for dy in others:
        a(dy)
        got.append(a.copy())                        # on the same stream, behind the call
    for n, dy in enumerate(others):
        for key in want[n]:
            assert torch.equal(got[n][key].view(torch.int32), want[n][key].view(torch.int32)), (key, n)
    beside = moe.moe_path_calls(BESIDE)
    calls = [PreparedBackward(medium_layer(seed), keep=seed % 2 == 0) for seed in range(6)]
    want = [c.ordered() for c in calls]
    streams = [torch.cuda.Stream() for _ in calls]

    def work(i):
        with torch.cuda.stream(streams[i]):
            for _ in range(3):
                calls[i].spoil()
                calls[i]()

    torch.cuda.synchronize()
    for _ in range(2):
        for i in range(len(calls)):
            work(i)
    torch.cuda.synchronize()
    for c, w in zip(calls, want):
        c.check(w, "one thread")
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for c, w in zip(calls, want):
        c.check(w, "threads")
    assert moe.moe_path_calls(BESIDE) == beside + 6 * 3 * 3


def test_kept_buffers_come_together():
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=64, d=64, h=64, E=4), seed=0)
    s = shape_of(li)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    pre = torch.zeros(moe.moe_max_rows(s) * li.h, dtype=torch.float16, device=DEV)
    W1, W2 = upload(li.W1, "bf16"), upload(li.W2, "bf16")
    f32 = lambda n: torch.zeros(n, dtype=torch.float32, device=DEV)
    ws = torch.empty(moe.moe_backward_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    for keep in ((pre, None), (None, pre)):
        with pytest.raises(moe.MoeError):
            moe.moe_layer_backward(s, L.x, b["Wgp"], None, 0, W1, W2, b["W1p"], b["expert_idx"], b["gate"],
                                   b["offsets"], b["slot_of"], b["src_of"], b["xe"], b["ye"], keep[0], keep[1],
                                   f32(li.T * li.d), f32(li.T * li.d), f32(li.d * li.E), f32(li.E * li.d * li.h),
                                   f32(li.E * li.d * li.h), f32(li.T * li.k), ws)


def test_refusals():
    li = wl.make_layer(wl.CONFIGS["tiny_fp32"], seed=0)
    assert moe.moe_backward_workspace_bytes(shape_of(li)) == 0          # fp32 layers: unsupported
    s = shape_of(wl.make_layer(wl.scaled("gpt2s_moe", T=64, d=64, h=64, E=4), seed=0), renorm=True)
    assert moe.moe_backward_workspace_bytes(s) == 0
