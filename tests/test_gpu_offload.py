"""The expert FFN with host-resident weights must give the resident expert FFN's output bit
for bit (same kernels and tiles, experts launched one after the other), for any number of
resident slots; and through it the oracle's output within the layer's tolerance."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_17223_amd as moe
import workloads as wl
from gpu_util import DEV, DeviceLayer, rel_rms_err, shape_of

pytestmark = pytest.mark.gpu
PULLED = 1            # moe_path_calls: weights read over the link by a kernel

CASES = {
    "small": wl.scaled("gpt2s_moe", T=1000, d=256, h=512),
    "ragged": wl.scaled("gpt2s_moe", T=333, d=72, h=200, E=5, k=2, cf=0.8),
    "skewed": wl.scaled("skewed", T=2048, d=256, h=384),
    "stack_layer_tall": wl.scaled("infer_stack", T=256, d=512, h=2048),
}


@pytest.mark.parametrize("name", list(CASES))
def test_offloaded_ffn_equals_resident_ffn(name):
    li = wl.make_layer(CASES[name], seed=0)
    s = shape_of(li)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    want = b["ye"].clone()
    A = int(b["offsets"].cpu().numpy()[-1])
    W1h, W2h = b["W1p"].cpu().pin_memory(), b["W2p"].cpu().pin_memory()
    ws = torch.empty(moe.moe_offload_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    for resident in (1, 2, 3, li.E, li.E + 5):
        staging = torch.empty(moe.moe_offload_staging_bytes(s, resident), dtype=torch.uint8, device=DEV)
        ye = torch.full_like(want, 5.0)
        for _ in range(2):                         # twice: slots and events are reused
            moe.moe_expert_ffn_offloaded(s, b["xe"], b["offsets"], W1h, W2h, None, None, ye, staging,
                                         resident, ws)
        torch.cuda.synchronize()
        assert torch.equal(ye[:A * li.d].view(torch.int16), want[:A * li.d].view(torch.int16)), resident
        got = ye.float().cpu().numpy().reshape(-1, li.d)[:A]
    # and against the oracle, on its own packed rows
    o = oracle.moe_layer(li.x, li.Wg, li.W1, li.W2, k=li.k, capacity=li.C, bias=li.gate_bias,
                         bias_stride=li.bias_token_stride)
    ref = oracle.ffn_rows(o.xe, o.off, li.W1, li.W2, np.arange(o.A, dtype=np.int32))
    assert rel_rms_err(got, ref) <= 2e-2


@pytest.mark.parametrize("T,d,h", [(3, 8, 8), (3, 72, 200), (5, 256, 512), (40, 264, 1032)])
def test_weights_in_page_locked_and_in_pageable_memory_give_the_same(T, d, h):
    """The kernel that reads page-locked weights against the runtime's copies: matrices smaller than
    one pass of its blocks, and with remainders; experts without rows among them."""
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=T, d=d, h=h, E=13), seed=1)
    s = shape_of(li)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    A = int(b["offsets"].cpu().numpy()[-1])
    want = b["ye"].clone()[:A * d].view(torch.int16)
    counts = np.diff(b["offsets"].cpu().numpy())
    assert T > 5 or (counts == 0).any()
    W1, W2 = b["W1p"].cpu(), b["W2p"].cpu()
    ws = torch.empty(moe.moe_offload_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    staging = torch.empty(moe.moe_offload_staging_bytes(s, 2), dtype=torch.uint8, device=DEV)
    for W1h, W2h in ((W1.pin_memory(), W2.pin_memory()), (W1, W2), (W1.pin_memory(), W2)):
        staging.fill_(0xFF)
        ye = torch.full_like(b["ye"], 5.0)
        calls = moe.moe_path_calls(PULLED)
        moe.moe_expert_ffn_offloaded(s, b["xe"], b["offsets"], W1h, W2h, None, None, ye, staging, 2, ws)
        torch.cuda.synchronize()
        assert moe.moe_path_calls(PULLED) - calls == (W1h.is_pinned() and W2h.is_pinned())
        assert torch.equal(ye[:A * d].view(torch.int16), want)


def test_page_locked_weights_changed_between_calls():
    """The host writes new weights over the old ones: the kernel that reads them sees no earlier call's
    values, also where experts take turns on one slot."""
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=200, d=128, h=256, E=5), seed=3)
    s = shape_of(li)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    A = int(b["offsets"].cpu().numpy()[-1])
    W1, W2 = b["W1p"].cpu(), b["W2p"].cpu()
    W1h, W2h = W1.clone().pin_memory(), W2.clone().pin_memory()
    ws = torch.empty(moe.moe_offload_workspace_bytes(s), dtype=torch.uint8, device=DEV)

    def call(w1, w2, resident):
        ye = torch.full_like(b["ye"], 5.0)
        staging = torch.empty(moe.moe_offload_staging_bytes(s, resident), dtype=torch.uint8, device=DEV)
        moe.moe_expert_ffn_offloaded(s, b["xe"], b["offsets"], w1, w2, None, None, ye, staging, resident, ws)
        torch.cuda.synchronize()
        return ye[:A * li.d].view(torch.int16)

    for i, resident in enumerate((2, 1, 3, 2)):
        p1 = torch.roll(W1.reshape(-1), 8 * i).reshape(W1.shape)
        p2 = torch.roll(W2.reshape(-1), 16 * i).reshape(W2.shape)
        W1h.copy_(p1)
        W2h.copy_(p2)
        assert torch.equal(call(W1h, W2h, resident), call(p1, p2, resident)), i


@pytest.mark.parametrize("E,resident", [(1, 1), (5, 1), (5, 2), (5, 5)])
def test_page_locked_weights_under_capture(E, resident):
    """Both copy streams join the caller's, also with one expert or one slot; a replay reads the weights
    that the host memory holds then.  Eager calls between the replays, in the same staging area."""
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=200, d=128, h=256, E=E, k=min(E, 2)), seed=3)
    s = shape_of(li)
    L = DeviceLayer(li, s)
    L.layer(1)
    b = L.b
    A = int(b["offsets"].cpu().numpy()[-1])
    W1, W2 = b["W1p"].cpu(), b["W2p"].cpu()
    W1h, W2h = W1.clone().pin_memory(), W2.clone().pin_memory()
    ws = torch.empty(moe.moe_offload_workspace_bytes(s), dtype=torch.uint8, device=DEV)
    staging = torch.empty(moe.moe_offload_staging_bytes(s, resident), dtype=torch.uint8, device=DEV)
    ye = torch.full_like(b["ye"], 5.0)

    def call(w1, w2):
        moe.moe_expert_ffn_offloaded(s, b["xe"], b["offsets"], w1, w2, None, None, ye, staging, resident, ws)

    call(W1h, W2h)
    torch.cuda.synchronize()
    graph, calls = torch.cuda.CUDAGraph(), moe.moe_path_calls(PULLED)
    with torch.cuda.graph(graph):
        call(W1h, W2h)
    assert moe.moe_path_calls(PULLED) == calls + 1
    for rep in range(3):
        p1 = torch.roll(W1.reshape(-1), 8 * rep).reshape(W1.shape)
        p2 = torch.roll(W2.reshape(-1), 16 * rep).reshape(W2.shape)
        call(p1, p2)
        torch.cuda.synchronize()
        want = ye.clone()
        W1h.copy_(p1)
        W2h.copy_(p2)
        ye.fill_(5.0)
        staging.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(ye.view(torch.int16), want.view(torch.int16)), rep
        assert (ye[A * li.d:] == 5.0).all()


def test_sizes_and_refusals():
    li = wl.make_layer(wl.scaled("gpt2s_moe", T=64, d=64, h=128, E=4), seed=0)
    s = shape_of(li)
    per = 64 * 128 * 2
    assert moe.moe_offload_staging_bytes(s, 2) == 2 * 2 * per
    assert moe.moe_offload_staging_bytes(s, 9) == 4 * 2 * per          # never more slots than experts
    assert moe.moe_offload_staging_bytes(s, 0) == 0
    f32 = shape_of(wl.make_layer(wl.CONFIGS["tiny_fp32"], seed=0))
    assert moe.moe_offload_staging_bytes(f32, 2) == 0 and moe.moe_offload_workspace_bytes(f32) == 0
