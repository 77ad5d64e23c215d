"""Calls on several streams: what one caller's launches leave to another's."""
import time

import pytest
import torch

import paper_2210_17223_amd as moe
from gpu_util import DEV

pytestmark = pytest.mark.gpu


class Layer:
    """A bf16 layer of random operands; only its time is looked at."""

    def __init__(self, T, d, E, h, k):
        s = self.s = moe.Shape.make(T, d, E, h, k, T, dtype="bf16", act="gelu")
        g = torch.Generator(device=DEV).manual_seed(1)
        normal = lambda *shape, std=0.02: torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=g)
        self.x = normal(T, d, std=1.0)
        b = self.b = moe.alloc_buffers(s, 1, DEV)
        moe.moe_pack_gate(s, normal(d, E), b["Wgp"])
        moe.moe_pack_weights(s, normal(E, d, h), normal(E, h, d), b["W1p"], b["W2p"])
        torch.cuda.synchronize()

    def __call__(self):
        b = self.b
        moe.moe_layer_chunked(self.s, 1, self.x, b["Wgp"], None, 0, b["W1p"], None, b["W2p"], None, b["expert_idx"],
                              b["gate"], b["counts"], b["offsets"], b["slot_of"], b["src_of"], b["xe"], b["ye"], b["y"],
                              None, b["workspace"])


def test_a_decode_step_gets_in_beside_large_layers():
    """The large layer's GEMMs take 2 ms each on blocks that have a compute unit to themselves and give it up every 0.2 ms.  Nine
    of ten decode steps (five launches) then take less than 1.0 ms, where behind whole GEMMs it was 2.0 and with a tile per
    block 0.75; 1.5 is asked for.  (Two streams that share a hardware queue take turns: several pairs are tried.)"""
    large, small = Layer(32768, 2048, 8, 8192, 2), Layer(16, 768, 16, 3072, 2)
    for layer in (large, small):
        layer()
    torch.cuda.synchronize()
    seen = []
    for _ in range(12):
        a, b = torch.cuda.Stream(), torch.cuda.Stream()
        end, times = torch.cuda.Event(), []
        with torch.cuda.stream(a):
            for _ in range(8):
                large()
            end.record()
        with torch.cuda.stream(b):
            while not end.query():
                at = time.perf_counter()
                small()
                done = torch.cuda.Event()
                done.record()
                done.synchronize()
                times.append(time.perf_counter() - at)
        torch.cuda.synchronize()
        times.sort()
        seen.append(times[len(times) * 9 // 10] * 1e3)
        if seen[-1] < 1.5:
            break
    assert seen[-1] < 1.5, seen
