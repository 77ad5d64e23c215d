"""moe_calib_gemm against fp64 products of the same operands."""
import pytest
import torch

import paper_2210_17223_amd as moe
from gpu_util import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gelu", [False, True])
def test_whole_gemm_of_long_and_short_contractions(gelu):
    """Below four stages of 64 the call takes another kernel than from there on; both in one process, in both orders, on
    full and partial tiles and more of them than a block takes at once."""
    g = torch.Generator(device=DEV).manual_seed(4)
    E, N = 3, 768
    ends = [0, 300, 301, 557]
    for K in (192, 256, 64, 512, 128):
        A = torch.randn(ends[-1], K, device=DEV, generator=g).to(torch.bfloat16)
        W = (torch.randn(E, N, K, device=DEV, generator=g) * 0.1).to(torch.bfloat16)
        out = torch.zeros(ends[-1], N, device=DEV, dtype=torch.float16)
        items = [(e, r, min(r + 256, ends[e + 1]), n) for e in range(E) for r in range(ends[e], ends[e + 1], 256)
                 for n in range(0, N, 256)] * 40         # (the same tiles again: 480 entries for 256 blocks)
        items = torch.tensor(items, dtype=torch.int32, device=DEV).reshape(-1)
        n_items = torch.tensor([items.numel() // 4], dtype=torch.int32, device=DEV)
        moe.moe_calib_gemm(A, W, out, items, n_items, N, K, 0, gelu)
        torch.cuda.synchronize()
        want = torch.cat([A[ends[e]:ends[e + 1]].double() @ W[e].double().T for e in range(E)])
        if gelu:
            want = 0.5 * want * (1.0 + torch.erf(want / 2.0 ** 0.5))
        # one fp16 rounding (2^-11 of the value), fp32 sums and the GeLU's own error, a tenth of that
        assert ((out.double() - want).abs() <= 2.0 ** -10 * want.abs() + 2e-4 * want.abs().max()).all(), K


@pytest.mark.parametrize("K", [128, 1088, 8192])
def test_every_tile_of_several_shares(K):
    """Shares of 32, 7 and 1 tiles: entries past 256 of them go to further blocks.  Every tile is another one, of 1 to 4
    rows; the last block's share is not full."""
    g = torch.Generator(device=DEV).manual_seed(5)
    N, ends = 2048, [0]
    while len(ends) <= 1201:
        ends.append(ends[-1] + 1 + len(ends) * 7 % 4)
    A = torch.randn(ends[-1], K, device=DEV, generator=g).to(torch.bfloat16)
    W = (torch.randn(1, N, K, device=DEV, generator=g) * 0.1).to(torch.bfloat16)
    out = torch.full((ends[-1], N), 7e4, device=DEV).to(torch.float16)           # (infinity where no tile is written)
    items = torch.tensor([(0, a, b, n) for a, b in zip(ends, ends[1:]) for n in range(0, N, 256)], dtype=torch.int32,
                         device=DEV).reshape(-1)
    n_items = torch.tensor([items.numel() // 4 - 3], dtype=torch.int32, device=DEV)
    moe.moe_calib_gemm(A, W, out, items, n_items, N, K, 0, False)
    torch.cuda.synchronize()
    assert torch.isinf(out[ends[-2]:, N - 768:]).all()                            # the three entries past n_items
    out[ends[-2]:, N - 768:] = 0.0
    want = A.double() @ W[0].double().T
    want[ends[-2]:, N - 768:] = 0.0
    assert ((out.double() - want).abs() <= 2.0 ** -10 * want.abs() + 2e-4 * want.abs().max()).all()
