"""Long-chunk projections in every tile shape of the product, at the edges of
its tiles, of the 16-token shrink tiles and of the 64-column delta chunks, with
padding and unused adapters full of NaN.

Against plain float64. y is rounded once (2^-8 of it: bf16 keeps 8 bits), U_s is rounded to bf16
before the up-projection (2^-8 of every product with it), and every sum is
float32: of K products, of K products inside U_s and of r products (2^-24 of
the absolute values' sum each)."""
import pytest
import torch

import paper_2608_15241_amd as lk
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

CASES = [
    # T, K, N, n_ad, r_max, ranks: the tile that the sizes select
    (2000, 64, 4032, 4, 16, None),                     # 128 x 256
    (1000, 128, 4032, 9, 24, [24, 3, 17, 24, 8, 1, 24, 24, 9]),   # 128 x 128
    (300, 64, 6976, 3, 40, [40, 11, 33]),              # 64 x 128
    (257, 192, 320, 5, 8, [8, 8, 5, 8, 8]),            # 64 x 64
    (257, 64, 64, 1, 128, [77]),
    (321, 512, 192, 256, 8, None),                     # four bitmap words
    (700, 4160, 128, 2, 64, [64, 41]),                 # K slices of unequal length
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_K%d_N%d_ad%d_r%d" % c[:5])
@pytest.mark.parametrize("residual", [False, True], ids=["", "res"])
def test_tiles_against_float64(case, residual):
    T, K, N, n_ad, r_max, ranks = case
    say("lora tiles", case, residual)
    g = torch.Generator().manual_seed(T + N)
    ranks = ranks or [r_max] * n_ad
    x = torch.randn(T, K, generator=g).bfloat16()
    W = (torch.randn(N, K, generator=g) * 0.02).bfloat16()
    A = torch.full((n_ad, r_max, K), float("nan")).bfloat16()
    B = torch.full((n_ad, N, r_max), float("nan")).bfloat16()
    # runs of tokens of one adapter, some with none; the last adapter unused
    idx = torch.randint(-1, max(n_ad - 1, 1), (T // 7 + 1,), generator=g).repeat_interleave(7)[:T]
    for a, r in enumerate(ranks):
        if a < n_ad - 1 or n_ad == 1:
            A[a, :r] = (torch.randn(r, K, generator=g) * r ** -0.5).bfloat16()
            B[a, :, :r] = (torch.randn(N, r, generator=g) * 0.01).bfloat16()
    idx[::50] = n_ad + 1  # out of range: no adapter
    idx = idx.int()
    scale = torch.rand(T, generator=g) + 0.5
    res = torch.randn(T, N, generator=g).bfloat16() if residual else None
    y = lk.local_lora_linear(x.cuda(), W.cuda(), A.cuda(), B.cuda(),
                             torch.tensor(ranks, dtype=torch.int32).cuda(), idx.cuda(),
                             scale.cuda(), residual=None if res is None else res.cuda())
    torch.cuda.synchronize()

    ref = x.double() @ W.double().t()
    terms = x.double().abs() @ W.double().abs().t()
    delta = torch.zeros_like(ref)
    if residual:
        ref += res.double()
        terms += res.double().abs()
    for a, r in enumerate(ranks):
        t = (idx == a).nonzero().view(-1)
        if t.numel():
            s = scale[t].double()[:, None]
            u = s * (x[t].double() @ A[a, :r].double().t())
            ua = s * (x[t].double().abs() @ A[a, :r].double().abs().t())
            b = B[a, :, :r].double().t()
            ref[t] += u @ b
            delta[t] = u.abs() @ b.abs()
            terms[t] += ua @ b.abs()
    bound = 2.0 ** -8 * (ref.abs() + delta) + (K + r_max + 4) * 2.0 ** -24 * terms
    assert torch.all((y.cpu().double() - ref).abs() <= 1.01 * bound)
