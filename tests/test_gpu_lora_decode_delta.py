"""Decode-size projections: the adapters' deltas at the edges of the 16-token
tiles, of the 32-column steps and of a batch of 16 of them, with NaN past every
rank, in an unused adapter and in one adapter in use, which may reach no token
of another.

Against plain float64. y is rounded once (2^-8 of it: bf16 keeps 8 bits), U_s is
rounded to bf16 before the up-projection (2^-8 of every product with it), and
every sum is float32: of K products, of K products inside U_s and of r products
(2^-24 of the absolute values' sum each)."""
import pytest
import torch

import paper_2608_15241_amd as lk
from tests.gpu_helpers import say

pytestmark = pytest.mark.gpu

CASES = [
    # T, K, N, n_ad, r_max, ranks
    (1, 64, 64, 1, 8, [8]),
    (3, 192, 128, 4, 16, [16, 0, 5, 16]),
    (15, 256, 192, 17, 24, None),
    (16, 128, 320, 20, 64, None),                           # 16 adapters of 2 steps in a tile
    (17, 64, 128, 3, 40, [33, 40, 32]),
    (33, 256, 6144, 5, 128, [128, 97, 96, 1, 128]),
    (64, 4160, 192, 16, 64, [8, 16, 32, 64] * 4),
    (65, 64, 576, 70, 128, [128] * 70),                     # 64 steps in a tile
    (129, 128, 64, 12, 16, None),
    (256, 512, 256, 256, 8, None),
    # 24 columns: a thread's own loads of B, as up to 16
    (1, 64, 64, 1, 24, [24]),
    (33, 128, 192, 5, 24, [24, 0, 17, 9, 24]),
    (256, 64, 320, 40, 24, None),
    # more than 64 tokens: tiles of 3, 6, 6 and 4 x 16 features, 1 to 4 extra row tiles
    (100, 128, 6144, 5, 16, None),
    (129, 128, 12288, 3, 16, None),
    (200, 192, 6144, 2, 8, [8, 5]),
    (256, 64, 8192, 40, 64, None),
    (70, 128, 6144, 64, 96, None),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_K%d_N%d_ad%d_r%d" % c[:5])
@pytest.mark.parametrize("residual", [False, True], ids=["", "res"])
def test_decode_deltas_against_float64(case, residual):
    T, K, N, n_ad, r_max, ranks = case
    say("lora decode delta", case, residual)
    g = torch.Generator().manual_seed(T + N)
    ranks = ranks or [r_max] * n_ad
    x = torch.randn(T, K, generator=g).bfloat16()
    W = (torch.randn(N, K, generator=g) * 0.02).bfloat16()
    A = torch.full((n_ad, r_max, K), float("nan")).bfloat16()
    B = torch.full((n_ad, N, r_max), float("nan")).bfloat16()
    idx = torch.randint(-1, max(n_ad - 1, 1), (T,), generator=g)  # the last adapter unused
    bad = int(idx[T // 2]) if T > 8 and n_ad > 2 else -1           # in use, all NaN
    for a, r in enumerate(ranks):
        if (a < n_ad - 1 or n_ad == 1) and a != bad:
            A[a, :r] = (torch.randn(r, K, generator=g) * max(r, 1) ** -0.5).bfloat16()
            B[a, :, :r] = (torch.randn(N, r, generator=g) * 0.01).bfloat16()
    idx[1::50] = n_ad + 1  # out of range: no adapter
    scale = torch.rand(T, generator=g) + 0.5
    res = torch.randn(T, N, generator=g).bfloat16() if residual else None
    y = lk.local_lora_linear(x.cuda(), W.cuda(), A.cuda(), B.cuda(),
                             torch.tensor(ranks, dtype=torch.int32).cuda(), idx.int().cuda(),
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
        if t.numel() and a != bad:
            s = scale[t].double()[:, None]
            u = s * (x[t].double() @ A[a, :r].double().t())
            ua = s * (x[t].double().abs() @ A[a, :r].double().abs().t())
            b = B[a, :, :r].double().t()
            ref[t] += u @ b
            delta[t] = u.abs() @ b.abs()
            terms[t] += ua @ b.abs()
    bound = 2.0 ** -8 * (ref.abs() + delta) + (K + r_max + 4) * 2.0 ** -24 * terms
    y = y.cpu().double()
    fine = (idx != bad) | (bad < 0)
    assert torch.all((y - ref).abs()[fine] <= 1.01 * bound[fine])
    if bad >= 0 and ranks[bad] > 0:
        assert torch.all(torch.isnan(y[idx == bad]))
