"""Long-chunk projections in every tile shape of the product, at the edges of
its tiles, of the 16-token shrink tiles and of the 64-column delta chunks, with
padding and unused adapters full of NaN.

Against plain float64. y is rounded once (2^-8 of it: bf16 keeps 8 bits), U_s is rounded to bf16
before the up-projection (2^-8 of every product with it), and every sum is
float32: of K products, of K products inside U_s and of r products (2^-24 of
the absolute values' sum each)."""
import ctypes
import os

import pytest
import torch

import paper_2608_15241_amd as lk
from tests.gpu_helpers import say

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MIXED = [24, 3, 17, 24, 8, 1, 24, 24, 9]

CASES = [
    # T, K, N, n_ad, r_max, ranks, the tile that the sizes select
    (2000, 64, (4032,), 4, 16, None, "128 x 256"),
    (1000, 128, (4032,), 9, 24, MIXED, "64 x 128"),
    (1000, 512, (4032,), 9, 24, MIXED, "128 x 128"),          # U_s from sums over K slices
    (900, 1024, (4096,), 40, 64, [64, 8, 33, 0, 41] * 8, "128 x 128"),
    (1000, 512, (1408, 1280, 1408), 9, 24, MIXED, "128 x 128"),  # bf16 U_s, three projections
    (1300, 1024, (12288,), 3, 16, None, "128 x 256"),         # several rounds
    (300, 64, (6976,), 3, 40, [40, 11, 33], "64 x 128"),
    (257, 192, (320,), 5, 8, [8, 8, 5, 8, 8], "64 x 64"),
    (257, 64, (64,), 1, 128, [77], "64 x 64"),
    (321, 512, (192,), 256, 8, None, "64 x 64"),              # 32 chunks of stacked columns
    (700, 4160, (128,), 2, 64, [64, 41], "64 x 64"),          # K slices of unequal length
]


# the choice alone: one round and several at a served width
MORE = [(1300, 4096, (12288,), 0, 0, None, "128 x 256"),
        (2048, 4096, (4096, 4096, 4096), 0, 0, None, "128 x 256"),
        (1000, 4096, (4096,), 0, 0, None, "128 x 128"),
        (1300, 4096, (4096, 1024, 1024), 0, 0, None, "64 x 128"),
        (300, 4096, (4096,), 0, 0, None, "64 x 128")]


@pytest.mark.parametrize("case", CASES + MORE,
                         ids=lambda c: "T%d_K%d_N%d" % (c[0], c[1], sum(c[2])))
def test_tiles_are_the_named_ones(case):
    T, K, Ns, tile = case[0], case[1], case[2], case[6]
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2608_15241_amd", "liblocal.so"))
    at = lib.localk_prefill_tile(ctypes.c_int64(T), ctypes.c_int64(K), len(Ns),
                                 (ctypes.c_int64 * len(Ns))(*Ns))
    assert ["128 x 256", "128 x 128", "64 x 128", "64 x 64"][at] == tile


@pytest.mark.gpu
@pytest.mark.parametrize("case,residual", [(c, r) for r in (False, True) for c in CASES
                                           if not r or len(c[2]) == 1],  # grouped: no residual
                         ids=lambda c: "" if c is False else "res" if c is True else
                         "T%d_K%d_N%d_ad%d_r%d" % (c[0], c[1], sum(c[2]), c[3], c[4]))
def test_tiles_against_float64(case, residual):
    T, K, Ns, n_ad, r_max, ranks = case[:6]
    say("lora tiles", case, residual)
    g = torch.Generator().manual_seed(T + sum(Ns))
    ranks = ranks or [r_max] * n_ad
    x = torch.randn(T, K, generator=g).bfloat16()
    # runs of tokens of one adapter, some with none; the last adapter unused
    idx = torch.randint(-1, max(n_ad - 1, 1), (T // 7 + 1,), generator=g).repeat_interleave(7)[:T]
    idx[::50] = n_ad + 1  # out of range: no adapter
    idx = idx.int()
    scale = torch.rand(T, generator=g) + 0.5
    res = torch.randn(T, Ns[0], generator=g).bfloat16() if residual else None
    Ws, As, Bs = [], [], []
    for N in Ns:
        Ws.append((torch.randn(N, K, generator=g) * 0.02).bfloat16())
        A = torch.full((n_ad, r_max, K), float("nan")).bfloat16()
        B = torch.full((n_ad, N, r_max), float("nan")).bfloat16()
        for a, r in enumerate(ranks):
            if a < n_ad - 1 or n_ad == 1:
                A[a, :r] = (torch.randn(r, K, generator=g) * max(r, 1) ** -0.5).bfloat16()
                B[a, :, :r] = (torch.randn(N, r, generator=g) * 0.01).bfloat16()
        As.append(A)
        Bs.append(B)
    rk = torch.tensor(ranks, dtype=torch.int32).cuda()
    cuda = lambda ts: [t.cuda() for t in ts]
    if len(Ns) > 1:
        ys = lk.local_lora_linear_grouped(x.cuda(), cuda(Ws), cuda(As), cuda(Bs), [rk] * len(Ns),
                                          idx.cuda(), scale.cuda())
    else:
        ys = [lk.local_lora_linear(x.cuda(), Ws[0].cuda(), As[0].cuda(), Bs[0].cuda(), rk,
                                   idx.cuda(), scale.cuda(),
                                   residual=None if res is None else res.cuda())]
    torch.cuda.synchronize()

    for y, W, A, B in zip(ys, Ws, As, Bs):
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


@pytest.mark.gpu
@pytest.mark.parametrize("T,n_ad", [(257, 1), (320, 3), (700, 70)])
def test_order_of_the_tokens_does_not_matter(T, n_ad):
    # the shrink gathers tokens of one adapter from groups of 64: runs of tokens and
    # the same tokens in any order give the same bits
    say("lora tiles, order of the tokens", T, n_ad)
    g = torch.Generator().manual_seed(T)
    K, N, r = 192, 128, 24
    x = torch.randn(T, K, generator=g).bfloat16()
    W = (torch.randn(N, K, generator=g) * 0.02).bfloat16()
    A = torch.randn(n_ad, r, K, generator=g).bfloat16()
    B = torch.randn(n_ad, N, r, generator=g).bfloat16()
    idx = torch.randint(-1, n_ad, (T,), generator=g).sort().values.int()
    scale = torch.rand(T, generator=g) + 0.5
    ranks = torch.tensor([r - a % 20 for a in range(n_ad)], dtype=torch.int32)
    rest = [t.cuda() for t in (W, A, B, ranks)]

    def run(order):
        return lk.local_lora_linear(x[order].cuda(), *rest, idx[order].cuda(),
                                    scale[order].cuda()).cpu()

    y = run(torch.arange(T))
    mixed = torch.randperm(T, generator=g)
    assert torch.equal(run(mixed).view(torch.int16), y[mixed].view(torch.int16))
