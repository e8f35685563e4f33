"""The adapter gradients at the edges of their tiles: 16-token shrink tiles,
64-token units, adapters of one unit and of several, spans of 2048 tokens, column
tiles that end inside a wave, ranks on both sides of every rank tile, K slices of
a wave that are empty, and values that are not finite.

Against plain float64. The bound is that of float32 sums: a gradient entry is
a sum of at most T products with u (or dy B), itself a sum of at most D = K or
N products, so its error is at most (T + D + 8) 2^-24 times the sum of the
absolute values of all products."""
import numpy as np
import pytest
import torch

import paper_2608_15241_amd as lk
from tests.gpu_helpers import dev, say

pytestmark = pytest.mark.gpu


def _inputs(T, K, N, n_ad, r_max, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(T, K, generator=g).bfloat16()
    dy = torch.randn(T, N, generator=g).bfloat16()
    A = (torch.randn(n_ad, r_max, K, generator=g) * r_max ** -0.5).bfloat16()
    B = (torch.randn(n_ad, N, r_max, generator=g) * 0.01).bfloat16()
    idx = torch.randint(-1, n_ad, (T,), generator=g, dtype=torch.int32)
    ranks = torch.tensor([max(1, r_max - 3 * a) for a in range(n_ad)], dtype=torch.int32)
    scale = torch.rand(T, generator=g) + 0.5
    return x, dy, A, B, ranks, idx, scale


def _run(x, dy, A, B, ranks, idx, scale):
    c = [t.cuda() for t in (x, dy, A, B)]
    dA, dB = lk.local_lora_grad(*c, ranks.cuda(), idx.cuda(), scale.cuda())
    torch.cuda.synchronize()
    return dA.cpu(), dB.cpu()


def _reference(x, dy, A, B, ranks, idx, scale, cast):
    """Gradients in the type `cast` gives, zero past the ranks."""
    dA, dB = cast(torch.zeros(A.shape)), cast(torch.zeros(B.shape))
    for a, r in enumerate(ranks.tolist()):
        t = (idx == a).nonzero().view(-1)
        if t.numel():
            u = cast(x[t]) @ cast(A[a, :r]).t()
            g = cast(dy[t]) @ cast(B[a, :, :r])
            s = cast(scale[t])[:, None]
            dB[a, :, :r] = cast(dy[t]).t() @ (s * u)
            dA[a, :r] = (s * g).t() @ cast(x[t])
    return dA, dB


CASES = [(1, 64, 64, 1, 8), (15, 64, 192, 2, 16), (16, 128, 64, 1, 24), (17, 192, 128, 3, 32),
         (63, 320, 64, 1, 40), (64, 256, 64, 64, 8), (65, 256, 192, 1, 64), (257, 128, 256, 1, 72),
         (300, 192, 320, 9, 128), (700, 64, 128, 3, 16), (1030, 128, 64, 1, 16),
         (4030, 64, 128, 1, 8), (4200, 192, 64, 1, 24), (6700, 64, 64, 2, 72)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "T%d_K%d_N%d_ad%d_r%d" % c)
def test_edges_against_float64(case):
    say("grad products", case)
    T, K, N, n_ad, r_max = case
    inp = _inputs(T, K, N, n_ad, r_max, T + K)
    got = _run(*inp)
    ref = _reference(*inp, cast=lambda t: t.double())
    mag = _reference(*inp, cast=lambda t: t.double().abs())
    for g, r, m, D in zip(got, ref, mag, (N, K)):
        assert torch.all((g.double() - r).abs() <= (T + D + 8) * 2.0 ** -24 * m)


@pytest.mark.parametrize("T", [1, 64, 65, 128, 2048, 2049, 4100])
def test_size_of_the_bank_does_not_matter(T):
    # one adapter's tokens, alone and in a bank of 70: the same bits, zeros elsewhere
    say("grad products, one adapter of a bank", T)
    x, dy, A, B, ranks, idx, scale = _inputs(T, 128, 64, 70, 16, T)
    idx[:] = 33
    dA, dB = _run(x, dy, A, B, ranks, idx, scale)
    one = slice(33, 34)
    dA1, dB1 = _run(x, dy, A[one], B[one], ranks[one], idx - 33, scale)
    assert torch.equal(dA[one], dA1) and torch.equal(dB[one], dB1)
    for d in (dA, dB):
        assert not d[:33].any() and not d[34:].any()


@pytest.mark.parametrize("where", ["x", "dy", "scale"])
def test_values_that_are_not_finite(where):
    # an infinity or NaN reaches the entries that float32 products give it to,
    # as what they give, and no others
    say("grad products, not finite:", where)
    x, dy, A, B, ranks, idx, scale = _inputs(150, 128, 192, 3, 16, 5)
    idx[:] = torch.arange(150) % 3
    if where == "scale":
        scale[7] = float("inf")
    else:
        t = {"x": x, "dy": dy}[where]
        t[4, 5], t[70, 100], t[11, 0] = float("inf"), float("-inf"), float("nan")
    inp = (x, dy, A, B, ranks, idx, scale)
    for g, r in zip(_run(*inp), _reference(*inp, cast=lambda t: t.float())):
        assert torch.equal(g.isnan(), r.isnan())
        assert torch.equal(g.isinf(), r.isinf())
        assert torch.equal(g[g.isinf()] > 0, r[r.isinf()] > 0)


@pytest.mark.parametrize("T", [1, 70])
@pytest.mark.parametrize("s,x_std,dy_std", [(1e-34, 1.0, 1.0), (1e-36, 1.0, 1.0),
                                            (1e10, 1.0, 1e-39), (1e10, 1e-39, 1.0)],
                         ids=["s1e-34", "s1e-36", "dy1e-39", "x1e-39"])
def test_values_near_the_smallest(T, s, x_std, dy_std):
    # coefficients whose low parts, and rows whose values, are below the smallest
    # normal number (2^-126): no product may lose them. Every intermediate may be
    # off by half the smallest float32 (2^-150) besides, times its partner.
    say("grad products, small values", T, s, x_std, dy_std)
    x, dy, A, B, ranks, idx, scale = _inputs(T, 64, 64, 2, 16, 31)
    idx = torch.arange(T, dtype=torch.int32) % 2
    x, dy = (x.double() * x_std).bfloat16(), (dy.double() * dy_std).bfloat16()
    inp = (x, dy, A, B, ranks, idx, scale * s)
    got = _run(*inp)
    ref = _reference(*inp, cast=lambda t: t.double())
    mag = _reference(*inp, cast=lambda t: t.double().abs())
    for g, r, m, v in zip(got, ref, mag, (x, dy)):
        small = (T + 72) * 2.0 ** -149 * (1 + max(s, 1.0) * float(v.double().abs().max())) \
            * (1 + 8.0 * T)
        assert torch.all((g.double() - r).abs() <= (T + 72) * 2.0 ** -24 * m + small)
