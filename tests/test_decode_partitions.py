"""Partitions of the decode attention: their length and the waves that share one
follow the size of the call, so every form is compared with the oracle, and the
workspace never grows when a call gets smaller."""
import ctypes
import math
import os

import numpy as np
import pytest
import torch

import paper_2608_15241_amd as lk
from tests.gpu_helpers import assert_attn, assert_lse, dev, dev_u16, f64, host_u16, say
from tests.test_gpu_attention import _decode_case, _oracle_decode, _run_decode

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = ctypes.c_void_p(0x1000)


@pytest.mark.parametrize("checked", [False, True])
@pytest.mark.parametrize("hkv,group", [(1, 1), (4, 1), (32, 1), (8, 4), (1, 16)])
def test_workspace_does_not_grow_when_a_call_shrinks(hkv, group, checked):
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2608_15241_amd", "liblocal.so"))
    f = lib.local_paged_attn_decode_checked if checked else lib.local_paged_attn_decode
    more = [FAKE, ctypes.c_int64(8), FAKE, FAKE] if checked else []

    def size(B, mb):
        n = ctypes.c_size_t(0)
        assert f(FAKE, B, hkv * group, hkv, 128, FAKE, FAKE, FAKE, FAKE, ctypes.c_int64(100000),
                 16, FAKE, mb, FAKE, FAKE, FAKE, ctypes.c_float(0.1), FAKE, FAKE, *more, None,
                 ctypes.byref(n), None) == 0
        return n.value

    for mb in (1, 31, 64, 255, 256, 257, 300, 384, 500, 512, 513, 900, 1024, 1025, 1500, 4000):
        sizes = [size(B, mb) for B in range(1, 130)]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), mb
        longest = 32 if mb <= 256 else 48 if mb <= 512 else 64
        for B, n in enumerate(sizes, 1):  # at least what the longest partitions take
            assert n >= B * hkv * group * -(-mb // longest) * (128 + 2) * 4


def _longest_parts(mb):
    return -(-mb // (32 if mb <= 256 else 48 if mb <= 512 else 64))


def _least_workspace(B, Hq, mb, D, checked):
    """What local.h promises to accept."""
    up = lambda v: (v + 255) // 256 * 256
    n = max(B, 1) * Hq * _longest_parts(mb) * (D + 2) * 4
    units = max(B, 1) * _longest_parts(mb)
    return up(n) + up(8 * units) + up(4 * units) if checked else n


@pytest.mark.parametrize("checked", [False, True])
@pytest.mark.parametrize("B,hkv,group,D,mb", [
    (0, 8, 4, 128, 64), (1, 1, 1, 64, 1), (1, 32, 1, 128, 16), (1, 8, 4, 128, 1024),
    (4, 8, 4, 128, 257), (5, 8, 1, 128, 512), (23, 32, 1, 128, 32), (64, 8, 4, 128, 256)])
def test_smallest_workspace_is_accepted(B, hkv, group, D, mb, checked):
    # the size without short partitions, as callers computed it before those came;
    # q NULL: an accepted workspace shows as LOCAL_ERR_NULL, before any launch
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2608_15241_amd", "liblocal.so"))
    f = lib.local_paged_attn_decode_checked if checked else lib.local_paged_attn_decode
    more = [FAKE, ctypes.c_int64(8), None if B == 0 else FAKE, FAKE] if checked else []

    def status(ws_bytes):
        n = ctypes.c_size_t(ws_bytes)
        return f(None, B, hkv * group, hkv, D, FAKE, FAKE, FAKE, FAKE, ctypes.c_int64(100000), 16,
                 FAKE, mb, FAKE, FAKE, FAKE, ctypes.c_float(0.1), FAKE, FAKE, *more, FAKE,
                 ctypes.byref(n), None)

    least = _least_workspace(B, hkv * group, mb, D, checked)
    accepted = 0 if B == 0 and not checked else 1  # LOCAL_OK (nothing to do) or LOCAL_ERR_NULL
    assert status(least) == accepted
    assert status(least - 1) == 4  # LOCAL_ERR_WORKSPACE


# (batch, Hq, Hkv, D, longest context, table width or None, blocks of a partition, waves)
CASES = [
    (1, 4, 4, 64, 1, None, 16, 4),        # one block
    (3, 32, 8, 128, 256, None, 16, 4),    # one partition of 16 blocks, full
    (4, 32, 8, 128, 4100, None, 16, 4),   # 257-block table: 48 -> 16 blocks
    (5, 8, 8, 128, 8192, None, 16, 1),    # 512-block table, one query head per KV head
    (2, 32, 8, 128, 16384, None, 32, 4),  # 64 -> 32 blocks
    (1, 16, 1, 64, 9000, None, 32, 4),    # 16 query heads per KV head (the largest merge)
    (11, 32, 32, 128, 500, None, 16, 2),  # 704 units
    (12, 32, 32, 128, 500, None, 16, 1),  # 768 units
    (20, 32, 32, 128, 60, 16, 16, 2),     # two waves, most of them without a block
    (24, 32, 32, 128, 700, None, 32, 1),
    (50, 32, 32, 128, 60, 64, 32, 1),     # partitions mostly without a block
    (40, 32, 32, 128, 300, 64, 32, 1),    # one query head per KV head: no pairs of waves
    (24, 32, 8, 128, 3000, 256, 32, 2),   # grouped heads, 1536 units: pairs
    (40, 32, 8, 128, 400, 256, 32, 2),    # ... 2560, most partitions not there
    (41, 32, 8, 128, 400, 256, 32, 1),    # ... 2624
    (65, 12, 4, 64, 1500, None, 32, 1),   # ranked over two registers of requests
    (130, 8, 4, 64, 1100, None, 32, 2),   # ... three, two waves
    (520, 1, 1, 64, 90, None, 16, 2),     # too many requests to rank
]


@pytest.mark.parametrize("B,Hq,Hkv,D,longest,width,blocks,waves", CASES)
def test_decode_forms_are_the_named_ones(B, Hq, Hkv, D, longest, width, blocks, waves):
    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2608_15241_amd", "liblocal.so"))
    form = lib.localk_decode_form(B, Hq, Hkv, width or -(-longest // 16))
    assert (form % 256, form // 256) == (blocks, waves)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,D,longest,width", [c[:6] for c in CASES])
def test_decode_partition_forms(B, Hq, Hkv, D, longest, width):
    say("decode partitions", B, Hq, Hkv, D, longest, width)
    rng = np.random.default_rng(B * 1000 + longest)
    ctx = rng.integers(0 if B > 2 else 1, longest + 1, size=B)
    ctx[0] = longest
    if B > 4:
        ctx[1], ctx[2], ctx[3] = min(longest, 256), min(longest, 257), min(longest, 255)
    c = _decode_case(rng, ctx, Hq, Hkv, D, stale_frac=0.3, max_blocks=width)
    out, lse, k, v = _run_decode(c)
    ro, rl, rk, rv = _oracle_decode(c)
    assert_attn(f64(out), ro, "out", D)
    assert_lse(lse.cpu().numpy(), rl, "lse")
    assert np.array_equal(host_u16(k), rk) and np.array_equal(host_u16(v), rv)


@pytest.mark.gpu
@pytest.mark.parametrize("checked", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,D,longest", [(2, 32, 8, 128, 5000), (5, 8, 8, 64, 900)])
def test_smallest_workspace(B, Hq, Hkv, D, longest, checked):
    # the longest partitions in exactly their partials, and not a byte past them
    say("decode smallest workspace", B, Hq, Hkv, D, longest, checked)
    rng = np.random.default_rng(B + longest)
    ctx = rng.integers(1, longest + 1, size=B)
    ctx[0] = longest
    c = _decode_case(rng, ctx, Hq, Hkv, D, stale_frac=0.3)
    least = _least_workspace(B, Hq, c["table"].shape[1], D, checked)
    guarded = torch.full((least + 4096,), 0x5A, dtype=torch.uint8, device="cuda")

    class Least:
        def get(self, nbytes):
            assert nbytes > least  # the call would rather have short partitions
            return guarded[:least]

    kc, vc = dev_u16(c["kc"]), dev_u16(c["vc"])
    fn = lk.local_paged_attn_decode_checked if checked else lk.local_paged_attn_decode
    res = fn(dev_u16(c["q"]), kc, vc, dev(c["table"]), dev(c["ctx"]), dev(c["bv"]), dev(c["rv"]),
             1.0 / math.sqrt(D), k_new=dev_u16(c["kn"]), v_new=dev_u16(c["vn"]), Hkv=Hkv,
             workspace=Least())
    torch.cuda.synchronize()
    ro, rl, rk, rv = _oracle_decode(c)
    assert_attn(f64(res[0]), ro, "out", D)
    assert_lse(res[1].cpu().numpy(), rl, "lse")
    assert np.array_equal(host_u16(kc), rk) and np.array_equal(host_u16(vc), rv)
    if checked:
        stale = [(b, j) for b in range(B) for j in range(-(-int(ctx[b]) // 16))
                 if c["bv"][c["table"][b, j]] != c["rv"][b]]
        assert int(res[3].item()) == len(stale)
        assert res[2][:len(stale)].cpu().tolist() == [list(p) for p in stale]
    assert torch.all(guarded[least:] == 0x5A)
