"""Partitions of the decode attention: their length and the waves that share one
follow the size of the call, so every form is compared with the oracle, and the
workspace never grows when a call gets smaller."""
import ctypes
import os

import numpy as np
import pytest

from tests.gpu_helpers import assert_attn, assert_lse, f64, host_u16, say
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


# (batch, Hq, Hkv, D, longest context, table width or None)
CASES = [
    (1, 4, 4, 64, 1, None),        # one block
    (3, 32, 8, 128, 256, None),    # one partition of 16 blocks, full
    (4, 32, 8, 128, 4100, None),   # 257-block table: 48 -> 16 blocks
    (5, 8, 8, 128, 8192, None),    # 512-block table, one query head per KV head
    (2, 32, 8, 128, 16384, None),  # 64 -> 32 blocks, four waves
    (1, 16, 1, 64, 9000, None),    # 16 query heads per KV head (the largest merge)
    (12, 32, 32, 128, 500, None),  # two waves
    (24, 32, 32, 128, 700, None),  # one wave, 32-block partitions
    (50, 32, 32, 128, 60, 64),     # two waves, most of them without a block
    (65, 12, 4, 64, 1500, None),   # ranked over two registers of requests
    (130, 8, 4, 64, 1100, None),   # ... three, two waves
    (520, 1, 1, 64, 90, None),     # too many requests to rank
]


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,D,longest,width", CASES)
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
