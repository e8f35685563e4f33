"""Key ranges of the prefill attention: their length follows the load of the whole
call, so calls of few tiles are compared with the oracle at the lengths where a tile
starts to take two, three and four ranges, and around one workgroup's mean load."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2608_15241_amd as lk
from tests.gpu_helpers import assert_attn, assert_lse, dev, dev_u16, f64, host_u16, say
from tests.test_gpu_attention import _prefill_case

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, D, prefixes, chunks
    (4, 1, 64, [239, 240, 241], [16, 16, 16]),              # 15 to 17 blocks: 1 or 2 ranges
    (4, 4, 128, [500, 512, 760, 1000], [12, 17, 9, 40]),    # 32, 34, 49, 65 blocks
    (8, 2, 128, [0, 3], [700, 129]),                        # tiles on the diagonal, split
    (2, 2, 64, [4000], [1]),                                # one row, four ranges
    (32, 8, 128, [700, 1500, 90, 300, 2900, 0], [30, 128, 129, 257, 61, 20]),  # mean load 16 to 64
    (32, 32, 64, [1000] * 8, [150] * 8),                    # mean load about 64
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%d_%d_%d_%d" % (c[0], c[1], c[2], len(c[3])))
@pytest.mark.parametrize("stale", [0.0, 0.9])
def test_key_ranges(case, stale):
    Hq, Hkv, D, prefix, chunk = case
    say("prefill key ranges", case, stale)
    rng = np.random.default_rng(Hq + D + len(prefix))
    c = _prefill_case(rng, prefix, chunk, Hq, Hkv, D, stale)
    kc_d, vc_d = dev_u16(c["kc"]), dev_u16(c["vc"])
    out, lse = lk.local_paged_attn_prefill(
        dev_u16(c["q"]), dev(c["qi"]), kc_d, vc_d, dev(c["table"]), dev(c["ctx"]),
        dev(c["bv"]), dev(c["rv"]), 1.0 / math.sqrt(D), k_new=dev_u16(c["kn"]),
        v_new=dev_u16(c["vn"]), Hkv=Hkv)
    torch.cuda.synchronize()
    kc, vc = c["kc"].copy(), c["vc"].copy()
    oracle.kv_append(kc, vc, Hkv, D, c["table"], c["qi"], c["ctx"], c["kn"], c["vn"])
    ro, rl = oracle.paged_attn(c["q"], c["qi"], Hq, Hkv, D, kc, vc, c["table"], c["ctx"],
                               c["bv"], c["rv"], 1.0 / math.sqrt(D))
    assert np.array_equal(host_u16(kc_d), kc) and np.array_equal(host_u16(vc_d), vc)
    assert_attn(f64(out), ro, "out", D)
    assert_lse(lse.cpu().numpy(), rl, "lse")
