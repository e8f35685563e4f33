"""Key ranges of the prefill attention: they are shorter in calls of few tiles, so
such calls are compared with the oracle at the lengths where a tile starts to take
two, three and four ranges, on both sides of every limit."""
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
    # Hq, Hkv, D, prefixes, chunks, units, split tiles
    # 32 (tile, head) pairs or fewer (64 at D = 64), the longest tile above 19: 2, 3, 4
    # ranges above 16, 32, 48 blocks
    (4, 1, 64, [239, 241, 288], [16, 16, 16], 3, 0),            # 16, 17, 19
    (4, 1, 64, [239, 241, 289], [16, 16, 16], 5, 2),            # 16, 17, 20
    (4, 4, 128, [496, 497, 752, 1000], [16, 16, 16, 40], 12, 4),  # 32, 33, 48, 65
    (2, 2, 64, [4000], [1], 4, 1),                              # one row, four ranges
    # up to 64, the longest above 38
    (8, 2, 128, [0, 3], [700, 129], 14, 4),                     # 8, 16 .. 40, 44 | 9, 9
    (32, 8, 128, [592, 256], [16, 16], 2, 0),                   # 38, 17
    (32, 8, 128, [593, 752], [16, 16], 6, 2),                   # 39, 48
    # up to 128, the longest above 50
    (32, 8, 128, [784, 250, 10, 10], [16] * 4, 4, 0),           # 50, 17
    (32, 8, 128, [785, 250, 768, 10], [28, 6, 22, 12], 10, 2),  # 51, 16, 50
    # up to 160, the longest above 48 and not above 288: 2 and 3 above 32 and 64
    (32, 8, 128, [752, 600, 10, 10, 10], [16] * 5, 5, 0),       # 48, 39
    (32, 8, 128, [753, 496, 1009, 10, 10], [16] * 5, 8, 2),     # 49, 32, 65
    (32, 8, 128, [4593, 496, 1009, 10, 10], [16] * 5, 8, 1),    # 289, 32, 65
    # up to 192, the longest above 64 and not above 96: 2 above 48
    (32, 8, 128, [1008, 760, 753, 5, 10, 30], [16] * 6, 6, 0),  # 64, 49, 49
    (32, 8, 128, [1024, 752, 753, 1520, 10, 30], [16] * 6, 9, 3),  # 65, 48, 49, 96
    (32, 8, 128, [1024, 752, 753, 1521, 10, 30], [16] * 6, 7, 1),  # 65, 48, 49, 97
    # more: 2, 3, 4 above 96, 192, 288
    (32, 8, 128, [700, 1500, 90, 300, 2900, 0], [30, 128, 129, 257, 61, 20], 11, 2),
    (32, 32, 64, [1000] * 8, [150] * 8, 16, 0),                 # 71, 72
    (32, 8, 128, [224] * 12, [128] * 12, 12, 0),                # many short tiles
    (32, 8, 128, [0, 0], [400, 400], 8, 0),                     # two short prompts
]


class _Buffer:
    """A workspace that keeps what the call left in it."""

    def get(self, nbytes):
        self.buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        return self.buf


def _plan(buf, T, B, Hq, D):
    """The planner's counts of units and of split tiles, which the workspace holds
    after the partial results (whole tiles of 128 rows, four ranges each)."""
    parts = (T // 128 + B) * Hq * 4 * 128 * (D + 2) * 4
    at = (parts + 255) // 256 * 256
    return tuple(buf[at:at + 8].view(torch.int32).tolist())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%d_%d_%d_%d_%d" % (*c[:3], len(c[3]), sum(c[3])))
@pytest.mark.parametrize("stale", [0.0, 0.9])
def test_key_ranges(case, stale):
    Hq, Hkv, D, prefix, chunk = case[:5]
    say("prefill key ranges", case, stale)
    rng = np.random.default_rng(Hq + D + len(prefix))
    c = _prefill_case(rng, prefix, chunk, Hq, Hkv, D, stale)
    kc_d, vc_d = dev_u16(c["kc"]), dev_u16(c["vc"])
    ws = _Buffer()
    out, lse = lk.local_paged_attn_prefill(
        dev_u16(c["q"]), dev(c["qi"]), kc_d, vc_d, dev(c["table"]), dev(c["ctx"]),
        dev(c["bv"]), dev(c["rv"]), 1.0 / math.sqrt(D), k_new=dev_u16(c["kn"]),
        v_new=dev_u16(c["vn"]), Hkv=Hkv, workspace=ws)
    torch.cuda.synchronize()
    assert _plan(ws.buf, sum(chunk), len(chunk), Hq, D) == case[5:]
    kc, vc = c["kc"].copy(), c["vc"].copy()
    oracle.kv_append(kc, vc, Hkv, D, c["table"], c["qi"], c["ctx"], c["kn"], c["vn"])
    ro, rl = oracle.paged_attn(c["q"], c["qi"], Hq, Hkv, D, kc, vc, c["table"], c["ctx"],
                               c["bv"], c["rv"], 1.0 / math.sqrt(D))
    assert np.array_equal(host_u16(kc_d), kc) and np.array_equal(host_u16(vc_d), vc)
    assert_attn(f64(out), ro, "out", D)
    assert_lse(lse.cpu().numpy(), rl, "lse")
