"""The reduction of small payloads (a block's waves take a peer each) at the edges of its tiles and of the rule that chooses it."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_03760_amd import fcv2
from paper_2508_03760_amd import workloads as W

pytestmark = pytest.mark.gpu

SR, F32, INT, IDX16 = fcv2.F_SPIKE, fcv2.F_META_FP32, fcv2.F_META_INT, fcv2.F_IDX_BF16
DEV = "cuda:0"


def check(xs, n, fmt):
    recs = [O.quantize_pack(x, *fmt) for x in xs]
    want, want_sum = O.reduce_requant(recs, n, fmt, want_sum=True)
    dev = [torch.from_numpy(r.copy()).to(DEV) for r in recs]
    got, got_sum = fcv2.reduce_requant(dev, n, fmt, want_sum=True)
    assert np.array_equal(got.cpu().numpy(), want)
    assert np.array_equal(got_sum.cpu().numpy().view(np.uint32), want_sum.view(np.uint32))
    assert torch.equal(fcv2.reduce_requant(dev, n, fmt), got)


@pytest.mark.parametrize("bits,group,flags", [(2, 32, SR | INT), (3, 128, SR), (4, 64, 0), (5, 256, SR), (6, 32, SR | F32), (7, 128, SR | IDX16),
                                              (8, 256, SR), (8, 32, INT)])
@pytest.mark.parametrize("peers", [1, 2, 3, 8, 9])  # 2 to 8 take the small kernel
@pytest.mark.parametrize("n", [256, 768, 1024, 1280, 5 * 1024 + 256])  # tiles have 1024 elements
def test_tiles_and_peers(bits, group, flags, peers, n):
    check([W.tensor(2, p, rows=1, cols=n).reshape(-1) for p in range(peers)], n, (bits, group, flags))


@pytest.mark.parametrize("n,group,flags", [(32, 32, SR), (1024 + 32, 32, SR | INT), (1 << 20, 64, SR), ((1 << 20) + 64, 64, SR),
                                           (1 << 19, 128, 0), ((1 << 19) + 128, 128, 0)])
def test_ends_of_the_range(n, group, flags):
    check([W.tensor(2, p, rows=1, cols=n).reshape(-1) for p in range(4)], n, (3, group, flags))


@pytest.mark.parametrize("bits,group", [(2, 32), (5, 128), (8, 64)])
def test_scales_beyond_the_fast_decoding(bits, group):
    n = 2048
    rng = np.random.default_rng(bits)
    xs = []
    for p in range(5):
        v = rng.standard_normal(n).astype(np.float32) * np.float32(2.0) ** np.where(np.arange(n) // group % 3 == p % 3, 118, 3).astype(np.float32)
        xs.append((v.view(np.uint32) >> 16).astype(np.uint16))
    check(xs, n, (bits, group, SR))
