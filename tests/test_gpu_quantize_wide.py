"""8-bit codes of tensors large enough to leave through LDS in whole lines: the last wave partly filled, slices, both sides of the rule."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_03760_amd import fcv2
from paper_2508_03760_amd import workloads as W

pytestmark = pytest.mark.gpu

SR, INT = fcv2.F_SPIKE, fcv2.F_META_INT


@pytest.mark.parametrize("n,slices,group,flags", [(1 << 22, 1, 128, SR), ((1 << 22) + 32, 1, 32, SR), ((1 << 22) + 2048 * 3 + 32 * 33, 1, 32, INT),
                                                  ((1 << 22) + 3 * 2048 * 4, 4, 64, SR | INT)])
def test_eight_bit_codes_of_large_tensors(n, slices, group, flags):
    x = W.tensor(2, 0, rows=1, cols=n).reshape(-1)
    xd = torch.from_numpy(x.view(np.int16)).to("cuda:0").view(torch.bfloat16)
    if slices == 1:
        got, want = fcv2.quantize_pack(xd, 8, group, flags).cpu().numpy(), O.quantize_pack(x, 8, group, flags)
    else:
        got = fcv2.quantize_pack_slices(xd, slices, 8, group, flags).cpu().numpy()
        want = np.stack([O.quantize_pack(p, 8, group, flags) for p in x.reshape(slices, -1)])
    assert np.array_equal(got, want)
