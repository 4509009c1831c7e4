"""Results that a call allocates itself: every byte defined, as if the memory had been cleared before (padding zero, rows of
the send buffer that no copy takes zero, row_src past the copies -1), on memory that held other values."""
import numpy as np
import pytest
import torch

from paper_2508_03760_amd import fcv2
from paper_2508_03760_amd import workloads as W

pytestmark = pytest.mark.gpu

SR, F32, INT, IDX16 = fcv2.F_SPIKE, fcv2.F_META_FP32, fcv2.F_META_INT, fcv2.F_IDX_BF16
DEV = "cuda:0"


def _bf16(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).to(DEV).view(torch.bfloat16)


def _soil(*sizes):
    """Leaves blocks of these sizes, full of ones, to the allocator: the next allocations of the sizes get them."""
    held = [torch.full((s,), 0xFF, dtype=torch.uint8, device=DEV) for s in sizes]
    torch.cuda.synchronize()
    del held


@pytest.mark.parametrize("bits,group,flags", [(2, 32, SR | INT), (3, 128, SR), (4, 256, 0), (5, 64, SR | F32), (6, 32, INT), (7, 128, SR | IDX16),
                                              (8, 64, SR | INT | IDX16)])
@pytest.mark.parametrize("ngroups", [1, 3, 77])
def test_records_have_zero_padding(bits, group, flags, ngroups):
    n = group * ngroups
    size = fcv2.get_layout(n, bits, group, flags).total_bytes
    xs = [_bf16(W.tensor(2, p, rows=1, cols=n).reshape(-1)) for p in range(3)]
    want = [fcv2.quantize_pack(x, bits, group, flags, out=torch.zeros(size, dtype=torch.uint8, device=DEV)) for x in xs]
    _soil(size)
    assert torch.equal(fcv2.quantize_pack(xs[0], bits, group, flags), want[0])
    for fmt in ((bits, group, flags), (8 if bits < 8 else 3, group, flags)):
        size_out = fcv2.get_layout(n, *fmt).total_bytes
        kept = fcv2.reduce_requant(want, n, (bits, group, flags), fmt, out=torch.zeros(size_out, dtype=torch.uint8, device=DEV))
        _soil(size_out)
        assert torch.equal(fcv2.reduce_requant(want, n, (bits, group, flags), fmt), kept)
    k, m = 3, 2048 * ngroups
    x = _bf16(W.tensor(2, 5, rows=k, cols=m))
    size = fcv2.get_layout(m, bits, group, flags).total_bytes
    kept = fcv2.quantize_pack_slices(x, k, bits, group, flags, out=torch.zeros((k, size), dtype=torch.uint8, device=DEV))
    _soil(k * size)
    assert torch.equal(fcv2.quantize_pack_slices(x, k, bits, group, flags), kept)


@pytest.mark.parametrize("T,H,K,E,bits,group,flags", [(1, 128, 1, 4, 3, 128, SR), (37, 2560, 6, 64, 4, 32, SR), (301, 768, 4, 300, 8, 256, 0),
                                                      (5, 32768, 3, 7, 5, 64, SR | INT)])
@pytest.mark.parametrize("dropped", [0.0, 0.3, 1.0])
def test_dispatch_defines_rows_past_the_copies(T, H, K, E, bits, group, flags, dropped):
    x = _bf16(W.tensor(3, 1, rows=T, cols=H))
    ids = torch.from_numpy(W.topk_routing(W.seed_for(3) + 21, T, E, K)).to(DEV)
    ids[torch.rand(ids.shape, generator=torch.Generator().manual_seed(4)).to(DEV) < dropped] = -1
    size = fcv2.get_layout(H, bits, group, flags, fcv2.ROW_ALIGN).total_bytes
    want = fcv2.dispatch_quant(x, ids, E, bits, group, flags, send_buf=torch.zeros((T * K, size), dtype=torch.uint8, device=DEV),
                               row_src=torch.full((T * K,), -1, dtype=torch.int32, device=DEV))
    _soil(T * K * size, T * K * 4, (E + 1) * 4)
    for got, w in zip(fcv2.dispatch_quant(x, ids, E, bits, group, flags), want):
        assert torch.equal(got, w)
