"""Spike selection at its edges: groups of one sign with ties (the position rule turns round there), zeros of both signs, the largest
magnitudes and infinities (the integer form of the selection), mixed into ordinary groups of the same wave; every byte of
the record against the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2508_03760_amd import fcv2
from paper_2508_03760_amd import workloads as W

pytestmark = pytest.mark.gpu

SR, INT = fcv2.F_SPIKE, fcv2.F_META_INT


def _groups(kind, ngroups, group, rng):
    z = rng.standard_normal((ngroups, group)).astype(np.float32)
    if kind == "positive ties":
        z = np.round(np.abs(z) * 2) / 2
    elif kind == "negative ties":
        z = -np.round(np.abs(z) * 2) / 2 - 0.5
    elif kind == "zeros of both signs":
        z = np.where(rng.random(z.shape) < 0.5, np.float32(0.0), np.float32(-0.0)) * np.sign(np.abs(z))
        z[::3] = np.maximum(rng.standard_normal(z[::3].shape), 0)
    elif kind == "constant":
        z[:] = rng.choice([-2.0, -0.0, 0.0, 3.0], size=(ngroups, 1))
    elif kind == "largest":
        z *= np.float32(2.0**120)
        z[:, 3] = 3.0e38
    elif kind == "infinite":
        z[:, group // 2] = np.inf
        z[1::2, 1] = -np.inf
    return z


@pytest.mark.parametrize("kind", ["positive ties", "negative ties", "zeros of both signs", "constant", "largest", "infinite"])
@pytest.mark.parametrize("group", [32, 64, 128, 256])
def test_selection_edges(kind, group):
    rng = np.random.default_rng(7)
    per = 2048 // group  # groups of a wave
    special, plain = _groups(kind, 3 * per + 1, group, rng), rng.standard_normal((3 * per + 1, group)).astype(np.float32)
    mixed = np.concatenate([special, np.where(rng.random((len(plain), 1)) < 0.2, special, plain)])
    x = W.f32_to_bf16_bits(mixed.astype(np.float32)).reshape(-1)
    xd = torch.from_numpy(x.view(np.int16)).to("cuda").view(torch.bfloat16)
    for bits, flags in ((3, SR), (5, 0), (4, SR | INT), (8, SR)):
        got = fcv2.quantize_pack(xd, bits, group, flags).cpu().numpy()
        want = O.quantize_pack(x, bits, group, flags)
        L = O.get_layout(x.size, bits, group, flags)
        assert got.size == L.total_bytes and np.array_equal(got, want), f"{kind} b{bits} g{group} f{flags}"
