"""Spike selection at its edges: groups of one sign with ties (the position rule turns round there), zeros of both signs, the largest
magnitudes and infinities (the integer form of the selection), infinities in groups of one sign where no position stands below
them (the last element of a lane), mixed into ordinary groups of the same wave; every byte of the record against the oracle."""
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


def _one_sign(ngroups, group, epl, sign, value, rng):
    """Groups all >= +0 (sign 1) or all negative (sign -1), each with `value` * sign at the last element of a lane of epl elements; in half
    of the groups the same lane holds the extreme of the other side.  Every wave of the kernel that gives a lane epl
    elements sees its infinities there and nowhere else."""
    z = np.abs(rng.standard_normal((ngroups, group))).astype(np.float32) + np.float32(0.5)
    z[1::3] = np.round(z[1::3])  # ties
    z[rng.random(z.shape) < 0.01] = 0.0
    at = np.arange(ngroups)
    last = at * epl % group + epl - 1
    z[at[::2], last[::2] - rng.integers(1, epl, size=len(at[::2]))] = 0.0
    z[at, last] = value
    return z * np.float32(sign)


def _wave_pools(group, value, rng):
    """(lane size, sign, bf16 bits) of a few waves of such groups, alone and among ordinary ones."""
    per = 2048 // group
    for epl in (8, 16, 32):
        for sign in (1, -1):
            special = _one_sign(3 * per + 1, group, epl, sign, value, rng)
            plain = rng.standard_normal(special.shape).astype(np.float32)
            mixed = np.concatenate([special, np.where(rng.random((len(plain), 1)) < 0.3, special, plain)])
            yield epl, sign, W.f32_to_bf16_bits(mixed).reshape(-1)


def _bf16(u):
    return torch.from_numpy(u.view(np.int16)).to("cuda").view(torch.bfloat16)


FORMATS = ((2, SR), (3, SR), (4, SR | INT), (7, SR | fcv2.F_META_FP32), (8, SR))


@pytest.mark.parametrize("group", [32, 64, 128, 256])
def test_infinity_in_a_group_of_one_sign(group):
    """An infinity is a spike like any other value (quantize_pack and dispatch_quant, staged and direct rows)."""
    rng = np.random.default_rng(group)
    for epl, sign, x in _wave_pools(group, np.inf, rng):
        for bits, flags in FORMATS:
            want = O.quantize_pack(x, bits, group, flags)
            assert np.array_equal(fcv2.quantize_pack(_bf16(x), bits, group, flags).cpu().numpy(), want), (epl, sign, bits)
        for H, T in ((1024, 7), (16640, 1)):
            t = np.resize(x, (T, H))
            ids = rng.integers(0, 3, size=(T, 2)).astype(np.int32)
            send, offs, src = fcv2.dispatch_quant(_bf16(t), torch.from_numpy(ids).to("cuda"), 3, 4, group, SR)
            send_o, offs_o, src_o = O.dispatch_quant(t, ids, 3, 4, group, SR)
            assert np.array_equal(offs.cpu().numpy(), offs_o) and np.array_equal(src.cpu().numpy(), src_o), (epl, sign, H)
            assert np.array_equal(send.cpu().numpy(), send_o), (epl, sign, H)


@pytest.mark.parametrize("group", [32, 64, 128, 256])
def test_sum_that_overflows_in_a_group_of_one_sign(group):
    """The same in reduce_requant, where the infinity is a sum of finite spikes: the kernel of small payloads (2 to 8 peers), the general
    one (9 peers) and the one of two widths."""
    rng = np.random.default_rng(1000 + group)
    for (epl, sign, x), (_, _, y) in zip(_wave_pools(group, 3.0e38, rng), _wave_pools(group, 3.0e38, rng)):
        for bits, flags in FORMATS:
            recs = [O.quantize_pack(v, bits, group, flags) for v in (x, y)]
            recs += [recs[1]] * 7
            dev = [torch.from_numpy(r).to("cuda") for r in recs]
            for n_peers, bits_out in ((3, bits), (9, bits), (3, bits - 1 if bits > 2 else 3)):
                f_in, f_out = (bits, group, flags), (bits_out, group, flags)
                want, want_sum = O.reduce_requant(recs[:n_peers], x.size, f_in, f_out, want_sum=True)
                assert np.isinf(want_sum).any()
                got = fcv2.reduce_requant(dev[:n_peers], x.size, f_in, f_out).cpu().numpy()
                assert np.array_equal(got, want), (epl, sign, bits, n_peers, bits_out)
