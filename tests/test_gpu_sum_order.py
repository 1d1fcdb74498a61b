"""The order in which the kernels add up what they keep: it fixes the last
bits of the LSE and of the correction, and through them the FP8 codes of P and
dS that lie at a rounding boundary, so it does not change with the schedule of
a kernel.  Inputs whose scores, probabilities and products are powers of two,
so that every rounding is one of the sums'."""
import numpy as np
import pytest
import torch

import paper_2609_37852_amd as pk

pytestmark = pytest.mark.gpu

LN2 = float(np.float32(np.log(2.0)))     # softmax_scale: the kernels' factor tau log2(e) is then 1
PAIRS = [(64, 64), (128, 128), (192, 128), (256, 256)]


def _first_channel(x, d):
    """x [n] as a [1, n, 1, d] tensor, zero but for its first channel."""
    t = torch.zeros((1, len(x), 1, d), device="cuda")
    t[0, :, 0, 0] = torch.as_tensor(np.asarray(x, np.float32), device="cuda")
    return t


@pytest.mark.parametrize("flags", [0, pk.FLAG_ISOLATE3])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("dqk,dv", PAIRS)
def test_forward_sum_runs_over_the_keys_in_order(dqk, dv, causal, flags):
    """A lane's exponentials (keys with j % 8 < 4, or the others) are one FP32
    sum, keys ascending: after a one at key 0, terms of 2^-24 are half a unit
    in the last place and leave it as it is; in the other lane half's sum
    they stay.  Two interleaved sums would keep half of the first ones too."""
    n = 2048
    s = np.full(n, -24.0)
    s[0] = 0.0
    nq = n if causal else 32
    p = pk.Problem(1, nq, 1, 1, dqk, dv, LN2, causal=int(causal), seqlen_kv=0 if causal else n, flags=flags)
    mx = [pk.attn_fp8_quantize(t) for t in (_first_channel(np.ones(nq), dqk), _first_channel(s, dqk), _first_channel(s, dv))]
    lse = pk.attn_fp8_fwd(p, *mx)[1][0, 0].double().cpu().numpy()
    rest = np.cumsum(np.arange(n) % 8 >= 4)
    want = np.log1p((rest if causal else np.full(nq, rest[-1])) * 2.0 ** -24)
    # an FP32 logarithm near 1 and two roundings: 2^-21; two interleaved sums are up to 2^-15 off
    assert np.abs(lse - want).max() <= 2.0 ** -21, np.abs(lse - want).max()


def _group_sums(x, t):
    """Row sums of x [rows, keys] as the correction takes them: of each 32 keys
    the two lane halves' (keys with j % 8 < 4, or the others; ascending), each
    in type t, their total in t, and these totals in FP64, ascending."""
    g = x.astype(t).reshape(len(x), -1, 4, 2, 4)       # [rows, group, 8 keys, half, 4 keys]
    half = np.zeros(g.shape[:2] + (2,), t)
    for a in range(4):
        for b in range(4):
            half = half + g[:, :, a, :, b]
    total = np.zeros(len(x))
    for i in range(g.shape[1]):
        total = total + (half[:, i, 0] + half[:, i, 1]).astype(np.float64)
    return total


@pytest.mark.parametrize("n,nq,B", [(64, 32, 1), (288, 288, 1), (96, 96, 1200)])   # the last: two query blocks per wave
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("mode,flags", [(pk.DELTA_MATCHING, 0), (pk.DELTA_MATCHING, pk.FLAG_ISOLATE3),
                                        (pk.DELTA_MATCHING_COMPENSATED, 0)])
@pytest.mark.parametrize("dqk,dv", PAIRS)
def test_correction_sums_in_groups_of_32_keys(dqk, dv, mode, flags, causal, n, nq, B):
    """P dP and P summed in FP32 (compensated: FP64) within each group of 32
    keys and in FP64 over the groups: bit for bit, with P = 2^-a and dP = 2^b of
    exponents wide enough that most sums round."""
    rng = np.random.default_rng(dqk + n)
    nq = n if causal else nq
    comp = mode == pk.DELTA_MATCHING_COMPENSATED
    a = rng.integers(0, 17, n)                         # each an E4M3 value
    b = rng.integers(0, 80 if comp else 40, n)
    sign = rng.choice([-1.0, 1.0], n)
    p = pk.Problem(B, nq, 1, 1, dqk, dv, LN2, causal=int(causal), seqlen_kv=0 if causal else n, flags=flags)
    ins = (_first_channel(np.ones(nq), dqk), _first_channel(-a, dqk), _first_channel(sign * 2.0 ** b, dv),
           _first_channel(np.ones(nq), dv))
    mx = [pk.attn_fp8_quantize(t.expand(B, -1, -1, -1).contiguous()) for t in ins]
    # two query blocks per wave from 4 workgroups per compute unit on (2 at d = 256; never at 192 / 128)
    assert B == 1 or B > 4 * torch.cuda.get_device_properties(0).multi_processor_count
    got = pk.attn_fp8_delta(p, mode, *mx, lse=torch.zeros((B, 1, nq), device="cuda"))
    assert torch.equal(got, got[:1].expand_as(got).contiguous())
    see = np.tril(np.ones((n, n))) if causal else np.ones((nq, n))
    P = see * 2.0 ** -a
    t = np.float64 if comp else np.float32
    d = _group_sums(P * (sign * 2.0 ** b), t) / _group_sums(P, t)
    hi = d.astype(np.float32)
    want = np.stack([hi, (d - hi.astype(np.float64)).astype(np.float32)], -1)
    assert np.array_equal(got[0, 0].cpu().numpy(), want)
