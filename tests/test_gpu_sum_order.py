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
