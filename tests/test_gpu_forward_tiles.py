"""The forward at the edges of its key tiles and units against the oracle:
one key group, a tile exactly, a tile and a group, enough tiles to pass
through every buffer of the rotation, with and without the mask at every head
dim, and rows whose maximum rises far above the running reference in the
middle of the sequence (the rescale of O, of the sums and of codes not yet
multiplied).  Bounds as in the parity cases: relative Frobenius error <= 2e-2
for O and its median 32-row block, 2^-3 for every block, LSE within 1e-3."""
import numpy as np
import pytest
import torch

import paper_2609_37852_amd as pk
from paper_2609_37852_amd import synth
from _helpers import REL_TOL, block_errors, check_blocks, np64, problem, rel_err, run_oracle, to_dev

pytestmark = pytest.mark.gpu

D64, D128, D192, D256 = "tiny_mha_128", "gqa_d128_64k_nope", "mla_d192_4k", "gqa_d256_8k_qknorm"
CASES = [(r, n, n, True, False) for r in (D64, D128, D192, D256) for n in (32, 128, 160)]
CASES += [(r, 64, nk, False, False) for r in (D64, D128, D192, D256) for nk in (32, 64, 128, 288)]
CASES += [(D128, 416, 416, True, False), (D192, 544, 544, True, False), (D192, 96, 480, False, False)]
CASES += [(r, 384, 384, True, True) for r in (D64, D128, D192, D256)] + [(D192, 64, 512, False, True)]


@pytest.mark.parametrize("recipe,N,Nk,causal,rise", CASES)
def test_forward_tiles(recipe, N, Nk, causal, rise):
    w0 = synth.WORKLOADS[recipe]
    w = synth.with_shape(w0, B=1, N=N, Nk=0 if causal else Nk, Hq=2, Hkv=1 if w0.Hq != w0.Hkv else 2, causal=causal)
    d = synth.generate(w, seed=5)
    if rise:
        # each 64 keys score several times higher than the 64 before
        f = 3.0 ** (np.arange(w.nk) // 64)
        d["k"] = d["k"] * np.minimum(f, 81.0).astype(np.float32)[None, :, None, None]
    if w.dtype == "bf16":
        d["k"] = synth.round_bf16(d["k"])
    q, k, v = (to_dev(d[n], w.dtype) for n in ("q", "k", "v"))
    o, lse = pk.attn_fp8_fwd(problem(w), *(pk.attn_fp8_quantize(t) for t in (q, k, v)), o_dtype=torch.float32)
    ref = run_oracle(w, d)
    assert rel_err(np64(o), ref["O"]) <= REL_TOL
    check_blocks({"O": block_errors(np64(o), ref["O"])})
    assert np.max(np.abs(np64(lse) - ref["LSE"])) <= 1e-3 * max(1.0, float(np.max(np.abs(ref["LSE"]))))


# Rows whose maximum jumps by 2^J after `early` keys of score 0: V of the early keys is 2^100 in half the channels, of
# the later ones 1 in the others, so O shows the early weights 2^-J itself.  Exact in the codes (score J, weights of
# the early groups 2^-8 * 256, V); FP32 holds weights down to 2^-126 of the running maximum, and smaller ones are 0.
@pytest.mark.parametrize("dqk,dv", [(64, 64), (128, 128), (192, 128), (256, 256)])
@pytest.mark.parametrize("early,J", [(64, 104), (64, 120), (64, 128), (128, 120), (128, 208), (192, 128), (256, 120), (256, 144)])
@pytest.mark.parametrize("causal", [True, False])
def test_forward_far_jump(dqk, dv, early, J, causal):
    N = 512
    q, k, v = torch.zeros(1, N, 1, dqk), torch.zeros(1, N, 1, dqk), torch.zeros(1, N, 1, dv)
    q[..., 0], k[:, early:, :, 0] = 1.0, float(J)
    v[:, :early, :, :dv // 2], v[:, early:, :, dv // 2:] = 2.0 ** 100, 1.0
    p = pk.Problem(1, N, 1, 1, dqk, dv, float(np.float32(np.log(2.0))), causal=int(causal), seqlen_kv=0 if causal else N)
    o, lse = pk.attn_fp8_fwd(p, *(pk.attn_fp8_quantize(t.cuda()) for t in (q, k, v)), o_dtype=torch.float32)
    o, lse = np64(o)[0, :, 0], np64(lse)[0, 0]
    late = np.arange(N) - early + 1 if causal else np.full(N, N - early)      # later keys each query sees
    i = late > 0
    w = early * 2.0 ** -J / late[i]                                           # weight of all early keys
    low, high = o[i, :dv // 2], o[i, dv // 2:]
    rel = 4 * 2.0 ** -23                                                      # l's reciprocal and the product; the rest is exact
    flushed = early * 2.0 ** -126 / late[i] if J > 126 else 0.0               # weights below FP32's range are 0
    assert np.all(np.abs(low * 2.0 ** -100 - w[:, None]) <= (rel * w + flushed)[:, None])
    assert np.all(np.abs(high - 1.0) <= rel)
    assert np.all(np.abs(lse[i] - (J + np.log2(late[i])) * np.log(2.0)) <= 1e-4)
