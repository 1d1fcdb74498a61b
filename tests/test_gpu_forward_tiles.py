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
