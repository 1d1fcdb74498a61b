"""The backward with each key block's query tiles split into parts (problems
with few key blocks): against the same call with a workspace that lacks the
partial sums, which runs unsplit.  The parts' FP32 sums are added at the end,
so dK and dV agree to FP32 rounding of their terms and dQ, which no sum of
them touches, bit for bit; the instrumented kernel splits alike."""
import numpy as np
import pytest
import torch

import paper_2609_37852_amd as pk
from _helpers import unsplit_bytes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,Nk,Hq,Hkv,dqk,dv,causal,flags,lens", [
    (1, 512, 0, 16, 4, 128, 128, True, 0, None),
    (1, 352, 0, 5, 1, 128, 128, True, 0, None),          # ragged tiles, parts of unequal length
    (2, 480, 0, 8, 2, 64, 64, True, 0, [480, 96]),       # fewer tiles than parts in the short sequence
    (2, 480, 0, 8, 2, 128, 128, True, 0, [0, 320]),      # one sequence without tokens
    (1, 1056, 160, 8, 2, 128, 128, False, 0, None),
    (1, 544, 0, 4, 1, 256, 256, True, 0, None),
    (1, 1024, 0, 8, 2, 192, 128, True, 0, None),
    (1, 512, 0, 8, 2, 128, 128, True, pk.FLAG_PBWD_BLOCK_SCALED, None),
    (1, 512, 0, 8, 2, 128, 128, True, pk.FLAG_ISOLATE3, None),
    (1, 512, 0, 8, 2, 128, 128, True, pk.FLAG_PROTECTED_DP, None),
])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_split_equals_unsplit(B, N, Nk, Hq, Hkv, dqk, dv, causal, flags, lens, dtype):
    Nk = Nk or N
    g = torch.Generator(device="cuda").manual_seed(3)
    q, do = (torch.randn((B, N, Hq, d), generator=g, device="cuda") for d in (dqk, dv))
    k, v = (torch.randn((B, Nk, Hkv, d), generator=g, device="cuda") for d in (dqk, dv))
    L = torch.tensor(lens, dtype=torch.int32, device="cuda") if lens else None
    p = pk.Problem(B, N, Hq, Hkv, dqk, dv, float(np.float32(dqk ** -0.5)), causal=int(causal),
                   seqlen_kv=0 if causal else Nk, flags=flags, seqlens_q=L)
    mq, mk, mv, mdo = (pk.attn_fp8_quantize(t) for t in (q, k, v, do))
    o, lse = pk.attn_fp8_fwd(p, mq, mk, mv, lse=torch.zeros((B, Hq, N), device="cuda"), o=torch.zeros_like(do))
    need, base = pk.attn_fp8_bwd_workspace_size(p), unsplit_bytes(p)
    assert need > base, "this problem is not split"

    def run(nbytes, rowstats=False):
        out = tuple(torch.full(t.shape, 3.0, dtype=dtype, device="cuda") for t in (q, k, v))
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        if flags & pk.FLAG_PROTECTED_DP:
            return pk.attn_fp8_bwd_protected_dp(p, mq, mk, mdo, lse, do, v, o, workspace=ws, out=out, rowstats=rowstats)[:3]
        return pk.attn_fp8_bwd(p, pk.DELTA_MATCHING, mq, mk, mv, mdo, lse, workspace=ws, out=out, rowstats=rowstats)[:3]

    split, one, stats = run(need), run(base), run(need, rowstats=True)
    assert torch.equal(split[0], one[0])
    for x, y, z in zip(split[1:], one[1:], stats[1:]):
        assert torch.equal(x, z)
        # FP32: at most n = 16 head x tile sums regrouped, 2^-24 of the largest partial sum each
        tol = 2.0 ** -7 if dtype == torch.bfloat16 else 1e-5
        assert (x.double() - y.double()).norm() <= tol * y.double().norm()
        assert torch.equal(x == 3.0, y == 3.0)      # the same rows left unwritten
    with pytest.raises(pk.AttnFp8Error):
        run(base - 256)
