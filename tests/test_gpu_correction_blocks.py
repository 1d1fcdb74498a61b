"""The matched correction with two 32-query blocks per wave (launches of two
rounds of workgroups and more) equals, bit for bit, the one-block kernel that
a single batch entry of the same problem takes: both form the same sums in
the same order, whichever tiles they count as full."""
import numpy as np
import pytest
import torch

import paper_2609_37852_amd as pk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,Nk,dqk,dv,causal,mode,flags,lens", [
    (32, 0, 128, 128, True, "matching", 0, False),
    (288, 0, 128, 128, True, "matching", 0, False),        # one full 256-query block, a ragged one
    (352, 0, 128, 128, True, "matching", 0, True),
    (224, 416, 128, 128, False, "matching", 0, False),     # three full key tiles, a ragged one
    (256, 128, 128, 128, False, "matching", 0, False),     # one key tile, no edge tile
    (544, 0, 64, 64, True, "matching", 0, False),
    (96, 288, 64, 64, False, "matching", 0, False),
    (288, 0, 256, 256, True, "matching", 0, False),
    (96, 160, 256, 256, False, "matching", 0, False),
    (320, 0, 128, 128, True, "compensated", 0, False),
    (288, 0, 128, 128, True, "matching", pk.FLAG_ISOLATE3, False),
    (160, 320, 128, 128, False, "matching", pk.FLAG_ISOLATE3, False),
])
def test_two_blocks_equal_one(N, Nk, dqk, dv, causal, mode, flags, lens):
    B, Hq, Hkv = 160, 8, 4
    # the kernel with two blocks is taken from 2 rounds of workgroups (256 queries each; 2 a compute unit, at d = 256 1) on
    threshold = 2 * (1 if dqk == 256 else 2) * torch.cuda.get_device_properties(0).multi_processor_count
    workgroups = (N + 255) // 256 * Hq
    assert workgroups < threshold < B * workgroups, "both sides of this test would run the same kernel"
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(11)
    Nk = Nk or N

    def normal(n, h, d):
        return torch.randn((B, n, h, d), generator=g, device=dev).bfloat16()

    q, k, v, do = normal(N, Hq, dqk), normal(Nk, Hkv, dqk), normal(Nk, Hkv, dv), normal(N, Hq, dv)
    q[..., 5] *= 8.0
    k[..., 5] *= 8.0
    L = torch.tensor([(b * 32) % (N + 32) for b in range(B)], dtype=torch.int32, device=dev) if lens else None
    m = pk.DELTA_MATCHING_COMPENSATED if mode == "compensated" else pk.DELTA_MATCHING
    tau = float(np.float32(dqk ** -0.5))

    def run(sl, seq):
        x = [t[sl].contiguous() for t in (q, k, v, do)]
        p = pk.Problem(x[0].shape[0], N, Hq, Hkv, dqk, dv, tau, causal=int(causal), seqlen_kv=0 if causal else Nk,
                       flags=flags, seqlens_q=seq)
        mx = [pk.attn_fp8_quantize(t) for t in x]
        lse = torch.zeros((x[0].shape[0], Hq, N), device=dev)
        pk.attn_fp8_fwd(p, *mx[:3], lse=lse)
        delta = torch.zeros((x[0].shape[0], Hq, N, 2), device=dev)
        return pk.attn_fp8_delta(p, m, *mx, lse=lse, delta=delta)

    many = run(slice(None), L)
    for b in (0, 1, 63, 159):
        one = run(slice(b, b + 1), L[b:b + 1].contiguous() if lens else None)
        assert torch.equal(many[b], one[0]), f"batch entry {b}"
    assert torch.isfinite(many).all() and many.abs().max() > 0
