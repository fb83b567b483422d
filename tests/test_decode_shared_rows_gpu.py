"""Decode attention (Eq. 1) whose queries share rows, around the sizes where a workgroup serves one, two or four of them: the
whole chain, the compact form's bits and the causal mask against the oracle, as for the other grouped-query shapes."""
import pytest
import torch

from paper_2509_21354_amd import binding as kb
from tests import test_gqa_causal_gpu as base
from tests.test_decode_plan import shape

pytestmark = pytest.mark.gpu

CASES = [
    # (config, causal)                                                                          sequences x queries
    (base._cfg(601, "bf16", d=128, L=1, B=8, H=16, H_kv=4, T=700, C=32, W=90, k=9), 0),        # 32 x 4: one each, 128 workgroups
    (base._cfg(602, "bf16", d=64, L=1, B=11, H=12, H_kv=3, T=500, C=16, W=60), 0),             # 33 x 4: pairs
    (base._cfg(603, "bf16", d=128, L=1, B=24, H=16, H_kv=4, T=420, C=32, W=70), 0),            # 96 x 4: pairs, 192 workgroups
    (base._cfg(604, "bf16", d=128, L=1, B=97, H=4, H_kv=1, T=420, C=32, W=70), 0),             # 97 x 4: four at a time
    (base._cfg(605, "bf16", d=128, L=1, B=5, H=10, H_kv=5, Tq=3, T=480, C=32, W=100), 1),      # 25 x 6: pairs, causal frame
    (base._cfg(606, "bf16", d=64, L=1, B=6, H=6, H_kv=6, Tq=5, T=480, C=16, W=100), 1),        # 36 x 5: pairs, the last one ragged
    (base._cfg(607, "bf16", d=128, L=1, B=3, H=6, H_kv=6, Tq=7, T=480, C=32, W=280), 1),       # 18 x 7: one each, causal frame
    (base._cfg(608, "f32", d=128, L=2, B=4, H=16, H_kv=4, T=300, C=8, W=50), 0),               # 32 x 4, fp32
    (base._cfg(609, "bf16", d=128, L=1, B=16, H=8, H_kv=4, T=1400, C=32, W=330), 0),           # 64 x 2: a long run keeps pairs
]


@pytest.mark.parametrize("cfg,causal", CASES, ids=[c.name for c, _ in CASES])
def test_queries_that_share_rows(cfg, causal):
    base.test_chain_and_attention_with_grouped_heads_and_causal_frames(cfg, causal)


@pytest.mark.parametrize("S,G,d,dtype,few,many", [
    (48, 2, 128, kb.BF16, 1, 2), (32, 4, 128, kb.BF16, 1, 2), (96, 4, 64, kb.BF16, 2, 4), (64, 2, 64, kb.F32, 1, 2), (48, 4, 128, kb.F32, 2, 4)])
def test_the_choice_changes_no_bit(S, G, d, dtype, few, many):
    """The choice looks at the capacity for kept summaries, which an indexed call and a compact store need not have in common:
    8 summaries kept of 8 and of 256, and in a store of 256 (Eq. 1)."""
    sh, kept = shape(S, G, 287, 256, d, dtype), 8
    assert (kb.kvev_debug_decode_queries(sh, 1, kept), kb.kvev_debug_decode_queries(sh, 1, 256)) == (few, many)
    T, N, win0 = sh.T, sh.N_cap, sh.T - 287
    gen = torch.Generator(device="cuda").manual_seed(3)
    dt = torch.float32 if dtype == kb.F32 else torch.bfloat16
    Q, K, V, Kb, Vb = (torch.randn((1, 1) + s + (d,), device="cuda", generator=gen).to(dt) for s in ((S * G, 1), (S, T), (S, T), (S, N), (S, N)))
    pick = torch.stack([torch.randperm(256, device="cuda", generator=gen)[:kept].sort().values for _ in range(S)]).int()
    count = torch.full((1, 1, S), kept, dtype=torch.int32, device="cuda")
    outs = []
    for cap in (kept, 256):
        idx = torch.zeros((1, 1, S, cap), dtype=torch.int32, device="cuda")
        idx[0, 0, :, :kept] = pick
        outs.append(torch.zeros_like(Q))
        kb.kvev_gated_attention(sh, Q, 1, K, V, Kb, Vb, idx, count, cap, outs[-1])
    store = [torch.zeros((1, 1, S, 256, d), dtype=dt, device="cuda") for _ in range(2)]
    for dst, src in zip(store, (Kb, Vb)):
        dst[0, 0, :, :kept] = src[0, 0].gather(1, pick.long()[..., None].expand(-1, -1, d))
    wsh = kb.make_shape(L=1, B=1, H=S * G, d=d, T=287, T_cap=287, C=8, N_cap=256, W=287, d_sum=32, d_g=64, dtype=dtype, H_kv=S)
    outs.append(torch.zeros_like(Q))
    kb.kvev_compact_attention(wsh, Q, 1, K[..., win0:, :].contiguous(), V[..., win0:, :].contiguous(), *store, count, 256, outs[-1])
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]) and float(outs[0].float().abs().max()) > 0
