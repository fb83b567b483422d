"""Decode attention (Eq. 1) whose queries share rows, around the sizes where a workgroup serves one, two or four of them: the
whole chain, the compact form's bits and the causal mask against the oracle, as for the other grouped-query shapes."""
import pytest

from tests import test_gqa_causal_gpu as base

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
