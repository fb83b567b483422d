"""How many of the queries that share rows a decode workgroup serves (Eq. 1), as the library plans it (no GPU needed)."""
import pytest

from paper_2509_21354_amd import binding as kb


def shape(S, G, raw, kept, d, dtype):
    """S key-value sequences, G query heads each, `raw` raw rows behind `kept` candidate summaries"""
    T = raw + 8 * kept
    return kb.make_shape(L=1, B=1, H=S * G, d=d, T=T, T_cap=T, C=8, N_cap=T // 8, W=raw, d_sum=32, d_g=64, dtype=dtype, H_kv=S)


@pytest.mark.parametrize("S,G,raw,kept,d,dtype,queries", [
    (32, 4, 287, 32, 128, kb.BF16, 1), (16, 4, 287, 256, 128, kb.BF16, 1), (32, 4, 287, 256, 128, kb.BF16, 2), (64, 2, 287, 32, 128, kb.BF16, 1),
    (32, 2, 319, 512, 128, kb.BF16, 2), (48, 2, 319, 512, 128, kb.BF16, 2), (48, 2, 287, 256, 128, kb.BF16, 2), (65, 2, 60, 8, 128, kb.BF16, 2),
    (96, 4, 319, 0, 128, kb.BF16, 2), (97, 4, 319, 0, 128, kb.BF16, 4), (64, 2, 319, 512, 64, kb.BF16, 2), (48, 8, 319, 512, 64, kb.BF16, 4),
    (32, 12, 319, 512, 64, kb.BF16, 4), (16, 4, 319, 512, 128, kb.BF16, 1), (48, 4, 319, 512, 128, kb.BF16, 4), (96, 4, 319, 512, 128, kb.BF16, 2), (96, 4, 420, 512, 64, kb.BF16, 2), (100, 1, 300, 512, 128, kb.BF16, 1),
    (32, 4, 160, 0, 128, kb.F32, 1), (64, 2, 32, 256, 128, kb.F32, 2), (96, 4, 160, 0, 128, kb.F32, 2), (96, 4, 250, 0, 128, kb.F32, 4),
    (64, 4, 420, 512, 64, kb.F32, 2), (96, 4, 340, 64, 64, kb.F32, 4), (96, 4, 340, 64, 128, kb.F32, 4)])
def test_queries_share_a_workgroup_where_their_rows_would_not_stay_in_cache(S, G, raw, kept, d, dtype, queries):
    assert kb.kvev_debug_decode_queries(shape(S, G, raw, kept, d, dtype), 1, kept) == queries
