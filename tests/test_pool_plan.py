"""Which form chunk pooling takes on the matrix cores (Eq. 2), as the library plans it (no GPU needed)."""
import pytest

from paper_2509_21354_amd import binding as kb


@pytest.mark.parametrize("L,tiles,C,d_sum,form", [
    (1, 512, 8, 128, "one tile"), (1, 513, 8, 128, "persistent"), (1, 1024, 8, 128, "packed"), (1, 1024, 32, 128, "one tile"),
    (4, 1024, 8, 128, "persistent"), (4, 1536, 8, 128, "packed"), (8, 1536, 8, 128, "persistent"), (8, 1920, 8, 128, "packed"),
    (32, 640, 8, 128, "persistent"), (32, 1024, 16, 128, "persistent"), (32, 1888, 32, 128, "persistent"), (32, 2048, 16, 128, "packed"),
    (1, 1536, 8, 64, "persistent"), (8, 2048, 8, 64, "packed"), (1, 2047, 16, 256, "one tile"), (1, 2048, 16, 256, "packed")])
def test_weights_are_re_laid_where_there_are_tiles_to_pay_for_it(L, tiles, C, d_sum, form):
    """The launch that re-lays the MLP weights does so for all layers: many layers of few tiles take them as they are."""
    n = tiles // L * 16
    sh = kb.make_shape(L=L, B=1, H=1, d=128, T=n * C, T_cap=n * C, C=C, N_cap=n, W=C, d_sum=d_sum, d_g=64, dtype=kb.BF16, H_kv=0)
    assert kb.kvev_debug_pool_form(sh, kb.POOL_MLP, n, True) == form
    assert kb.kvev_debug_pool_form(sh, kb.POOL_MLP, n, False) == form.replace("packed", "persistent")
    assert kb.kvev_debug_pool_form(sh, kb.POOL_MEAN, n, True) != "packed"
