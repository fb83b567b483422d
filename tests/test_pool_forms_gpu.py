"""Chunk pooling (Eq. 2) around the numbers of tiles (16 chunk rows of a layer) where the launch changes from 16 waves on one tile
to the persistent form: the summaries of one call are those of the same chunks pooled in small calls, bit for bit."""
import pytest
import torch

from paper_2509_21354_amd import binding as kb
from paper_2509_21354_amd import synth
from tests import test_parity_gpu as base

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,C,BH,N,d_sum,mode", [
    (128, 8, 32, 256, 128, kb.POOL_MLP),        # 512 tiles: 16 waves
    (128, 8, 27, 304, 128, kb.POOL_MLP),        # 513
    (64, 16, 9, 914, 64, kb.POOL_MLP),          # 515, the last one ragged
    (128, 29, 41, 500, 96, kb.POOL_MLP),        # 1282: a long chunk whose tail is padded
    (64, 24, 41, 400, 256, kb.POOL_MLP),        # 1025, wide hidden layer: 16 waves, two tasks a wave
    (64, 16, 9, 914, 32, kb.POOL_MLP),          # one k-step in the second layer
    (128, 16, 41, 400, 128, kb.POOL_MEAN),      # 1025
    (64, 8, 41, 400, 128, kb.POOL_MAX),
    (128, 8, 41, 400, 128, kb.POOL_MLP),        # 1025: weights re-laid first
])
def test_pooling_in_one_call_and_in_pieces(d, C, BH, N, d_sum, mode):
    cfg = base._cfg(501, "bf16", d=d, C=C, T=N * C, d_sum=d_sum, L=1, B=1, H=BH)
    g = torch.Generator().manual_seed(7)
    K, V = (torch.randn((1, 1, BH, N * C, d), generator=g).bfloat16().cuda() for _ in "KV")
    w = base.dev(synth.make_weights(cfg, "cpu"))
    sh = kb.make_shape(cfg, N_cap=N)
    outs = []
    for piece in (N, 97):
        Kbar, Vbar = (torch.zeros((1, 1, BH, N, d), dtype=torch.bfloat16, device="cuda") for _ in "KV")
        ws = kb.alloc_workspace(kb.workspace_bytes(kb.OP_CHUNK_POOL, sh, N))
        for c0 in range(0, N, piece):
            kb.kvev_chunk_pool(sh, K, V, mode, kb.mlp_weights(w, "K"), kb.mlp_weights(w, "V"), c0, min(N, c0 + piece), Kbar, Vbar, ws)
        torch.cuda.synchronize()
        outs.append((Kbar, Vbar))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert torch.isfinite(outs[0][0].float()).all() and outs[0][1].float().abs().max() > 0
