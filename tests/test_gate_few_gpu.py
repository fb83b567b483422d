"""The gate of few sequences (bf16, Eq. 3): at d_g = 512 on eight workgroups per 4, 8 or 16 sequences, which caches of 16 chunks and
more take while the launch fits the chip, and at d_g = 256 on four per 4 or 8: against the CPU oracle, and the things that must
not depend on how a call is cut."""
import numpy as np
import pytest
import torch

from oracle import kvev_oracle as orc
from paper_2509_21354_amd import binding as kb
from paper_2509_21354_amd import synth
from tests import test_parity_gpu as base

pytestmark = pytest.mark.gpu

CASES = [
    base._cfg(401, "bf16", d=128, T=17 * 32, C=32, d_g=512, L=1, B=1, H=1),      # one sequence
    base._cfg(402, "bf16", d=64, T=16 * 32, C=32, d_g=512, L=3, B=1, H=13),      # 12 groups of 4, the last of a layer with one sequence
    base._cfg(403, "bf16", d=128, T=19 * 32, C=32, d_g=512, L=4, B=2, H=32),     # 32 groups of 8: a workgroup on every compute unit
    base._cfg(404, "bf16", d=64, T=16 * 32, C=32, d_g=512, L=11, B=1, H=19),     # two groups in turn; three a layer, the last ragged, the fourth empty
    base._cfg(405, "bf16", d=128, T=18 * 32, C=32, d_g=512, L=32, B=1, H=9),     # two in turn in every layer, the second with one sequence
    base._cfg(406, "bf16", d=128, T=16 * 32, C=32, d_g=512, L=2, B=2, H=32),     # 32 groups of 4
    base._cfg(407, "bf16", d=128, T=17 * 32, C=32, d_g=512, L=3, B=1, H=42),     # 33: groups of 8
    base._cfg(408, "bf16", d=128, T=17 * 32, C=32, d_g=256, L=1, B=8, H=32),     # d_g = 256: 64 groups of 4
    base._cfg(409, "bf16", d=64, T=17 * 32, C=32, d_g=256, L=2, B=3, H=43),      # 66: groups of 8, the last of a layer with one sequence
    base._cfg(410, "bf16", d=64, T=16 * 32, C=32, d_g=256, L=2, B=1, H=6),        # a ragged second group of 4
]


@pytest.mark.parametrize("cfg", CASES, ids=lambda c: c.name)
def test_few_sequences(cfg):
    """... in one call, in pieces with scratch for two steps and for all, one step per call, and with the scratch of a plan for fewer
    chunks (at d_g = 512 that may hold no projections and take another form: the oracle's values, not the same bits)."""
    N = cfg.T // cfg.C
    w = synth.make_weights(cfg, "cpu")
    Kbar, Vbar = base._summaries(cfg, N)
    sh = kb.make_shape(cfg, N_cap=N)
    lead = (cfg.L, cfg.B, cfg.H)
    gw, Kb, Vb = base.dev(w), Kbar.cuda(), Vbar.cuda()
    plain = kb.workspace_bytes(kb.OP_LSTM_GATE, kb.make_shape(cfg, N_cap=15, T=15 * cfg.C), 0)
    outs = []
    for cuts, steps in (([(0, N)], N), ([(0, 1), (1, 6), (6, N)], 2), ([(t, t + 1) for t in range(N)], 1), ([(0, N)], None)):
        ws = kb.alloc_workspace(plain if steps is None else kb.workspace_bytes(kb.OP_LSTM_GATE, sh, steps))
        h = torch.full(lead + (cfg.d_g,), 7.0, device="cuda")
        c = torch.full_like(h, float("nan"))
        util = torch.full(lead + (N,), 9.0, device="cuda")
        gate = torch.full_like(util, 9.0)
        for a, b in cuts:
            kb.kvev_lstm_gate(sh, Kb, Vb, kb.lstm_weights(gw), a, b, h, c, util, gate, ws)
        torch.cuda.synchronize()
        assert int(ws[:4].view(torch.int32).item()) == 0
        outs.append((h, c, util, gate))
    for out in outs[1:3]:
        assert all(torch.equal(x, y) for x, y in zip(outs[0], out))
    ref = orc.lstm_gate(Kbar, Vbar, kb.lstm_weights(w), 0, N)
    for out in (outs[0], outs[3]):
        for got, r, tol in zip(out, ref, (1, 2, 1, 1)):
            assert np.abs(got.cpu().numpy() - r).max() <= tol * base.SCORE_TOL


def test_cases_reach_the_forms_they_claim():
    assert [base.gate_form(c) for c in CASES] == [(8, 4), (8, 4), (8, 8), (8, 16), (8, 16), (8, 4), (8, 8), (4, 4), (4, 8), (4, 4)]


@pytest.mark.parametrize("cfg", [CASES[1], CASES[2], CASES[3], CASES[8], CASES[9]], ids=lambda c: c.name)
def test_nan_stays_in_its_sequence(cfg):
    base.test_lstm_gate_nan_stays_in_its_sequence(cfg, 0)


@pytest.mark.parametrize("cfg", [CASES[1], CASES[2], CASES[3], CASES[9]], ids=lambda c: c.name)
def test_wait_expires(cfg):
    """A member that withholds its publications: every wait ends, scores and cell state come back NaN, the status word is set."""
    base.test_lstm_pair_wait_expires_cleanly(cfg)


@pytest.mark.parametrize("cfg,members", [(CASES[1], 8), (CASES[2], 8), (CASES[3], 8), (CASES[9], 4)], ids=lambda c: getattr(c, "name", str(c)))
def test_h_is_kept_until_all_are_heard(cfg, members):
    """No member replaces its units of the carried h before it has heard from all others."""
    N, t, width = 16, 2, cfg.d_g // members
    w = synth.make_weights(cfg, "cpu")
    Kbar, Vbar = base._summaries(cfg, N)
    sh = kb.make_shape(cfg, N_cap=N, T=N * cfg.C, T_cap=N * cfg.C)
    gw, Kb, Vb = base.dev(w), Kbar.cuda(), Vbar.cuda()
    ws = kb.alloc_workspace(kb.workspace_bytes(kb.OP_LSTM_GATE, sh, N))
    h0 = torch.zeros((cfg.L, cfg.B, cfg.H, cfg.d_g), device="cuda")
    c0, util = torch.zeros_like(h0), torch.zeros((cfg.L, cfg.B, cfg.H, N), device="cuda")
    gate = torch.zeros_like(util)
    kb.kvev_lstm_gate(sh, Kb, Vb, kb.lstm_weights(gw), 0, t, h0, c0, util, gate, ws)

    def step():
        h, c = h0.clone(), c0.clone()
        kb.kvev_lstm_gate(sh, Kb, Vb, kb.lstm_weights(gw), t, t + 1, h, c, util, gate, ws)
        torch.cuda.synchronize()
        return h, c

    good_h, good_c = step()
    kb.kvev_debug_pair_wait(4096, 1)
    try:
        h, c = step()
    finally:
        kb.kvev_debug_pair_wait()
    assert int(ws[:4].view(torch.int32).item()) == 1
    for m in range(members):
        u = slice(m * width, (m + 1) * width)
        if m == 1:
            assert torch.equal(c[..., u], good_c[..., u]) and torch.equal(h[..., u], good_h[..., u])
        else:
            assert torch.isnan(c[..., u]).all() and torch.equal(h[..., u], h0[..., u])


def test_projections_of_many_steps():
    """Scratch for more steps than 32 bits address the projections of (d_g = 512: 128 KiB a step): the bits of a call whose
    projections are made 128 steps at a time."""
    N = 32768 + 40
    cfg = base._cfg(411, "bf16", d=64, T=N, C=1, W=0, d_g=512, L=1, B=1, H=1)
    gen = torch.Generator(device="cuda").manual_seed(1)
    Kb, Vb = (torch.randn((1, 1, 1, N, 64), device="cuda", generator=gen).mul_(0.25).bfloat16() for _ in range(2))
    sh, gw = kb.make_shape(cfg, N_cap=N), base.dev(synth.make_weights(cfg, "cpu"))
    small = kb.workspace_bytes(kb.OP_LSTM_GATE, sh, 128)
    outs = []
    for nbytes in (small, small + (N - 128) * 131072):
        ws = kb.alloc_workspace(nbytes)
        h, c = (torch.zeros((1, 1, 1, 512), device="cuda") for _ in range(2))
        util, gate = (torch.zeros((1, 1, 1, N), device="cuda") for _ in range(2))
        kb.kvev_lstm_gate(sh, Kb, Vb, kb.lstm_weights(gw), 0, N, h, c, util, gate, ws)
        torch.cuda.synchronize()
        assert int(ws[:4].view(torch.int32).item()) == 0
        outs.append((h, c, util, gate))
    assert all(torch.equal(x, y) for x, y in zip(*outs))
    assert 0 < float(outs[0][2].std())


@pytest.mark.parametrize("L,BH,d,d_g,N", [
    (4, 16, 128, 256, 8), (9, 64, 128, 256, 64), (9, 64, 64, 256, 64), (32, 16, 128, 128, 64), (32, 16, 64, 128, 64), (12, 4, 64, 512, 2), (13, 4, 128, 512, 2)])
def test_plain_and_prepared_weights(L, BH, d, d_g, N):
    """W_hh re-laid beside the first projection, in a launch of its own and by kvev_lstm_prepare: the same bits."""
    cfg = base._cfg(412, "bf16", d=d, T=N * 8, C=8, d_g=d_g, L=L, B=1, H=BH)
    gen = torch.Generator(device="cuda").manual_seed(1)
    Kb, Vb = (torch.randn((L, 1, BH, N, d), device="cuda", generator=gen).mul_(0.25).bfloat16() for _ in range(2))
    sh, w = kb.make_shape(cfg, N_cap=N), kb.lstm_weights(base.dev(synth.make_weights(cfg, "cpu")))
    packed = kb.alloc_workspace(kb.workspace_bytes(kb.OP_LSTM_PREPARE, sh, 0))
    kb.kvev_lstm_prepare(sh, w, packed)
    outs = []
    for prepared in (False, True):
        ws = kb.alloc_workspace(kb.workspace_bytes(kb.OP_LSTM_GATE_PREPARED if prepared else kb.OP_LSTM_GATE, sh, N))
        h, c = (torch.zeros((L, 1, BH, d_g), device="cuda") for _ in range(2))
        util, gate = (torch.zeros((L, 1, BH, N), device="cuda") for _ in range(2))
        if prepared:
            kb.kvev_lstm_gate_prepared(sh, Kb, Vb, w, packed, 0, N, h, c, util, gate, ws)
        else:
            kb.kvev_lstm_gate(sh, Kb, Vb, w, 0, N, h, c, util, gate, ws)
        torch.cuda.synchronize()
        outs.append((h, c, util, gate))
    assert all(torch.equal(x, y) for x, y in zip(*outs)) and float(outs[0][2].std()) > 0
