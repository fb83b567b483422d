"""The fp32-arithmetic gate above 128 units (Eq. 3): bf16 storage up to 192 units, where the rows of W_hh stay in registers as pairs,
and the widths that read them every step, one and four sequences to a workgroup on both sides of the number of compute units."""
import numpy as np
import pytest
import torch

from oracle import kvev_oracle as orc
from paper_2509_21354_amd import binding as kb
from paper_2509_21354_amd import synth
from tests import test_parity_gpu as base

pytestmark = pytest.mark.gpu

CASES = [
    (base._cfg(421, "bf16", d=64, C=8, d_g=129, L=1, B=1, H=3), 17),       # the third unit of a lane group: one group's only; rows at odd elements
    (base._cfg(422, "bf16", d=128, C=8, d_g=132, L=2, B=1, H=2), 16),      # rows of whole groups of four
    (base._cfg(423, "bf16", d=128, C=8, d_g=163, L=2, B=1, H=3), 33),
    (base._cfg(424, "bf16", d=64, C=8, d_g=191, L=1, B=3, H=1), 15),
    (base._cfg(425, "bf16", d=128, C=8, d_g=192, L=1, B=1, H=2), 18),      # the widest
    (base._cfg(426, "bf16", d=64, C=8, d_g=162, L=3, B=18, H=19), 3),      # more sequences than four on every compute unit
    (base._cfg(427, "bf16", d=64, C=8, d_g=193, L=1, B=1, H=3), 17),       # read every step, one sequence a workgroup
    (base._cfg(428, "bf16", d=128, C=8, d_g=200, L=1, B=1, H=257), 17),    # ... four, the last workgroup with one
    (base._cfg(429, "f32", d=64, C=8, d_g=130, L=1, B=8, H=32), 5),        # a sequence for every compute unit
    (base._cfg(430, "f32", d=128, C=8, d_g=129, L=3, B=2, H=43), 5),       # 258 sequences, the last of a layer's workgroups with two
    (base._cfg(434, "bf16", d=64, C=8, d_g=163, L=1, B=1, H=1030), 40),   # a call of all steps keeps its rows, one of a single step reads them for four
    (base._cfg(435, "bf16", d=128, C=8, d_g=164, L=2, B=3, H=100), 40),    # the same at rows of whole groups of four
    (base._cfg(432, "f32", d=64, C=8, d_g=132, L=3, B=3, H=57), 5),        # 513: four a workgroup at aligned rows too, the last with three
]


@pytest.mark.parametrize("cfg,steps", CASES, ids=lambda c: getattr(c, "name", None))
def test_wide_gate_of_any_width(cfg, steps):
    """... against the oracle, and cut into calls the bits of one call; what lies beyond the last sequence stays as it was."""
    cfg = cfg.replace(T=steps * cfg.C)
    w = synth.make_weights(cfg, "cpu")
    Kbar, Vbar = base._summaries(cfg, steps)
    sh = kb.make_shape(cfg, N_cap=steps)
    lead = (cfg.L, cfg.B, cfg.H)
    gw, Kb, Vb = base.dev(w), Kbar.cuda(), Vbar.cuda()
    ws = kb.alloc_workspace(kb.workspace_bytes(kb.OP_LSTM_GATE, sh, steps))
    outs = []
    for cuts in ([0, steps], sorted({0, 1, steps // 2, steps - 1, steps})):
        h, c = (torch.full(lead + (cfg.d_g,), 7.0, device="cuda") for _ in range(2))
        util, gate = (torch.zeros(lead + (steps,), device="cuda") for _ in range(2))
        for a, b in zip(cuts, cuts[1:]):
            kb.kvev_lstm_gate(sh, Kb, Vb, kb.lstm_weights(gw), a, b, h, c, util, gate, ws)
        torch.cuda.synchronize()
        outs.append((h, c, util, gate))
    assert all(torch.equal(x, y) for x, y in zip(*outs))
    for got, ref in zip(outs[0], orc.lstm_gate(Kbar, Vbar, kb.lstm_weights(w), 0, steps)):
        assert np.abs(got.cpu().numpy() - ref).max() <= 1e-6          # a handful of fp32 roundings per step


def test_nan_stays_in_its_sequence():
    """At rows held as pairs: a NaN makes its own sequence's scores NaN from its step on, and no other's."""
    cfg = base._cfg(433, "bf16", d=64, C=8, T=18 * 8, d_g=150, L=1, B=1, H=5)
    N = cfg.T // cfg.C
    gw = base.dev(synth.make_weights(cfg, "cpu"))
    Kbar, Vbar = (x.cuda() for x in base._summaries(cfg, N))
    Kbar[0, 0, 2, 3, 7] = float("nan")
    lead = (cfg.L, cfg.B, cfg.H)
    h, c = (torch.zeros(lead + (cfg.d_g,), device="cuda") for _ in range(2))
    util, gate = (torch.zeros(lead + (N,), device="cuda") for _ in range(2))
    kb.kvev_lstm_gate(kb.make_shape(cfg, N_cap=N), Kbar, Vbar, kb.lstm_weights(gw), 0, N, h, c, util, gate, None)
    torch.cuda.synchronize()
    bad = torch.zeros(lead + (N,), dtype=torch.bool, device="cuda")
    bad[0, 0, 2, 3:] = True
    assert torch.equal(util.isnan(), bad) and torch.equal(gate.isnan(), bad)
    assert torch.equal(h.isnan().any(-1), bad[..., -1]) and torch.equal(c.isnan().any(-1), bad[..., -1])
