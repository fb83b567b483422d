"""How the recurrent gate (bf16, Eq. 3) uses the scratch it is given: the form and the steps per launch, as the library plans them
(no GPU needed)."""
import pytest

from paper_2509_21354_amd import binding as kb


def _shape(d_g, L=1, BH=1, N_cap=64, d=128):
    return kb.make_shape(L=L, B=1, H=BH, d=d, T=N_cap, T_cap=N_cap, C=1, N_cap=N_cap, W=0, d_sum=32, d_g=d_g, dtype=kb.BF16, H_kv=0)


def _fixed(shape):
    """scratch that does not grow with the steps (prepared weights), and what a step adds"""
    one, two = (kb.workspace_bytes(kb.OP_LSTM_GATE_PREPARED, shape, n) for n in (17, 18))
    return one - 17 * (two - one), two - one


@pytest.mark.parametrize("d_g", [64, 128, 256, 512])
@pytest.mark.parametrize("BH", [1, 16])
def test_projections_of_a_launch_stay_within_32_bits(d_g, BH):
    """The recurrence addresses the projections of a group of 16 sequences with 32 bits: a launch takes fewer steps than overflow
    them, however much scratch there is."""
    sh = _shape(d_g, BH=BH, N_cap=1 << 20)
    fixed, step = _fixed(sh)
    workgroups, block = kb.kvev_debug_lstm_plan(sh, True, 1 << 20, fixed + (step << 20))
    assert step == 16 * 4 * d_g * 4 and workgroups != 4
    assert 4096 <= block and block * step < 1 << 32
    assert block // 2 + 4096 < 1 << 16           # rows of the projection's grid: two steps each at least, and those that re-lay weights
    assert kb.kvev_debug_lstm_plan(sh, True, 1 << 20, fixed + 100 * step)[1] == 100
    assert kb.kvev_debug_lstm_plan(sh, True, 5, fixed + 100 * step)[1] == 5
    assert kb.kvev_debug_lstm_plan(sh, True, 5, step)[1] == 0


@pytest.mark.parametrize("L,BH", [(1, 1), (1, 16), (3, 13), (32, 16), (1, 17), (2, 64), (1, 512)])
@pytest.mark.parametrize("n", [1, 2, 8, 128])
@pytest.mark.parametrize("prepared", [False, True])
def test_scratch_serves_caches_of_other_capacities(L, BH, n, prepared):
    """d_g = 512 takes other forms for short caches: scratch that was asked for with one capacity is accepted with any."""
    op = kb.OP_LSTM_GATE_PREPARED if prepared else kb.OP_LSTM_GATE
    for asked in (1, 15, 16, 256):
        nbytes = kb.workspace_bytes(op, _shape(512, L, BH, asked), n)
        for used in (1, 15, 16, 256):
            assert kb.kvev_debug_lstm_plan(_shape(512, L, BH, used), prepared, used, nbytes)[1] >= min(n, used)


@pytest.mark.parametrize("L,BH,least", [(1, 512, 12), (15, 17, 12), (2, 256, 12), (1, 256, 6), (8, 32, 6), (1, 17, 6), (1, 16, 1), (32, 16, 1)])
def test_eight_workgroups_take_scratch_of_a_useful_block(L, BH, least):
    """d_g = 512: the form that begins every launch with all of W_hh from memory is taken when the scratch holds enough steps per
    launch, whatever the steps of a call; with less, four workgroups in one launch.  The query always answers enough."""
    sh = _shape(512, L, BH, N_cap=256)
    groups = L * ((BH + 15) // 16)
    fixed, step = 256 + groups * 65536, groups * 131072
    for steps in (1, 5, 64):
        for held in (1, 2, 5, 6, 11, 12, 64):
            workgroups, block = kb.kvev_debug_lstm_plan(sh, True, steps, fixed + held * step)
            assert (workgroups, block) == ((8, min(held, steps)) if held >= least else (4, steps))
    for n in (0, 1, 2, 8, 64):
        assert kb.kvev_debug_lstm_plan(sh, True, 64, kb.workspace_bytes(kb.OP_LSTM_GATE_PREPARED, sh, n))[0] == 8


@pytest.mark.parametrize("d_g,L,BH,steps,form", [
    (164, 1, 32, 1, "kept"), (164, 1, 32, 100, "kept"), (164, 1, 512, 1, "four"), (164, 1, 512, 32, "kept"), (164, 1, 1024, 32, "four"),
    (192, 1, 8192, 1, "four"), (192, 1, 8192, 500, "four"), (160, 300, 2, 1, "four"), (160, 300, 2, 8, "kept"), (160, 1024, 1, 1, "kept"),
    (163, 1, 32, 1, "one"), (163, 1, 32, 2, "kept"), (163, 1, 512, 1, "four"), (163, 1, 512, 8, "kept"), (163, 1, 1024, 8, "four"),
    (163, 1, 1024, 32, "kept"), (129, 1, 8192, 2, "four"), (163, 300, 1, 8, "kept"), (193, 1, 32, 8, "one"), (200, 1, 512, 8, "four")])
def test_rows_are_kept_where_there_are_steps_to_pay_for_it(d_g, L, BH, steps, form):
    """bf16, 129 to 192 units: a workgroup that keeps its rows in registers serves one sequence and starts with all of them; short
    calls of many sequences read them every step for four."""
    sh = kb.make_shape(L=L, B=1, H=BH, d=128, T=512, T_cap=512, C=1, N_cap=512, W=0, d_sum=32, d_g=d_g, dtype=kb.BF16, H_kv=0)
    assert kb.kvev_debug_lstm_form(sh, steps) == form
