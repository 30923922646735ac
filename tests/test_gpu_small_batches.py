"""Scoring and refresh plan of small batches on both sides of the lines where their launches change, against the oracles,
bit for bit."""
import numpy as np
import pytest

from tests.test_gpu_parity import _check_plan, _plan_gpu, _plan_inputs, _plan_oracle, _score_case, cs, say   # noqa: F401

pytestmark = pytest.mark.gpu

PLAN_CASES = [
    # streams, window, stride, T, n_text, p_iframe, p_empty, slack
    (1, 1, 1, 9, 0, 0.0, 0.0, 0),                 # one frame, nothing overlaps
    (1, 24, 23, 11, 3, 0.3, 0.1, 1),              # the widest window of one launch, one overlap frame
    (3, 24, 1, 20, 5, 0.2, 0.2, 1025),            # padding past one workgroup's share
    (3, 25, 1, 20, 5, 0.2, 0.2, 1025),            # ... and the first of three launches
    (256, 5, 1, 6, 2, 0.2, 0.1, 3),               # 1,024 overlap frames of 256 streams
    (257, 4, 1, 6, 2, 0.2, 0.1, 3),
    (60, 20, 1, 5, 1, 0.2, 0.3, 0),               # more than 1,024 overlap frames
    (65, 12, 4, 30, 7, 0.2, 0.1, 0),              # the streams of the first workgroup in two waves
    (130, 8, 8, 12, 1, 0.3, 0.2, 100),            # stride = window
]


@pytest.mark.parametrize("case", range(len(PLAN_CASES)))
def test_plan_refresh_lines(cs, case):
    n_streams, window, stride, t_per, n_text, p_i, p_e, slack = PLAN_CASES[case]
    say(f"plan_refresh line {case}: streams={n_streams} W={window} S={stride} T={t_per} text={n_text}")
    ins = _plan_inputs(np.random.default_rng(7300 + case), n_streams, window, stride, t_per, n_text, p_i, p_e)
    want = _plan_oracle(*ins, n_text, t_per)
    reuse_cap, q_cap = int(want["src_slot"].size) + slack, int(want["q_pos"].size) + slack
    _check_plan(_plan_gpu(cs, *ins, n_text, t_per, reuse_cap, q_cap), want, *ins[:4], reuse_cap, q_cap)


@pytest.mark.parametrize("n_streams", [6, 257])
def test_plan_refresh_old_table_too_short(cs, n_streams):
    """Reused rows whose old slot has no table entry are dropped and flagged, in one launch as in three."""
    say(f"plan_refresh: old block table too short, {n_streams} streams")
    n_text, t_per = 8, 32
    ins = _plan_inputs(np.random.default_rng(7400), n_streams, 8, 1, t_per, n_text, 0.15, 0.0)
    want = _plan_oracle(*ins, n_text, t_per)
    n_reuse, n_q = int(want["src_slot"].size), int(want["q_pos"].size)
    old_types, old_counts, new_types, new_counts, bt_old, bt_new = ins
    got = _plan_gpu(cs, old_types, old_counts, new_types, new_counts, bt_old[:, :2].copy(), bt_new, n_text, t_per, n_reuse, n_q)
    assert got["totals"].tolist() == [n_reuse, n_q, 4, 0]
    assert np.array_equal(got["q_slot"][:n_q], want["q_slot"])
    lost = got["src_slot"][:n_reuse] < 0
    assert lost.any() and np.all(got["dst_slot"][:n_reuse][lost] == -1)
    assert np.array_equal(got["src_slot"][:n_reuse][~lost], want["src_slot"][~lost])
    assert np.array_equal(got["dst_slot"][:n_reuse][~lost], want["dst_slot"][~lost])


SCORE_CASES = [
    # streams, frames per stream, grid, group
    (5, [1] * 5, (16, 16), 1),
    (16, [1] * 16, (16, 16), 1),                  # a stream a wave: the most of one workgroup
    (17, [1] * 17, (16, 16), 1),
    (16, [2] * 16, (16, 16), 1),                  # 32 sweeps
    (16, [2] * 15 + [3], (16, 16), 1),
    (15, [1] * 15, (7, 9), 1),                    # patch counts that are odd
    (6, [0, 32, 0, 0, 0, 0], (5, 5), 1),          # all work in one wave, to its last kept ballot word
    (6, [0, 30, 0, 0, 1, 1], (16, 16), 1),
    (6, [1] * 6, (26, 46), 1),                    # five sweeps a frame
    (7, [1] * 7, (26, 46), 1),
    (10, [1, 0] * 5, (32, 32), 2),                # group 2: tiles of four waves
]


@pytest.mark.parametrize("case", range(len(SCORE_CASES)))
def test_score_compact_lines(cs, case):
    n_streams, fps, (gh, gw), g = SCORE_CASES[case]
    say(f"score_compact line {case}: streams={n_streams} frames={sum(fps)} grid={gh}x{gw} g={g}")
    _score_case(cs, np.random.default_rng(7500 + case), n_streams, fps, gh, gw, g, 150, 800, True, True, case % 2 == 0)
