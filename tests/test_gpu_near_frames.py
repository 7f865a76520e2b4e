"""The score kernel over wide windows: sums over the frames near a hypothesis's last label, the others where they can count.
Against the oracle, step by step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode, peaked_ctc

pytestmark = pytest.mark.gpu


def _decode(edit, lens, steps=12, **over):
    w = gen.workload("cfg1")
    w.update(dict(n_utt=len(lens), vocab=300, beam=4, cand_k=40, win_m1=-1, win_m2=-1, end_flags=3), **over)
    w["eos_id"] = w["vocab"] - 1
    lens = np.asarray(lens, np.int32)
    ctc = gen.workload_ctc(w, np.maximum(lens, 1))
    edit(ctc)
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=steps, check_utts=[u for u in range(len(lens)) if lens[u] > 0])
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4


# every: frames between labels, so that few frames, about one round of loads (128 frames) or several are near
@pytest.mark.parametrize("every,lens", [(4, [300, 129]), (33, [500, 131]), (90, [700, 0, 257]), (5, [1500])])
@pytest.mark.parametrize("over", [{}, dict(end_flags=7, eos_run=10), dict(win_m1=200, win_m2=170), dict(win_m1=30, win_m2=60, win_union=1),
                                  dict(cand_k=64, beam=13), dict(cand_k=1), dict(cand_k=30), dict(cand_k=49)])
def test_peaked_posteriors(every, lens, over):
    _decode(lambda c: peaked_ctc(c, every), lens, **over)


# so sharp that most candidates lie tens of nats down where a label is near: frames on both sides of the near ones count.  (Height h: the
# stored variables step by 2 h from frame to frame; a rounding of half a unit in the last place of 120 for each of a few operations of
# 12 labels stays below 2e-5 root mean square)
@pytest.mark.parametrize("height,every", [(30.0, 7), (30.0, 60), (60.0, 3), (60.0, 20)])
@pytest.mark.parametrize("over", [{}, dict(end_flags=7, eos_run=10), dict(win_m1=100, win_m2=70), dict(win_m1=80, win_m2=80, end_flags=7, eos_run=4),
                                  dict(cand_k=64, beam=13), dict(cand_k=1), dict(cand_k=0, vocab=60), dict(vocab=6000)])
def test_sharp_posteriors(height, every, over):
    _decode(lambda c: peaked_ctc(c, every, height), [520, 131], **over)


# utterances about as long as the forms for narrow windows hold (128 frames from a multiple of four on): whole, wide margins, a batch-wide window
@pytest.mark.parametrize("longest", [124, 125, 126, 129])
@pytest.mark.parametrize("over", [{}, dict(end_flags=7, eos_run=10), dict(win_m1=200, win_m2=170), dict(win_m1=90, win_m2=60, win_union=1),
                                  dict(cand_k=0, vocab=60), dict(beam=13)])
def test_longest_utterance_of_the_narrow_forms(longest, over):
    _decode(lambda c: peaked_ctc(c, 9), [longest, longest - 1, 30], **over)


# the large batches' select kernel, its three widths of a new hypothesis: a wave (windows beyond 256 frames), 32 lanes, 16 (up to 128 frames,
# where no near frames are looked for)
@pytest.mark.parametrize("over", [{}, dict(win_m1=100, win_m2=100), dict(win_m1=50, win_m2=60)])
def test_large_batch(over):
    w = gen.workload("cfg1")
    w.update(dict(n_utt=300, vocab=120, beam=8, cand_k=20, win_m1=-1, win_m2=-1, end_flags=3), **over)
    w["eos_id"] = w["vocab"] - 1
    lens = np.asarray([250 + u % 11 for u in range(300)], np.int32)
    ctc = gen.workload_ctc(w, lens)
    peaked_ctc(ctc, 6)
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=8, check_utts=[0, 10, 299])
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4


# candidates so unlikely that the frames left out could count, some of them impossible; values that are no log-probabilities, whose
# far frames outweigh the near ones
@pytest.mark.parametrize("value", [-70.0, -np.inf, "far", "above0"])
@pytest.mark.parametrize("over", [{}, dict(end_flags=7, eos_run=10)])
def test_frames_that_are_not_near_count(value, over):
    def edit(ctc):
        peaked_ctc(ctc, 5, ids=np.arange(150, 280))
        if value == "far":                                   # likely at the far end alone
            ctc[:, :, 1:140] = -60.0
            ctc[:, -9:, 1:140] = -0.5
        elif value == "above0":
            ctc += 3.0
            ctc[:, -9:, 1:140] = 45.0
        else:
            ctc[:, :, 1:140] = value
    _decode(edit, [300, 171], **over)
