"""More than 64 candidates per hypothesis: the score kernel's forms for them (narrow and wider windows, whole utterances of less than one
round of loads to several), the last round of candidates full, nearly empty and between, the eos-run rule's two-part sums, more
candidates than lanes.  Against the oracle, step by step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode, peaked_ctc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [65, 96, 128, 253, 254, 255, 256, 257, 300])
@pytest.mark.parametrize("window,lens", [((12, 12), [90, 41]), ((80, 80), [310, 150]), ((-1, -1), [520, 255, 64]), ((200, 130), [700, 260])])
@pytest.mark.parametrize("rule", [dict(end_flags=3), dict(end_flags=7, eos_run=10)])
def test_many_candidates(k, window, lens, rule):
    w = gen.workload("cfg1")
    w.update(n_utt=len(lens), vocab=1500, beam=4, cand_k=k, win_m1=window[0], win_m2=window[1], **rule)
    w["eos_id"] = w["vocab"] - 1
    lens = np.asarray(lens, np.int32)
    ctc = gen.workload_ctc(w, lens)
    peaked_ctc(ctc, 20)
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=5)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
