"""The per-utterance select kernel (more than 2048 groups in a batch) in every form that the host picks: lanes per new
hypothesis by the window, waves by the beam; the batch-wide window's shares among them.  Against the oracle, step by step
(tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


# 16, 32 and 64 lanes by the window's margins; 4, 8 and 16 waves by the beam; absent windows of more than one pass (512
# frames), and, for the batch-wide window, every utterance followed by the oracle: it couples them
# (batch-wide: the longest utterance says how wide it can be, 60, 200 and 300 frames for the three)
@pytest.mark.parametrize("window", [(12, 12, 0), (80, 80, 0), (-1, -1, 0), (5, 20, 60), (5, 20, 200), (4, -1, 300)])
@pytest.mark.parametrize("beam", [3, 7, 12, 32])
def test_per_utterance_select(beam, window):
    U = 2048 // beam + 1
    lens = np.array([14 + u % 5 for u in range(U)], np.int32)
    lens[[1, U // 2, U - 1]] = [600, 90, 1100] if window[2] == 0 else [window[2], 0, 45]
    w = gen.workload("cfg1")
    w.update(n_utt=U, vocab=24, beam=beam, cand_k=8, win_m1=window[0], win_m2=window[1], win_union=int(window[2] > 0), end_flags=3,
             max_len_ratio=0.0, max_len_abs=8)
    w["eos_id"] = w["vocab"] - 1
    ctc = gen.workload_ctc(w, np.maximum(lens, 1))
    check = [u for u in range(U) if lens[u] > 0] if window[2] else [0, 1, U // 2, U - 2, U - 1]
    rep, res = lockstep_decode(w, ctc, lens, check_utts=check, max_steps=5)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
    assert rep["utt_steps"] >= 4 * len(check)
