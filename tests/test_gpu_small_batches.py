"""Batches about as large as the chip has compute units: up to 256 (utterance, beam slot) groups the score kernel fetches a row
before it knows whether the slot holds a hypothesis; numbers of utterances that are no multiple of eight."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


# (dead slots' rows hold NaN, see helpers.host_att)
@pytest.mark.parametrize("n_utt,beam", [(1, 1), (1, 10), (5, 3), (9, 4), (16, 16), (17, 15), (17, 16), (8, 32), (9, 32)])
@pytest.mark.parametrize("over", [{}, dict(vocab=403), dict(att_is_logits=1), dict(win_union=1)])
def test_small_batches(n_utt, beam, over):
    w = gen.workload("cfg1")
    w.update(dict(vocab=400, cand_k=20, win_m1=8, win_m2=12, end_flags=7, eos_run=4), n_utt=n_utt, beam=beam, **over)
    w["eos_id"] = w["vocab"] - 1
    lens = np.asarray([0 if u == 4 else 40 + 3 * u for u in range(n_utt)], np.int32)
    ctc = gen.workload_ctc(w, np.maximum(lens, 1))
    # (raw scores: log-probabilities are scores whose log_softmax they are themselves, to rounding)
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=6, check_utts=[u for u in range(n_utt) if lens[u] > 0])
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
