"""Every id a candidate: the best of all (slot, candidate) pairs from the best of each chunk of 16 or 32 candidates.  Fewer chunks than
beam slots, about as many chunks as the lanes hold (4096 entries of a beam's slots and one more, or none, per chunk; 1986 ids, beam 32: 124 chunks of 16; 1987 ids: one more,
so chunks of 32), more of them, numbers of ids that are powers of two, posteriors
and attention rows that are the same for most ids (more chunks reach the pivot than fit, equal scores go by slot and id), one work-group per slot and one per utterance.  Against the oracle, step by step (tolerances
as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,beam,utts", [(70, 32, 2), (530, 32, 2), (1300, 3, 2), (2100, 20, 2), (9001, 32, 2), (2050, 32, 2), (2051, 32, 2), (1986, 32, 2), (1987, 32, 2), (1024, 20, 2), (4096, 20, 2), (4096, 32, 2), (1300, 3, 690), (90, 32, 70)])
@pytest.mark.parametrize("same", [0, 3])                     # ids that differ from the others (0: all do)
def test_best_of_all_pairs(vocab, beam, utts, same):
    w = gen.workload("cfg1")
    w.update(n_utt=utts, vocab=vocab, beam=beam, cand_k=0, win_m1=-1, win_m2=-1, end_flags=3, max_len_ratio=0.0, max_len_abs=6)
    w["eos_id"] = w["vocab"] - 1
    lens = np.array([9 + 5 * (u % 3 == 0) for u in range(utts)], np.int32)
    ctc = gen.workload_ctc(w, lens)
    kw = {}
    if same:
        ctc[:, :, 1 + same:] = ctc[:, :, 1 + same:2 + same]
        kw = dict(att_fn=lambda a: np.where(np.isnan(a), a, np.where(np.arange(vocab) < 1 + same, a, np.float32(-9.0))).astype(np.float32))
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=4, check_utts=[0, 1, utts - 1] if utts > 2 else None, **kw)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4


# scores far below zero, whose upper halves lie close together (how many chunks reach the pivot there: tests/test_kernel_units.py)
def test_scores_far_below_zero():
    w = gen.workload("cfg1")
    w.update(n_utt=2, vocab=3001, beam=20, cand_k=0, win_m1=-1, win_m2=-1, end_flags=3, max_len_ratio=0.0, max_len_abs=6)
    w["eos_id"] = w["vocab"] - 1
    lens = np.array([24, 19], np.int32)
    rep, _ = lockstep_decode(w, gen.workload_ctc(w, lens), lens, max_steps=4, att_fn=lambda a: (a - np.float32(128.0)).astype(np.float32))
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
