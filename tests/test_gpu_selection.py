"""Candidate selection of the score kernel at the sizes where its forms change: registers per lane for the row, rows
that do not start or end on a 16-byte boundary, rows with fewer granules than lanes, short lists of more than 64 entries,
equal values at the K-th place.  Against the oracle, step by step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


def _decode(steps=5, att_fn=None, **over):
    w = gen.workload("cfg1")
    w.update(dict(n_utt=2, t_lo=30, t_hi=60, beam=3, cand_k=40, win_m1=12, win_m2=12, end_flags=7, eos_run=3), **over)
    w["eos_id"] = w["vocab"] - 1
    lens = gen.workload_lengths(w)
    rep, _ = lockstep_decode(w, gen.workload_ctc(w, lens), lens, max_steps=steps, att_fn=att_fn)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
    assert rep["utt_steps"] == 2 * steps


# edges of the forms (3, 5, 10 and 16 granules of four ids per lane, 256 lanes; no form beyond), and rows of every
# alignment (the row of slot j starts at j * V)
@pytest.mark.parametrize("vocab", [3072, 3073, 5003, 5120, 5121, 10240, 10241, 16384, 16385])
def test_row_sizes(vocab):
    _decode(vocab=vocab, steps=3)


# fewer granules than lanes: whole waves without any, a wave with a few; about as many as candidates; hardly any
@pytest.mark.parametrize("vocab,k", [(1023, 40), (777, 64), (270, 60), (165, 40), (45, 40), (9, 3)])
def test_small_rows(vocab, k):
    _decode(vocab=vocab, cand_k=k)


# short lists around and beyond what one wave holds
@pytest.mark.parametrize("k", [1, 2, 44, 52, 60, 64, 65, 128])
def test_list_sizes(k):
    _decode(vocab=4001, cand_k=k, steps=4)


# values that are equal at the K-th place (rounded to 1/8), few enough of them for the short list
def test_equal_values_at_the_last_place():
    _decode(vocab=1200, cand_k=33, att_fn=lambda a: np.where(np.isnan(a), a, np.round(a * 8) / 8).astype(np.float32))


# one value far above the rest: the pivot lies beyond the linear scale of the bisection
def test_values_far_below_the_best():
    def spread(a):
        return np.where(np.isnan(a), a, np.where(a > np.nanmax(a, axis=-1, keepdims=True) - 1e-6, a, a * 8 - 40)).astype(np.float32)
    _decode(vocab=2000, att_fn=spread)


# rows on another scale than log-probabilities: above zero, far below it, on both sides of it, and spread so far that the last candidate
# lies far below the best
@pytest.mark.parametrize("scale,shift", [(1.0, 40.0), (1.0, -60.0), (1.0, 9.0), (6.0, 50.0)])
@pytest.mark.parametrize("over", [dict(vocab=2000), dict(vocab=777, cand_k=64)])
def test_rows_on_another_scale(scale, shift, over):
    _decode(steps=4, att_fn=lambda a: (a * np.float32(scale) + np.float32(shift)).astype(np.float32), **over)


# ids that the decoder masks with -inf: fewer numbers in a row than candidates (masked ids of the lowest numbers fill the list,
# each once), in rows of every alignment
@pytest.mark.parametrize("vocab", [45, 61, 270, 1203, 5003])
@pytest.mark.parametrize("k", [30, 64, 80])
def test_masked_ids(vocab, k):
    def masked(a):
        some = np.arange(vocab) % (vocab // 20) == 1
        return np.where(np.isnan(a) | some, a, np.float32(-np.inf))
    _decode(vocab=vocab, cand_k=min(k, vocab - 5), att_fn=masked)
