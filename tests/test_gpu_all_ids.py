"""Every id a candidate: the matrix form of the prefix scores and the list builder, at the edges of their tiles (16
candidates, 16 slots, 16-frame blocks, chunks of 64 candidates for large batches) and where a sum leaves the range of
the product.  Against the oracle, step by step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


def _decode(steps=5, check=None, lens=None, edit=None, **over):
    w = gen.workload("cfg1")
    w.update(dict(n_utt=2, t_lo=30, t_hi=60, beam=3, cand_k=0, win_m1=-1, win_m2=-1, end_flags=3), **over)
    w["eos_id"] = w["vocab"] - 1
    lens = gen.workload_lengths(w) if lens is None else np.asarray(lens, np.int32)
    ctc = gen.workload_ctc(w, lens)
    if edit is not None:
        edit(ctc)
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=steps, check_utts=check)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4


# (66 and 67 ids: k_score still / the matrix form with one candidate beyond a whole number of tiles)
@pytest.mark.parametrize("vocab", [66, 67, 81, 82, 83, 1026, 1027, 5122, 5123, 8194, 8195])
def test_candidate_tiles(vocab):
    _decode(vocab=vocab, steps=3)


@pytest.mark.parametrize("beam", [1, 15, 16, 17, 32])
def test_slot_tiles(beam):
    _decode(vocab=130, beam=beam)


@pytest.mark.parametrize("frames", [1, 2, 15, 16, 17, 31, 33, 257, 1600])
def test_frame_blocks(frames):
    _decode(vocab=100, lens=[frames, max(1, frames - 1)], steps=min(4, frames))


def test_windows_of_the_slots_together():
    _decode(vocab=150, beam=6, t_lo=120, t_hi=300, win_m1=9, win_m2=14, steps=20)


# 64 candidates per work-group (chunks x utterances >= 512), an unused slot among them
def test_large_batch():
    _decode(vocab=700, n_utt=50, beam=4, lens=[40 + u % 7 if u != 5 else 0 for u in range(50)], check=[0, 6, 49], steps=3)


# ids that never occur, and ids so unlikely that every product of their sums underflows: log0 / redone frame by frame
@pytest.mark.parametrize("value", [-np.inf, -95.0])
def test_sums_beyond_the_range_of_the_product(value):
    def edit(ctc):
        ctc[:, :, 40:47] = value
    _decode(vocab=90, edit=edit)
