"""Short lists of more than 64 entries (about 1.2 times the number of candidates): two entries per lane; equal values at the K-th place,
which send the ranking to the work-group, rows that do not start or end on a 16-byte boundary, raw scores.  Against the oracle, step by
step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [48, 53, 60, 63, 64])
@pytest.mark.parametrize("vocab", [1027, 5000, 9001])
@pytest.mark.parametrize("window,grid", [((12, 12), 0), ((80, 80), 16), ((-1, -1), 4)])   # (grid: attention values to its inverse)
def test_short_list_of_two_entries_per_lane(k, vocab, window, grid):
    w = gen.workload("cfg1")
    w.update(n_utt=2, vocab=vocab, beam=4, cand_k=k, win_m1=window[0], win_m2=window[1], end_flags=3)
    w["eos_id"] = w["vocab"] - 1
    lens = np.array([230, 60], np.int32)
    ctc = gen.workload_ctc(w, lens)
    kw = dict(att_fn=lambda a: (np.round(a * grid) / grid).astype(np.float32)) if grid else {}
    rep, _ = lockstep_decode(w, ctc, lens, max_steps=5, **kw)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4
