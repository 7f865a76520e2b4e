"""Every id a candidate: the matrix form of the prefix scores, at the edges of its tiles (16
candidates, 16 slots, 16-frame blocks, chunks of 32 candidates for large batches) and where a sum leaves the range of
the product.  Against the oracle, step by step (tolerances as in test_gpu_parity.py)."""
import numpy as np
import pytest

import gen
from helpers import lockstep_decode, peaked_ctc

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


@pytest.mark.parametrize("frames", [1, 2, 15, 16, 17, 31, 33, 256, 257, 258, 1600])
def test_frame_blocks(frames):
    _decode(vocab=100, lens=[frames, max(1, frames - 1)], steps=min(4, frames))


def test_windows_of_the_slots_together():
    _decode(vocab=150, beam=6, t_lo=120, t_hi=300, win_m1=9, win_m2=14, steps=20)


# 32 candidates per work-group (chunks x utterances >= 1024), an unused slot among them
def test_large_batch():
    _decode(vocab=700, n_utt=50, beam=4, lens=[40 + u % 7 if u != 5 else 0 for u in range(50)], check=[0, 6, 49], steps=3)


# ids that never occur, and ids so unlikely that every product of their sums underflows: log0 / redone frame by frame
@pytest.mark.parametrize("value", [-np.inf, -95.0])
def test_sums_beyond_the_range_of_the_product(value):
    def edit(ctc):
        ctc[:, :, 40:47] = value
    _decode(vocab=90, edit=edit)


# posteriors that are all but certain of a label every few frames: a hypothesis has terms for a short stretch of frames only (the
# rest underflows against the largest), which moves along the utterance and is read alone; rows end inside a block of frames
@pytest.mark.parametrize("every,lens,over", [(5, [330, 199], {}), (3, [129, 64], dict(beam=17)), (40, [300, 161], {}), (5, [200, 97], dict(win_m1=60, win_m2=30))])
def test_short_stretches_of_frames(every, lens, over):
    _decode(**dict(dict(vocab=100, beam=5, lens=lens, edit=lambda c: peaked_ctc(c, every), steps=14), **over))


# candidates so unlikely that the frames left out at first count, likely at the far end alone, and values that are no
# log-probabilities; 16 and 32 candidates, one and two tiles of slots per work-group
@pytest.mark.parametrize("value", [-30.0, -70.0, "far", "above0"])
@pytest.mark.parametrize("over", [{}, dict(beam=17), dict(beam=17, n_utt=50, vocab=700), dict(n_utt=50, vocab=700)])
def test_frames_left_out_count(value, over):
    n = over.get("n_utt", 2)

    def edit(ctc):
        peaked_ctc(ctc, 5, ids=np.arange(50, 90))
        if value == "far":
            ctc[:, :, 1:45] = -60.0
            ctc[:, -9:, 1:45] = -0.5
        elif value == "above0":
            ctc += 3.0
            ctc[:, -9:, 1:45] = 45.0
        else:
            ctc[:, :, 1:45] = value
    _decode(**dict(dict(vocab=100, beam=4, lens=[300 - 3 * u for u in range(n)], edit=edit, steps=6, check=[0, n - 1]), **over))


# candidates can be looked at without keep_candidates: the score kernel's own list, the matrix form, sets through memory
@pytest.mark.parametrize("vocab,over", [(40, {}), (40, dict(end_flags=7, eos_run=3)), (100, {}), (100, dict(win_union=1)), (700, {}), (9001, {}), (400, dict(cand_k=300))])
def test_peek_without_keep_candidates(vocab, over):
    import torch
    import paper_2101_05600_amd as m
    U, Wb, T = 2, 3, 40
    g = torch.Generator(device="cuda").manual_seed(3)
    ctc = torch.log_softmax(2 * torch.randn((U, T, vocab), generator=g, device="cuda"), -1)
    ctc[0, :, 11] = float("-inf")
    att = torch.log_softmax(2 * torch.randn((U, Wb, vocab), generator=g, device="cuda"), -1)
    got = []
    for keep in (0, 1):
        cfg = m.make_config(**dict(dict(n_utt=U, t_max=T, vocab=vocab, beam=Wb, blank_id=3, keep_candidates=keep, win_m1=20, win_m2=20), **over))
        h = m.ctcbs_create(cfg, ctc, np.array([T, T - 9], np.int32))
        try:
            for _ in range(3):
                assert m.ctcbs_step(h, att, None) == m.OK
            got.append([m.ctcbs_peek(h, w).copy() for w in (m.PEEK_CAND_ID, m.PEEK_CAND_CTC, m.PEEK_CAND_JOINT)])
        finally:
            m.ctcbs_destroy(h)
    K = vocab - 2 if "cand_k" not in over else over["cand_k"]
    for a, b in zip(*got):
        # (joint scores may be put together on the host: three fp64 roundings of values below 1e3)
        assert a.size == U * Wb * K and np.allclose(a, b, rtol=0, atol=1e3 * 3 * 2.0 ** -53 if a is got[0][2] else 0)
    if "cand_k" not in over:
        assert np.array_equal(got[0][0].reshape(U * Wb, K)[0], [i for i in range(vocab) if i not in (3, vocab - 1)])


# slots are prepared for the next step where the select kernel makes them (2048 groups at most): of an utterance that finishes, of one
# that goes on beside it, and, with more groups, by a launch
@pytest.mark.parametrize("utts", [2, 690])
def test_a_finished_utterance_beside_others(utts):
    import torch
    import paper_2101_05600_amd as m
    Wb, T, V = 3, 24, 100
    lens = np.full(utts, T, np.int32)
    lens[0] = 2
    g = torch.Generator(device="cuda").manual_seed(5)
    ctc = torch.log_softmax(2 * torch.randn((1, T, V), generator=g, device="cuda"), -1).expand(utts, T, V).contiguous()
    att = torch.log_softmax(2 * torch.randn((utts, Wb, V), generator=g, device="cuda"), -1)
    h = m.ctcbs_create(m.make_config(n_utt=utts, t_max=T, vocab=V, beam=Wb, blank_id=0, win_m1=9, win_m2=9, max_len_ratio=1.0, end_flags=0, keep_candidates=0), ctc, lens)
    try:
        seen = []
        for _ in range(5):
            assert m.ctcbs_step(h, att, None) == m.OK
            seen.append([m.ctcbs_peek(h, w).reshape(utts, -1).copy() for w in (m.PEEK_WIN_S, m.PEEK_WIN_E, m.PEEK_CAND_CTC, m.PEEK_CAND_JOINT)])
    finally:
        m.ctcbs_destroy(h)
    s, e, ctc5, joint5 = seen[4]
    assert (s[0] == 0).all() and (e[0] == -1).all()
    for _, _, a, b in seen[2:]:                              # (what its last step, the second, left)
        assert np.array_equal(a[0], seen[1][2][0]) and np.array_equal(b[0], seen[1][3][0])
    assert (s[1:] >= 5).all() and (e[1:] <= T).all() and (e[1:] >= s[1:]).all() and (ctc5[1:] > -1e3).all() and (joint5[1:] > -1e3).all()


# A slot that holds no hypothesis any more, in an utterance that goes on, and a slot of an utterance that a later batch does not use: what their
# last step left, with and without keep_candidates (the same arithmetic on the host and on the GPU: to the last bit).
@pytest.mark.parametrize("utts", [2, 690])
def test_peek_at_slots_without_a_hypothesis(utts):
    import torch
    import paper_2101_05600_amd as m
    Wb, T, V = 3, 24, 100
    g = torch.Generator(device="cuda").manual_seed(8)
    ctc = torch.log_softmax(2 * torch.randn((1, T, V), generator=g, device="cuda"), -1).expand(utts, T, V).contiguous()
    rows = [torch.log_softmax(2 * torch.randn((utts, Wb, V), generator=g, device="cuda"), -1) for _ in range(5)]
    for k in (2, 3):                                         # from the third step on a single extension has a score
        rows[k] = torch.where(torch.arange(V, device="cuda") == 5, rows[k], float("-inf"))
        rows[k][:, 1:] = float("-inf")
    lens = np.full(utts, T, np.int32)
    last = utts - 1
    got = []
    for keep in (0, 1):
        h = m.ctcbs_create(m.make_config(n_utt=utts, t_max=T, vocab=V, beam=Wb, blank_id=0, max_len_ratio=1.0, end_flags=0, keep_candidates=keep), ctc, lens)
        try:
            seen = []
            peek = lambda: seen.append([m.ctcbs_peek(h, w).reshape(utts, Wb, V - 2).copy() for w in (m.PEEK_CAND_CTC, m.PEEK_CAND_JOINT)])
            for r in rows:
                assert m.ctcbs_step(h, r, None) == m.OK
                peek()
            used = lens.copy()
            used[last] = 0
            m.ctcbs_reset(h, ctc, used)
            for r in rows[:2]:
                assert m.ctcbs_step(h, r, None) == m.OK
                peek()
            got.append(seen)
        finally:
            m.ctcbs_destroy(h)
    for step, (a, b) in enumerate(zip(*got)):
        for x, y in zip(a, b):
            if step >= 1:                                    # (all slots have held a hypothesis)
                assert np.array_equal(x, y), step
    for seen in got:
        for k in (3, 4):
            for x, y in zip(seen[k], seen[2]):
                assert np.array_equal(x[:, 1:], y[:, 1:])    # dead from the fourth step on
        for k in (5, 6):
            for x, y in zip(seen[k], seen[4]):
                assert np.array_equal(x[last], y[last])
