"""Order of a group's candidate list, at every form of its construction: by the joint score as the fp64 it is, equal scores by
token id.  The first step's selection from hand-made posteriors and attention rows, where the order is known."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (vocab, candidates): every id (the score kernel's own list up to 66 ids, then the matrix form: the best of all pairs, no lists), restricted
# sets of more than one wave's and more than one work-group's: 4, 20 and 32 scores per lane, and those beyond 8192, read for each pass
FORMS = [(40, 0), (66, 0), (67, 0), (1000, 0), (4000, 0), (8194, 0), (8195, 0), (16386, 0), (16387, 0), (20001, 0), (200, 100), (400, 300), (5000, 4000), (9001, 7000), (9001, 8500)]


def first_step(vocab, cand_k, att, ctc, beam=4):
    import torch
    import paper_2101_05600_amd as m
    cfg = m.make_config(n_utt=1, t_max=ctc.shape[0], vocab=vocab, beam=beam, cand_k=cand_k, ctc_weight=0.5, keep_candidates=0)
    h = m.ctcbs_create(cfg, torch.from_numpy(ctc[None]).cuda(), np.array([ctc.shape[0]], np.int32))
    try:
        rows = torch.full((1, beam, vocab), float("nan"), device="cuda")
        rows[0, 0] = torch.from_numpy(att).cuda()
        out = m.StepOut()
        assert m.ctcbs_step(h, rows, out) == m.OK
        return m.view(out.d_token, (1, beam), np.int32).cpu().numpy()[0].tolist()
    finally:
        m.ctcbs_destroy(h)


def posteriors(vocab, ids, value=-3.0):
    ctc = np.full((6, vocab), -30.0, np.float32)
    ctc[:, 0] = -0.5
    ctc[:, ids] = value
    return ctc


@pytest.mark.parametrize("vocab,cand_k", FORMS)
def test_scores_that_agree_in_forty_bits_are_told_apart(vocab, cand_k):
    """Four ids with the same posteriors whose attention values differ by one unit in the last place of 2^-20: joint
    scores around -5 that differ by 6e-14, 2^-46 of them (fp64 holds 2^-52)."""
    ids = np.array([5, 17, vocab // 2, vocab - 3])
    att = np.full(vocab, -20.0, np.float32) - np.arange(vocab, dtype=np.float32) * np.float32(1e-3)
    v = np.float32(-2.0 ** -20)
    order = [2, 0, 3, 1]
    for place in order:
        att[ids[place]] = v
        v = np.nextafter(v, np.float32(-1.0))
    assert first_step(vocab, cand_k, att, posteriors(vocab, ids)) == [int(ids[i]) for i in order]


@pytest.mark.parametrize("vocab,cand_k", FORMS)
def test_equal_scores_go_by_id(vocab, cand_k):
    """A few equal scores, and all of them equal (more than the packed list holds, from 512 on: round by round)."""
    ids = np.array([9, 10, vocab // 2, vocab - 2])
    att = np.full(vocab, -20.0, np.float32)
    att[ids] = -1.0
    assert first_step(vocab, cand_k, att, posteriors(vocab, ids)) == ids.tolist()
    flat = np.full(vocab, -2.0, np.float32)
    ctc = posteriors(vocab, np.arange(1, vocab))
    assert first_step(vocab, cand_k, flat, ctc) == [1, 2, 3, 4]
    # two levels: the better ones are fewer than the beam
    flat[[vocab - 2, 7]] = -1.9
    assert first_step(vocab, cand_k, flat, ctc) == [7, vocab - 2, 1, 2]


# whole steps against the oracle where the scores are read again for each pass
@pytest.mark.parametrize("vocab,cand_k", [(16387, 0), (17003, 0), (9001, 7000), (9001, 8500)])
def test_many_candidates_against_the_oracle(vocab, cand_k):
    import gen
    from helpers import lockstep_decode
    w = gen.workload("cfg1")
    w.update(n_utt=2, t_lo=25, t_hi=40, vocab=vocab, beam=5, cand_k=cand_k, win_m1=-1, win_m2=-1, end_flags=3)
    w["eos_id"] = vocab - 1
    lens = gen.workload_lengths(w)
    rep, _ = lockstep_decode(w, gen.workload_ctc(w, lens), lens, max_steps=4)
    assert rep["max_ctc_err"] < 1e-4 and rep["max_score_err"] < 1e-4 and rep["utt_steps"] == 8
