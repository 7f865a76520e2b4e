"""Rounding of the kernels' sums (and a rule of the host): functions on their own in the CPU build of the kernel sources (tests/cpu_emu), where
every operation is IEEE fp32 and exp2 / log2 are libm's: against 64-bit sums of the same fp32 inputs."""
import ctypes
import os
import re
import subprocess
import sys

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, os.path.join(HERE, "cpu_emu"))

import build_emu  # noqa: E402

vp = ctypes.c_void_p


@pytest.fixture(scope="module")
def units(tmp_path_factory):
    return ctypes.CDLL(build_emu.build(str(tmp_path_factory.mktemp("units")), sanitize=False, units=True))


def ptr(a):
    return a.ctypes.data_as(vp)


def chain(units, lpc, it, x, f):
    out = np.empty(len(x), np.float32)
    assert x.shape[1] % 4 == 0 and units.unit_chain(lpc, it, ptr(x), ptr(f), len(x), x.shape[1] // 4, ptr(out)) == 0
    return out.astype(np.float64)


def exact(x, f):
    v = x.astype(np.float64) + f.astype(np.float64)
    m = v.max(1)
    return m + np.log(np.exp(v - m[:, None]).sum(1)), v


# One rounding per term and one of the result, two of the logarithm of what the terms add up to, at most one per addition on a
# term's way into that (2 IT per round and log2 LPC between lanes, 2^-23 of the sum each), and nothing else: an error e_t
# of a term reaches the sum as w_t e_t, w_t the term's share of it; spread evenly over one unit in the last place it is
# ulp / sqrt(12) rms.  400 sums: the rms itself is known to 4 %, and three times that is allowed.  (Terms
# scaled to units of log 2 lie 1.3 to 1.4 times higher.)
@pytest.mark.parametrize("lpc,it,rounds", [(16, 2, 1), (16, 3, 1), (16, 4, 2), (64, 4, 1)])
@pytest.mark.parametrize("magnitude", [5.0, 40.0, 300.0])
def test_prefix_sums_round_a_term_once(units, lpc, it, rounds, magnitude):
    rng = np.random.default_rng(int(magnitude) + lpc + it)
    n, T = 400, 4 * lpc * it * rounds
    x = -rng.gamma(2.0, 2.0, (n, T)).astype(np.float32) - np.float32(magnitude * rng.random((n, 1)))
    f = -rng.gamma(2.0, 1.5, (n, T)).astype(np.float32) - np.float32(magnitude * rng.random((n, 1)))
    f[rng.random((n, T)) < 0.2] = -1e30
    want, v = exact(x, f)
    w = np.exp(v - want[:, None])
    ulp = lambda a: np.spacing(np.abs(a).astype(np.float32)).astype(np.float64)
    log2s = (want - v.max(1)) / np.log(2.0)                # (rounded as log2 gives it, and after its correction)
    expected = ((w * ulp(np.maximum(v, -1e4))) ** 2).sum(1) / 12 + ulp(want) ** 2 / 12 + 2 * (np.log(2.0) * ulp(log2s)) ** 2 / 12
    expected = expected + (2 * it * rounds + np.log2(lpc)) * 2.0 ** -46 / 12
    err = chain(units, lpc, it, x, f) - want
    assert np.sqrt(np.mean(err ** 2)) < 1.12 * np.sqrt(np.mean(expected))


# log0, values so low that neighbouring floats lie whole units apart, and sums whose first round of loads is of that kind
@pytest.mark.parametrize("lpc,it", [(16, 2), (64, 4)])
def test_prefix_sums_of_values_far_out(units, lpc, it):
    T = 4 * lpc * it * 3
    levels = [0.0, -3.0e4, -2.0e6, -1.5e7, -2.0e8, -2.7e8, -4.0e8, -1.0e12, -1.0e25]
    rows, f_rows = [], []
    for level in levels:
        for late in (0, 1, 2):                             # which third holds the values
            x = np.full(T, -1e30, np.float32)
            x[late * T // 3:(late + 1) * T // 3] = level + np.linspace(-1, 0, T // 3)
            rows.append(x); f_rows.append(np.where(np.arange(T) % 5 == 0, -1e30, -0.5).astype(np.float32))
            rows.append(np.where(x < -1e29, np.float32(1.5 * level - 10.0), x)); f_rows.append(np.zeros(T, np.float32))
    rows.append(np.full(T, -1e30, np.float32)); f_rows.append(np.full(T, -1e30, np.float32))
    rows.append(np.full(T, -5.0, np.float32)); f_rows.append(np.full(T, -1e30, np.float32))
    x, f = np.array(rows, np.float32), np.array(f_rows, np.float32)
    got = chain(units, lpc, it, x, f)
    want, _ = exact(x, f)
    assert (got[-2:] == -1e30).all() or np.allclose(got[-2:], -1e30)
    # two roundings of half a unit each, and the sum's own
    tol = 1.5 * np.spacing(np.abs(want[:-2]).astype(np.float32)) + 1e-6
    assert (np.abs(got[:-2] - want[:-2]) <= tol).all(), (got[:-2] - want[:-2], tol)


# Two roundings, of exp2 and of the correction, and as much again for libm's exp2: 2^-24 of the value each; and what fp32's
# ln 2 lacks, 2.8e-9 of it.  Without the correction 87 times 2^-24 at -87.
def test_exponential_of_large_arguments(units):
    v = -np.concatenate([np.linspace(0, 87, 20001), np.geomspace(1e-7, 1, 500)]).astype(np.float32)
    got = np.empty_like(v)
    units.unit_exp(ptr(v), len(v), ptr(got))
    want = np.exp(v.astype(np.float64))
    assert (np.abs(got / want - 1) < 3 * 2.0 ** -24 + 2.8e-9 * np.abs(v)).all()
    edge = np.array([-1e30, -1e4, -200.0, 0.0], np.float32)
    got = np.empty_like(edge)
    units.unit_exp(ptr(edge), 4, ptr(got))
    assert (got[:3] == 0).all() and got[3] == 1


# Sums of products over thousands of frames: each product is rounded like its factor (exp, below 3 units of 2^-24) in a
# sum where that averages out; a block's 32 products are added one by one, at most 32 roundings of 2^-24 of the block's
# share, evenly spread ones 1/sqrt(3) of that; then the waves' last sum and two between the waves, 2^-24 each, the
# mantissa's logarithm (up to 1, one unit of its own and its product with ln 2) and the increment's own rounding.  A chain over
# all frames of a wave lies at 2 (1500 frames) to 4 times that (6000), a logarithm of the whole sum at 2 for sums around e^-14.
@pytest.mark.parametrize("T,Wb,low", [(60, 16, 0), (60, 16, 14), (1500, 16, 0), (3000, 20, 20)])
def test_long_sums_of_products(units, T, Wb, low):
    rng = np.random.default_rng(T)
    Tp, V = (T + 5 + 31) // 32 * 32, 18
    x = np.zeros((V, Tp), np.float32)
    x[:, 1:T + 1] = -rng.gamma(3.0, 2.0, (V, T)) - low
    F = np.zeros((Wb, Tp), np.float32)
    F[:, 1:T + 1] = np.exp(-rng.gamma(1.5, 1.0, (Wb, T)))
    out = np.empty((Wb, V - 2), np.float32)
    m = -rng.random(Wb).astype(np.float32)
    units.unit_dense(ptr(x), ptr(F), ptr(m), T, Tp, V, Wb, ptr(out))
    want = m[:, None].astype(np.float64) + np.log(F.astype(np.float64) @ np.exp(x[1:-1].astype(np.float64)).T)
    err = out - want
    u = 2.0 ** -24
    blocks = T / 32
    expected = (32 / 3 + 3) * u ** 2 / blocks + 3 * u ** 2 / 3
    expected += (2 + 1) * u ** 2 / 3 + np.mean(np.spacing(np.abs(out)).astype(np.float64) ** 2) / 12
    assert np.sqrt(np.mean(err ** 2)) < 1.12 * np.sqrt(expected)


# The pivot lets K of the lanes' maxima through, and few more whatever the row's scale: a sixteenth below the K-th largest
# (or what eight bits of mantissa leave: a 256th of it), and what equals it.  Rows of log-probabilities, of scores above zero, far below
# it, on both sides of it, and spread so far that the K-th value lies more than 32 below the largest.
@pytest.mark.parametrize("K", [3, 42, 66])
@pytest.mark.parametrize("centre,spread", [(-8.0, 2.0), (20.0, 3.0), (3e4, 3.0), (-60.0, 2.0), (-500.0, 3.0), (0.0, 4.0), (-0.5, 0.3), (-20.0, 60.0), (40.0, 90.0)])
def test_pivot_is_close_to_the_last_candidate(units, K, centre, spread):
    for seed in range(4):
        mx = (centre + spread * np.random.default_rng(seed).standard_normal(256)).astype(np.float32)
        out = np.empty(4, np.float32)
        units.unit_pivot(ptr(mx), K, ptr(out))
        kth = np.sort(mx)[-K].astype(np.float64)
        assert (out == out[0]).all() and (mx >= out[0]).sum() >= K
        assert out[0] > kth - max(0.125, abs(kth) / 128), (out[0], kth)


def top_pairs(units, inc, att, base, bits, lam=1.0, block=256):
    Wb, K = inc.shape
    J, slot, place, counts = np.full(Wb, np.nan), np.full(Wb, -1, np.int32), np.full(Wb, -1, np.int32), np.zeros(2, np.int32)
    base = np.ascontiguousarray(base, np.float64)
    units.unit_top(block, ctypes.c_double(lam), ptr(inc), ptr(att), ptr(base), Wb, K, bits, ptr(J), ptr(slot), ptr(place), ptr(counts))
    return J, slot, place, counts


def check_top(inc, base, got):
    # (lambda = 1: the joint score is base + increment, rounded once)
    Wb, K = inc.shape
    want = np.where(inc > -1e29, base[:, None] + inc.astype(np.float64), -np.inf).ravel()
    order = np.lexsort((np.arange(Wb * K), -want))[:Wb]
    order = order[want[order] > -1e29]
    J, slot, place, counts = got
    n = len(order)
    assert np.array_equal(J[:n], want[order]) and np.array_equal(slot[:n], order // K) and np.array_equal(place[:n], order % K)
    assert (slot[n:] == -1).all() and counts[0] >= n


# The best pairs of a beam, slots that share their best candidates as the hypotheses of a beam do; numbers of candidates whose chunks per
# slot are a power of two among them, more chunks than the lanes hold.  How many chunks reach the pivot: the Wb-th largest of 64 maxima
# lets those through that share a maximum with a better one, up to 2 Wb measured in decodes; bound 3 Wb and a few.  (Slots one after the other
# in the maxima: 4 to 9 Wb at numbers of chunks that are multiples of 64; a pivot of 14 bits of the range, scores on both sides of
# zero: up to 10 Wb.)
@pytest.mark.parametrize("Wb,K,bits", [(1, 65, 4), (3, 998, 5), (16, 1022, 4), (20, 4998, 5), (32, 510, 4), (32, 2048, 5), (32, 4094, 5)])
@pytest.mark.parametrize("level,spread", [(-1500.0, 4.0), (0.0, 3.0)])
def test_best_pairs_from_few_chunks(units, Wb, K, bits, level, spread):
    for zipf in (0, 1):
        rng = np.random.default_rng(100 * Wb + zipf)
        shared = spread * rng.standard_normal(K) - spread * 0.6 * np.log1p(np.arange(K)) * zipf
        inc = (shared[None] + 0.5 * rng.standard_normal((Wb, K))).astype(np.float32)
        base = level - 0.7 * spread * rng.random(Wb)
        got = top_pairs(units, inc, np.zeros((Wb, K), np.float32), base, bits)
        check_top(inc, base, got)
        assert got[3][1] <= 3 * Wb + 6, got[3]


# More chunks or more scores at the pivot than fit: all scores equal, two levels, equal in their upper halves; and hardly any score at all.
# Equal scores go by slot and place.
@pytest.mark.parametrize("Wb,K,bits,block", [(32, 2048, 4, 256), (20, 1022, 4, 1024), (3, 70, 4, 256)])
def test_best_pairs_of_scores_that_agree(units, Wb, K, bits, block):
    rng = np.random.default_rng(K)
    att = rng.standard_normal((Wb, K)).astype(np.float32)
    flat = np.full((Wb, K), -2.0, np.float32)
    base = np.full(Wb, -7.0)
    check_top(flat, base, top_pairs(units, flat, att, base, bits, block=block))
    two = flat.copy()
    two[-1, [K - 1, 5]] = -1.0
    check_top(two, base, top_pairs(units, two, att, base, bits, block=block))
    near = (flat + rng.permutation(Wb * K).reshape(Wb, K).astype(np.float32) * np.float32(2.0 ** -22)).astype(np.float32)
    check_top(near, base + 4000.0, top_pairs(units, near, att, base + 4000.0, bits, block=block))
    signs = np.where(rng.random((Wb, K)) < 0.5, 7.0, np.float32(7.0 - 2.0 ** -21)).astype(np.float32)      # (scores of zero, and a little below)
    check_top(signs, base, top_pairs(units, signs, att, base, bits, block=block))
    few = np.full((Wb, K), -1e30, np.float32)
    few[Wb // 2, 3] = -5.0
    few[0, K - 1] = -5.0
    check_top(few, base, top_pairs(units, few, att, base, bits, block=block))
    few[:] = -1e30
    check_top(few, base, top_pairs(units, few, att, base, bits, block=block))


# Sums over near frames that the frames left out may count for take in the frames that can, not all of them: in steps
# whose window is the whole utterance a third of the loads remains (the first of the three steps has no near frames: a
# term of its third is loaded 1.6 times, and of the others' 0.25 times to begin with).
def test_sums_of_sharp_posteriors_read_few_frames_more(tmp_path):
    column = "auto column = [&](int id, int i) {"
    so = build_emu.build(str(tmp_path), sanitize=False, units=True,
                         plant=("k_score.h", column, column + " __atomic_fetch_add(&emu::n_columns, 1, __ATOMIC_RELAXED);"))
    r = subprocess.run([sys.executable, os.path.join(HERE, "cpu_emu", "run_case.py"), so, "sharp_posteriors"],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert float(re.search(r"column_loads_per_term=([\d.]+)", r.stdout).group(1)) < 1.6 / 3 + 2 * 0.5 / 3, r.stdout


# Whose attention rows are fetched in batches that do not fetch them blindly: live slots' alone where that is known in time, from the record (short rows, many
# candidates) or because the beam cannot hold more than one hypothesis (one candidate each; 256 utterances, beam 20, 5000 ids: a
# decode took 3080 us with the dead slots' rows, 2490 without).
def test_no_rows_of_dead_slots(tmp_path):
    fetch = "auto fetch_row = [&]() {"
    so = build_emu.build(str(tmp_path), sanitize=False, units=True, defines=["CTCBS_EARLY_GROUPS=0"],
                         plant=("k_score.h", fetch, fetch + " if (threadIdx.x == 0) __atomic_fetch_add(&emu::n_columns, 1, __ATOMIC_RELAXED);"))
    for case in ("one_candidate", "pivot_k80", "pivot"):     # (each a process: the count is of all that it decodes)
        r = subprocess.run([sys.executable, os.path.join(HERE, "cpu_emu", "run_case.py"), so, case], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        rows, groups = re.search(r"counted=(\d+) groups=(\d+)", r.stdout).groups()
        assert 0 < int(rows) == int(groups), r.stdout


# The host's lead over the device: two intervals, for close looks five steps at most
@pytest.mark.parametrize("poll_every,steps", [(1, 2), (2, 4), (3, 5), (8, 5), (16, 5), (17, 34), (1000, 2000), (2 ** 31 - 1, 2 ** 21)])
def test_lead_of_the_host(units, poll_every, steps):
    assert units.unit_steps_ahead(poll_every) == steps


# The kernels' forms by the configuration: the score kernel's by the window and, in wide ones, by the places that its rounds leave empty, near frames looked for where that kernel sums them first
# (more than 64 candidates, and the kernels for every id, sum all frames), lanes per new hypothesis by the widest window.
@pytest.mark.parametrize("over,form,lps,near", [
    (dict(win_m1=50, win_m2=50), 0, 16, False), (dict(win_m1=62, win_m2=62), 0, 16, False), (dict(win_m1=62, win_m2=63), 1, 32, True),
    (dict(win_m1=80, win_m2=80), 1, 32, True), (dict(win_m1=94, win_m2=95), 2, 32, True), (dict(win_m1=126, win_m2=127), 2, 64, True),
    (dict(), 2, 64, True), (dict(t_max=125), 0, 16, False), (dict(t_max=126), 2, 32, True), (dict(t_max=253), 2, 32, True), (dict(t_max=254), 2, 64, True),
    (dict(cand_k=65), 2, 64, False), (dict(cand_k=65, win_m1=80, win_m2=80), 1, 32, False), (dict(cand_k=0), 2, 64, False),
    (dict(cand_k=0, end_flags=7, eos_run=3), 2, 64, False), (dict(cand_k=0, vocab=60), 1, 64, True), (dict(cand_k=0, vocab=42), 2, 64, True),
    (dict(cand_k=10), 1, 64, True), (dict(cand_k=32), 1, 64, True), (dict(cand_k=33), 2, 64, True), (dict(cand_k=48), 2, 64, True),
    (dict(cand_k=49), 1, 64, True), (dict(cand_k=64), 1, 64, True), (dict(cand_k=10, t_max=125), 0, 16, False),
    (dict(cand_k=10, win_m1=50, win_m2=90, win_union=1), 1, 64, True),
    (dict(win_m1=50, win_m2=50, win_union=1), 0, 64, False), (dict(win_m1=50, win_m2=50, win_union=1, t_max=125), 0, 16, False)])
def test_forms_by_the_configuration(units, over, form, lps, near):
    import paper_2101_05600_amd as m
    c = dict(n_utt=1, t_max=300, vocab=100, beam=2, blank_id=0, cand_k=40, win_m1=-1, win_m2=-1, end_flags=3)
    c.update(over)
    cfg = m.make_config(**c)
    ctc = np.full((c["t_max"], c["vocab"]), -4.6, np.float32)
    lens = np.array([c["t_max"]], np.int32)
    h = vp()
    assert units.ctcbs_create(ctypes.byref(cfg), ptr(ctc), ptr(lens), ctypes.byref(h)) == 0
    f = units.unit_forms(h)
    units.ctcbs_destroy(h)
    assert (f & 3, f >> 8, bool(f & 16)) == (form, lps, near)


# Posteriors that are no log-posteriors set the utterance's flag, without an atomic per tile (all XCDs meet at its address); ones rounded
# a little above zero do not.
@pytest.mark.parametrize("vocab,T,value,above", [(130, 40, 2.0, 1), (130, 40, 0.05, 0), (131, 20, np.inf, 1)])
def test_values_above_zero_set_a_flag_without_atomics(units, vocab, T, value, above):
    import paper_2101_05600_amd as m
    units.unit_atomic_ors.restype = ctypes.c_longlong
    cfg = m.make_config(n_utt=2, t_max=T, vocab=vocab, beam=2, blank_id=0, cand_k=20, win_m1=-1, win_m2=-1, end_flags=3)
    ctc = np.full((2, T, vocab), -3.0, np.float32)
    ctc[1, T - 2, vocab - 1] = value
    lens = np.array([T, T - 1], np.int32)
    h, before = vp(), units.unit_atomic_ors()
    assert units.ctcbs_create(ctypes.byref(cfg), ptr(ctc), ptr(lens), ctypes.byref(h)) == 0
    found = [units.unit_above0(h, u) for u in (0, 1)]
    units.ctcbs_destroy(h)
    assert found == [0, above] and units.unit_atomic_ors() == before


# fewer lanes with a value than the pivot is to let through: all values
def test_pivot_of_few_values(units):
    mx = np.full(256, -np.inf, np.float32)
    mx[:40] = np.linspace(-9, -3, 40)
    out = np.empty(4, np.float32)
    units.unit_pivot(ptr(mx), 42, ptr(out))
    assert (out == -np.inf).all()
    units.unit_pivot(ptr(mx), 40, ptr(out))
    assert (mx >= out[0]).sum() == 40 and out[0] > -9.2
