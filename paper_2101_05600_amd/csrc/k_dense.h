// Scoring when every id but blank and eos is a candidate (the paper's Eq. (3) as it stands, no pre-selection).
// The sum over frames of exp(f_t(g) + x_t(c)) is a product of two matrices -- exp(f_t(g)), beam slots by frames, and
// exp(x_t(c)) = p^c(z_t = c), frames by candidates -- so that one exp2 per (candidate, frame) serves all beam slots of an
// utterance and the rest is fp32 MFMA.  What is left is the time it takes to read the posteriors.
//   dense_terms    per (utterance, slot): window, F_t = exp(f_t - M) over it (M the largest f term; 0 outside) and the
//                  frames between its first and its last F that is not 0, ctc part of the eos score, and the one candidate the product does not fit: the repeat of the slot's last label (blank
//                  variable only, third alignment rule of Sec. 2.1).  By k_select_split where it has made the hypothesis, else (first
//                  step, large batches) by a launch of k_dense_prep;
//   k_dense_scores per (utterance, chunk of candidates): the product, i.e. the prefix-score increments, and the best joint score
//                  (Eq. (1)) that each slot has there;
//   the select kernels find the best of all (slot, candidate) pairs from those (dense_top).
// Range: a product below 2^-126 (87 nats under M) counts as nothing; a sum of such products -- below 1e-30 -- is redone
// frame by frame in the log domain.
// Rounding: the exponentials are exact to about an ulp of themselves whatever their argument's size, and sums of 32
// products are added up with what each addition loses carried on, so that the error does not grow with the number of
// frames (one chain of additions per wave: 3 times the error of a tree of short sums at 1500 frames, 6 times at 6000).
// The increment is rounded once, when the mantissa's logarithm joins the rest (add_log).  Against 64 bits, first step of
// 60 to 1500 frames, rms 2.6e-7 (half a unit of the increment); 5.0e-7 with one logarithm of
// the whole sum, 5.4e-7 for one exp2 per term.
// Not handled here (the host then launches k_score): top-K candidates, up to 64 ids, the eos-run rule, raw
// decoder scores, the batch-wide window.
#pragma once
#include "common.h"
#include "k_score.h"

// (as for HypRec::near_frames: e^-NEAR_DEPTH; e^NEAR_MARGIN, 2^26 and what a log-posterior of NEAR_X_MAX may add)
#define NEAR_F 7.8e-20f
#define NEAR_GAIN 7.3e7f
#define DENSE_RANGE 1.0e-30f   // a smaller sum may lack products that underflowed

// f term of frame t (log domain): gamma_{t-1}(g) relative to off' + B_r; only where t - 1 lies in the stored range
__device__ __forceinline__ float dense_f(const float* gphi, const double* Bu, double Bref, int t) {
  return canon0(gphi[t - 1] + (float)(Bu[t - 1] - Bref));
}

// e^(v + lo), v <= 0, |lo| at most a rounding error of v: what v log2(e) loses by its rounding -- as much of the result as
// |v| units in the last place -- is put back by one more step of the exponential's series
__device__ __forceinline__ float exp_exact(float v) {
  const float h = v * L2E, e = __builtin_amdgcn_exp2f(h);
  return fmaf(e, fmaf(h, -LN2, v), e);
}
__device__ __forceinline__ float exp_exact(float v, float lo) {
  const float h = v * L2E, e = __builtin_amdgcn_exp2f(h);
  return fmaf(e, fmaf(h, -LN2, v) + lo, e);
}

// M + log(sum), sum normal and positive, rounded once: of the logarithm only that of the mantissa is rounded by itself (it is
// below 1; a whole log2 of -20 is known to 1e-6), the exponent's multiple of ln 2 and M are added without loss
__device__ __forceinline__ float add_log(float M, float sum) {
  const int b = __float_as_int(sum);
  const float e = (float)((b >> 23) - 127), t = __builtin_amdgcn_logf(__int_as_float((b & 0x7fffff) | 0x3f800000)) * LN2;
  const float k = e * 0.693145751953125f;                      // (ln 2 in 15 bits: exact)
  const float h = M + k, d = h - M;
  return h + (((M - (h - d)) + (k - d)) + fmaf(e, 1.42860682e-6f, t));
}

// the largest value of each half of the wave (N = 32) or row of 16 lanes, in all of its lanes
template <int N>
__device__ __forceinline__ int lanes_max_i(int v) {
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, true));
  v = max(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true));
  if (N == 32) {
#if defined(__AMDGCN__)
    const auto rows = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);   // (each row beside its neighbour)
    v = max((int)rows[0], (int)rows[1]);
#else
    const int a = max(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16));
    const int b = max(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48));
    v = (threadIdx.x & 32) != 0 ? b : a;
#endif
  }
  return v;
}

template <int N> struct Const { static constexpr int value = N; };

__device__ __forceinline__ void dense_no_slot(DenseSlot* slot) { slot->s = 0x7fffffff; slot->e = -1; slot->far_s = -1; slot->far_e = 0; }

// What the product needs of a slot of utterance u at step l, by a whole work-group: its hypothesis r (live flag apart) with its forward
// variables gphi, gb.  dense_f_lds: Tp floats.  Behind the select kernel's part, in the same work-group, it takes 3 us a step less than
// as a launch (7 us: the launch, the records, then the variables from memory): 16 utterances of 1500 frames, 5000 ids, beam 20, a decode
// 9173 -> 8602 us, one 4626 -> 4158, one of 500 to 700, 1000 ids, beam 10 1284 -> 1086, 32 of 60 to 120, 3000 ids, beam 5 546 -> 487.
// Not in the form of one work-group per utterance, which would take its slots one after the other.
template <int BLOCK, class P>
__device__ __forceinline__ void dense_terms(const P& p, float* dense_f_lds, int u, const UttInfo& ui, int l, const HypRec& r, const float* gphi, const float* gb,
                                            float* F, DenseSlot* slot, DenseEos* eos) {
  __shared__ float s_red[BLOCK / 64], s_rs[BLOCK / 64];
  const int tid = threadIdx.x, w = uni(tid >> 6), Tp = p.Tp, T = ui.T;
  const double* Bu = p.Bcum + (size_t)u * Tp;
  const double Bref = r.bref;
  int s = l > 1 ? l : 1, e = T;
  if (p.win_m1 >= 0) s = max(s, r.tau - p.win_m1);
  if (p.win_m2 >= 0) e = min(e, r.tau_end + p.win_m2);
  s = checked(p, s, 1, T + 1, ERR_WINDOW);
  e = checked(p, e, -1, T, ERR_WINDOW);
  const int lo = max(s, r.rs + 1), hi = min(e, r.re + 1);      // frames that have an f term
  const bool rep_ok = r.last >= 0 && r.last != p.blank_id && r.last != p.eos_id && r.last < p.V;
  const float* xr = p.xT + ((size_t)u * p.V + (rep_ok ? r.last : 0)) * Tp;
  float m = LOG0F;
  Lse a;                                                       // the repeated label's sum
  a.m = LOG0F; a.s = 0.0f;
  // R frames per lane and round, their loads in flight together: three (one by one: 7.8 -> 6.9 us a launch at 1500 frames), one where that
  // is the whole window, whose frames would be asked for three times over (70 utterances of 1100 frames, beam 24, windows of 60: 6.2
  // us a launch one by one, 7.8 with three always, 7.1 now; at 1500 frames, whole, 7.0 -> 6.7: the last steps' windows are short)
  auto take = [&](auto rounds) {
    constexpr int R = decltype(rounds)::value;
    for (int t0 = lo; t0 <= hi; t0 += R * BLOCK) {
      float ph[R], pb[R], x[R];
      double B[R];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int t = min(t0 + k * BLOCK + tid, hi);
        ph[k] = FETCH(gphi + t - 1); pb[k] = FETCH(gb + t - 1); B[k] = FETCH(Bu + t - 1); x[k] = FETCH(xr + t);
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int t = t0 + k * BLOCK + tid;
        if (t > hi) break;
        const float bt = (float)(B[k] - Bref), f = canon0(ph[k] + bt);
        dense_f_lds[t] = f;
        m = fmaxf(m, f);
        Lse v;
        v.m = canon0(pb[k] + bt) + x[k]; v.s = 1.0f;
        a = lse_join(a, v);
      }
    }
  };
  if (hi - lo < BLOCK) take(Const<1>()); else if (hi - lo < 3 * BLOCK) take(Const<3>()); else take(Const<6>());
  m = row16_max(m);
  m = fmaxf(fmaxf(lane_f(m, 0), lane_f(m, 16)), fmaxf(lane_f(m, 32), lane_f(m, 48)));
  const float am = chain_max<64>(a.m), as = chain_sum<64>(a.s * __builtin_amdgcn_exp2f((a.m - am) * L2E));
  __shared__ float s_am[BLOCK / 64];
  if ((tid & 63) == 0) { s_red[w] = m; s_am[w] = am; s_rs[w] = as; }
  lds_barrier();
  float M = s_red[0];
#pragma unroll
  for (int i = 1; i < BLOCK / 64; ++i) M = fmaxf(M, s_red[i]);
  const bool some = M > LOG0_CLASS;                            // else: no term at all, every increment is log0
  __shared__ int s_lo[BLOCK / 64], s_hi[BLOCK / 64], s_nlo[BLOCK / 64], s_nhi[BLOCK / 64];
  __shared__ float s_far[BLOCK / 64];
  int f_lo = 0x7fffffff, f_hi = -1, n_lo = 0x7fffffff, n_hi = -1;   // (scalar: a wave's lanes hold 64 frames in a row)
  const bool near_ok = ui.above0 == 0;
  float far = 0.0f;
  for (int t = tid; t - tid < Tp; t += BLOCK) {
    float v = 0.0f;
    if (some && t >= lo && t <= hi) {
      const float f = dense_f_lds[t], d = f - M, b = d + M;
      v = exp_exact(d, (f - b) - (M - (b - d)));           // (f - M rounded, and what that lacks)
    }
    if (t < Tp) F[t] = v;
    const unsigned long long nz = __ballot(v != 0.0f);
    if (nz != 0ull) {
      const int t_w = t - (tid & 63);
      f_lo = min(f_lo, uni(t_w) + __ffsll((long long)nz) - 1);
      f_hi = uni(t_w) + 63 - __clzll((long long)nz);
      const bool is_near = near_ok ? !(v < NEAR_F) : v != 0.0f;
      const unsigned long long nr = __ballot(is_near);
      if (nr != 0ull) {
        n_lo = min(n_lo, uni(t_w) + __ffsll((long long)nr) - 1);
        n_hi = uni(t_w) + 63 - __clzll((long long)nr);
      }
      if (!is_near) far += v;                                  // (a frame between near ones is read, and counted here too)
    }
  }
  far = chain_sum<64>(far);
  if ((tid & 63) == 0) { s_lo[w] = f_lo; s_hi[w] = f_hi; s_nlo[w] = n_lo; s_nhi[w] = n_hi; s_far[w] = far; }
  lds_barrier();
  if (tid == 0) {
    Lse c;
    c.m = s_am[0]; c.s = s_rs[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) { Lse d; d.m = s_am[i]; d.s = s_rs[i]; c = lse_join(c, d); }
    DenseSlot q;
    q.last = rep_ok ? r.last : -1; q.f_lo = lo; q.f_hi = hi;
    q.mref = M; q.inc_rep = c.m < LOG0_CLASS ? LOG0F : c.m + fast_logf(c.s);
    q.ref = r.ref;
    q.s = s_lo[0]; q.e = s_hi[0];
    int ns = s_nlo[0], ne = s_nhi[0];
    float fs = s_far[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) {
      q.s = min(q.s, s_lo[i]); q.e = max(q.e, s_hi[i]);
      ns = min(ns, s_nlo[i]); ne = max(ne, s_nhi[i]);
      fs += s_far[i];
    }
    // (no frame at all: both ranges are empty alike)
    q.far_s = ns - q.s; q.far_e = q.e - ne; q.low = fs * NEAR_GAIN;
    q.offr = r.off + Bref;
    q.jbase = (1.0 - p.lambda) * r.att + p.beta * (double)l;
    *slot = q;
    const bool has = r.rs <= T && r.re >= T;
    const float ce = has ? gphi[T] : LOG0F;
    const bool v = ce > LOG0_CLASS;
    const double ctc = v ? q.offr + (ui.BT - Bref) + (double)ce : LOG0D;
    *eos = DenseEos{ctc, s, e};
  }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_dense_prep(Params p, int l, int cur) {
  extern __shared__ __align__(16) unsigned char dense_smem[];
  const int u = blockIdx.y;
  const size_t h = (size_t)u * p.Wb + blockIdx.x;
  const HypRec r = p.rec[cur][h];
  const UttInfo ui = p.uinfo[u];
  DenseSlot* slot = p.dense_slot + h;
  if (p.finished[u] || !r.live) {
    if (threadIdx.x == 0) dense_no_slot(slot);
    return;
  }
  dense_terms<BLOCK>(p, (float*)dense_smem, u, ui, l, r, p.gphi[cur] + h * p.Tp, p.gb[cur] + h * p.Tp, p.dense_F + h * p.Tp, slot, p.dense_eos + h);
}

// Grid: (chunks of 16 * NT candidates, U), four waves that share the frames of the window for all the work-group's candidates and
// slots, halves of a block of 32 frames in turn (together they walk along the columns), and their sums meet in LDS at the end.  MFMA
// 16x16x4: lane (n, q) = (lane & 15, lane >> 4) holds four consecutive frames of candidate n (of slot n), which serve four products
// whose frame index runs over the four q.  For the loads four neighbouring lanes hold the 64 bytes of a row, and LDS turns
// them round: loaded as the products want them, the 64 lanes of a load touch 54 cache lines, and the cache serves one a cycle.
// Only the frames between the first and the last F of any slot that is not 0 are read: where F underflows its products are
// exactly 0.  Peaked posteriors leave a few hundred frames round the slots' last labels (a label missed costs nats, F is 0
// from 87 on), 10 blocks of 47 at 16 utterances of 1500 frames, 5000 ids, beam 20; flat ones leave them all.  Of those the frames
// with an F of NEAR_F or more first, 6 blocks, and the others only if some sum does not exceed by 2^26 all that they could add (low:
// the slot's F left out, as if its posteriors were 1; on these inputs never): a launch 32.7 -> 24.2 us, of which 28.4 with
// the loads and tiles as they were; posteriors that leave nearly all frames 104 -> 100 us at beam 20, 93 -> 84 at beam 10.
// Bound there: the posteriors of those frames (480 MB); here: the phases of a work-group, so that what counts is how many fit a compute
// unit.  Five with two tiles of slots, seven otherwise: one half ahead, and a wave's sums in the place of its tiles.  Two halves ahead
// and sums beside the tiles (112 registers and 38 KB, four; 78 registers, six): 16 utterances of 1500 frames, 5000 ids, beam 20, a decode
// 9613 -> 9161 us, beam 10 7283 -> 7099, 8 utterances 7075 -> 6485, 32 14789 -> 14010, 64 of 200 to 400 frames, beam 17, 5478 -> 5131.
// Tried before that, slower with four: 16 candidates per work-group (120 us there), a wave for each 16
// candidates, no sums between waves, 25.4 and 122, four halves ahead (33 us), work-groups
// that stay and fetch the next candidates' frames before they finish the last (25.5 and 130).
// The joint scores and each slot's best of them took 5.4 us more a launch (24.7 -> 30.1 at 16 utterances of 1500 frames, 5000 ids,
// beam 20), the select kernel 2.8 more; the launch that made lists of all scores took 10.7.  A decode there 9978 -> 9620 us, of one utterance of
// 800 frames, beam 10, 2455 -> 2098.  In large batches of short inputs that was more than it saved, until the attention values no longer waited for
// the finished flag, waves without a slot did nothing, a slot's best took two thirds of the instructions, the first loads were fewer, and increments and
// attention values lay in rows of whole lines (dense_row: 128 utterances of 300 to 400 frames, 5000 ids, beam 20, 12945 -> 12110, the same as
// with no attention values stored; 16 of 1500 8285 -> 8035); us a decode with lists, then, now: those 128 14060 / 14340 / 12050, 690 of 100 to
// 200, 1000 ids, beam 3 4210 / 4410 / 3975, 2100 of 60 to 120, beam 1 6240 / 7290 / 6440 (there the lists were better by the selection's 7 us a launch),
// 16 of 1500, beam 20 9980 / 8480 / 8050.
template <int NT, int MT>
__global__ __launch_bounds__(256, MT * NT == 4 ? 5 : 7) void k_dense_scores(const float* __restrict__ xT, const float* __restrict__ F,
                                                         const DenseSlot* __restrict__ slots,
                                                         int Wb, int Tp, int V, int K, Params p, int l, int cur) {
  constexpr int NC = 16 * NT, AHEAD = MT * NT > 1 ? 1 : 2, SLOTS = 256 / NC;   // (slots whose sums are looked at together)
  // (a wave's tiles while it multiplies, its sums when it is done)
  constexpr int TURN = (MT + NT) * 64 * 4, SUMS = 16 * MT * (NC + 1), WAVE_LDS = ((TURN > SUMS ? TURN : SUMS) + 3) & ~3;
  __shared__ __align__(16) float s_wave[4][WAVE_LDS];
  __shared__ int s_last[MAX_BEAM], s_live[MAX_BEAM];
  __shared__ float s_m[MAX_BEAM], s_rep[MAX_BEAM], s_low[MAX_BEAM];
  __shared__ int s_far[4];
  __shared__ double s_jb[MAX_BEAM];
  constexpr int NS = 16 * MT / SLOTS;
  __shared__ float s_att[NS][256];                             // the lanes' attention values
  const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6), n = lane & 15, q = lane >> 4;
  const int u = blockIdx.y, c0 = (int)blockIdx.x * NC, Kr = dense_row(K);
  const size_t h0 = (size_t)u * Wb;
  PIN4(p.finished, p.uinfo, p.dense_att, p.blank_id);
  PIN4(p.eos_id, p.lambda, p.cand_att, p.cand_inc);
  // (all that depends on nothing is asked for together.  A load of four words a lane takes the address unit 16 cycles, and with some hundred
  // short-lived work-groups a compute unit that adds up: every wave asks for the slots' frames alone, the first one for the rest; the flag and the
  // length go the scalar way.  A launch of 67000 work-groups, 250 -> 234 us, 16 x 1500 frames, 1024 ids, beam 20, a decode 2860 -> 2825)
  int fin_word = FETCH_SCALAR((const int32_t*)p.finished + (u >> 2)), T = FETCH_SCALAR(&p.uinfo[u].T);
  DenseRange rg = slots[h0 + min(lane, Wb - 1)];
  DenseSlot d;
  if (w == 0) d = slots[h0 + min(lane, Wb - 1)];
  const int lo_ex = min(p.blank_id, p.eos_id), hi_ex = max(p.blank_id, p.eos_id);
  int me = tid;
  auto candidate = [&](int& cc, int& c, int& id) { cc = me & (NC - 1); c = c0 + cc; id = full_v_id(min(c, K - 1), lo_ex, hi_ex); };
  int cc, c, id;
  candidate(cc, c, id);
  const float* att_u = p.dense_att + h0 * (size_t)V;
  const int first = 64 / NC * w;                               // of the wave's slots among SLOTS (waves beyond the beam have nothing to do)
  float att[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i * SLOTS + first < Wb) att[i] = FETCH((const float*)((const char*)att_u + 4u * ((uint32_t)min(i * SLOTS + tid / NC, Wb - 1) * (uint32_t)V + (uint32_t)id)));
  LOADED(rg.s); LOADED(rg.e); LOADED(rg.far_s); LOADED(rg.far_e);
  const bool finished = (fin_word >> (8 * (u & 3)) & 0xff) != 0;
  if (blockIdx.x == 0 && u == 0 && w == 3) publish_progress(p.host_progress, p.n_finished, l);
  if (blockIdx.x == 0 && tid < Wb) {                  // the slot's own results: window, eos scores, work
    GroupOut g = {0, 0, 0, -1, LOG0D, LOG0D, 0, {0, 0, 0, 0, 0, 0}};
    if (!finished && rg.live()) {
      const DenseEos o = p.dense_eos[h0 + tid];
      const int W = o.e >= o.s ? o.e - o.s + 1 : 0;
      g.win_s = o.s; g.win_e = o.e; g.ctc_eos = o.ctc; g.cells = (long long)K * (long long)W;
      if (o.ctc > (double)LOG0_CLASS) g.joint_eos = p.lambda * o.ctc + (1.0 - p.lambda) * (double)p.dense_att[(h0 + tid) * V + p.eos_id] + d.jbase;
      p.dense_left[h0 + tid] = DenseLeft{d.offr, d.jbase};
    }
    p.grp[h0 + tid] = g;
  }
  if (finished) return;
  LOADED(d.low);                                               // (or it is waited for where it is asked for)
  const uint32_t live_slots = (uint32_t)__ballot(lane < Wb && rg.live());
  // the blocks that any slot has an F for, b0 .. e0 - 1, and those read at first, b1 .. e1 - 1
  int b0, e0, b1, e1;
  {
    if (tid < Wb) { s_last[tid] = d.last; s_live[tid] = rg.live(); s_m[tid] = d.mref; s_rep[tid] = d.inc_rep; s_low[tid] = fmaxf(d.low, DENSE_RANGE); s_jb[tid] = dense_base(p.lambda, d); }
    const bool live = lane < Wb && rg.live();                   // (slots in the first 32 lanes: two rows)
    auto lowest = [](int v) { v = row16_min_i(v); return min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)); };
    auto blocks = [&](int s, int e, int& from, int& to) {
      s = lowest(live ? s : 0x7fffffff); e = -lowest(live ? -e : 1);
      s = min(max(s, 1), T); e = min(e, T);
      from = s >> 5; to = e >= s ? (e >> 5) + 1 : from;
    };
    blocks(rg.s, rg.e, b0, e0); blocks(rg.s + rg.far_s, rg.e - rg.far_e, b1, e1);
    b1 = max(b1, b0); e1 = max(min(e1, e0), b1);
    if (e0 - b0 <= 4) { b1 = b0; e1 = e0; }                    // (two halves a wave at most: nothing to gain)
  }
  const float* xu = xT + (size_t)u * V * Tp;
  // (four lanes in a row hold 64 bytes of a candidate, or slot, for the loads; `turn` brings them to where the products need them)
  const int row = lane >> 2, piece = lane & 3;
  const float* bp[NT];
  uint32_t ap[MT];                                             // (bytes from the utterance's F on)
#pragma unroll
  for (int k = 0; k < NT; ++k) bp[k] = xu + (size_t)full_v_id(min(c0 + 16 * k + row, K - 1), lo_ex, hi_ex) * Tp + 4 * piece;
#pragma unroll
  for (int m = 0; m < MT; ++m) ap[m] = 4u * (uint32_t)(min(16 * m + row, Wb - 1) * Tp + 4 * piece);
  const char* F_u = (const char*)(F + h0 * Tp);
  f32x4 (*turn)[64] = (f32x4 (*)[64])s_wave[w];
  const int put = 16 * piece + ((row + 4 * piece) & 15), get = 16 * q + ((n + 4 * q) & 15);
  f32x4 acc[MT][NT], sum[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[m][k] = sum[m][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // Joint scores (Eq. (1)): the best of each slot's candidates here, from which the select kernel finds the utterance's best; the
  // attention values beside the increments (the caller's rows may be gone when someone looks)
  const int n_chunks = (K + NC - 1) / NC;                      // (the grid's width)
  double* best_c = p.dense_best + ((size_t)u * n_chunks + blockIdx.x) * dense_pitch(Wb);
  auto scored = [&](int j0, bool mine, int js, float inc, int cc, int c, int id) {
    const double J = dense_sum(p.lambda, s_jb[js], inc, s_att[j0 / SLOTS][tid]);
    // (the upper half of the score as an integer of its order; the lane with the largest stores its score.  No score: NaN, the least there)
    const long long b = __double_as_longlong(J);
    const bool some = mine & (inc > LOG0_CLASS) & (J > (double)LOG0_CLASS);
    const int hi = some ? (int)(b >> 32) : -1, sign = hi >> 31, ord = hi ^ (sign & 0x7fffffff);
    bool write = ord == lanes_max_i<NC>(ord);
    if (__popcll(__ballot(write)) != 64 / NC) {                // (uniform) scores equal in the upper half, or none at all
      const int lo = (int)b ^ (int)0x80000000 ^ sign, best_lo = lanes_max_i<NC>(write ? lo : (int)0x80000000);
      const unsigned long long same = __ballot(write & (lo == best_lo)) >> (lane & ~(NC - 1));   // (equal scores: the first lane)
      write = cc == __ffs((int)((uint32_t)same & (NC == 32 ? ~0u : 0xffffu))) - 1;
    }
    if (write && j0 + tid / NC < Wb) best_c[js] = __longlong_as_double((long long)((unsigned long long)(uint32_t)hi << 32 | (uint32_t)b));
    if (mine && p.keep_cand) {                                 // (for ctcbs_peek)
      const size_t gk = h0 * (size_t)K + ((uint32_t)js * (uint32_t)K + (uint32_t)c);
      p.cand_id[gk] = id; p.cand_joint[gk] = inc > LOG0_CLASS ? J : LOG0D;
      p.cand_ctc[gk] = inc > LOG0_CLASS ? slots[h0 + js].offr + (double)inc : LOG0D;
    }
  };
  // all of the loop's control is uniform.  whole: nothing is left out; far: a sum that the frames left out may count for
  bool whole = b1 == b0 && e1 == e0, far = false;
  float* inc_u = p.cand_inc + h0 * (size_t)Kr;
  uint32_t again = 0;                                          // a bit for each of the lane's sums that is to be redone
  // the frames read at first; where those left out can count, those before and those behind them too
  f32x4 x[AHEAD][NT], f[AHEAD][MT];
  int b = b1, end = e1, nh;
  auto fetch = [&](int i, int a) {
    i = min(i, nh - 1);
    const int t = 32 * b + 16 * (w + 4 * i);
#pragma unroll
    for (int k = 0; k < NT; ++k) x[a][k] = *(const f32x4*)(bp[k] + t);
#pragma unroll
    for (int m = 0; m < MT; ++m) f[a][m] = *(const f32x4*)(F_u + 4 * (size_t)t + ap[m]);
    SCHED_FENCE();
  };
  auto start = [&]() {
    nh = (2 * (end - b) + 3 - w) >> 2;                         // the wave's halves of a block
    if (nh > 0) {
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) fetch(a, a);
    }
  };
  // (the attention values when the first frames are on their way, so that nothing waits for both in turn; not where that spills:
  // 128 utterances of 300 to 400 frames, 5000 ids, beam 20, 13590 -> 14030 us a decode; 2100 of 60 to 120, 1000 ids, beam 1, 6970 -> 6920)
  constexpr bool FRAMES_FIRST = MT * NT < 4;
  if (FRAMES_FIRST) start();
  float* att_kept = p.cand_att + h0 * (size_t)Kr;
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int j = i * SLOTS + tid / NC;
    if (i * SLOTS + first >= Wb) break;                        // (uniform)
    s_att[i][tid] = att[i];
    if ((live_slots >> j & 1u) != 0u && c < K) STORE_ASIDE(att[i], (float*)((char*)att_kept + 4u * (uint32_t)(j * Kr + c)));
  }
#pragma unroll 1
  for (int part = 0; part < 3; ++part) {
    if (part > 0) { b = part == 1 ? b0 : e1; end = part == 1 ? b1 : e0; }
    if (part > 0 || !FRAMES_FIRST) start();
    if (nh > 0) {
#pragma unroll 1
      for (int i = 0; i < nh; i += AHEAD) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
          if (a == 0 || i + a < nh) {
#pragma unroll
            for (int k = 0; k < NT; ++k) turn[MT + k][put] = f32x4{exp_exact(x[a][k][0]), exp_exact(x[a][k][1]), exp_exact(x[a][k][2]), exp_exact(x[a][k][3])};
#pragma unroll
            for (int m = 0; m < MT; ++m) turn[m][put] = f[a][m];
            fetch(i + a + AHEAD, a);
            wave_lds_fence();
            f32x4 ex[NT], fv[MT];
#pragma unroll
            for (int k = 0; k < NT; ++k) ex[k] = turn[MT + k][get];
#pragma unroll
            for (int m = 0; m < MT; ++m) fv[m] = turn[m][get];
            wave_lds_fence();
#pragma unroll
            for (int o = 0; o < 4; ++o)
#pragma unroll
              for (int k = 0; k < NT; ++k)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(fv[m][o], ex[k][o], acc[m][k], 0, 0, 0);
            if ((AHEAD == 1 ? i : a) & 1) {                    // 32 frames join the sum; what that rounds away starts the next ones'
#pragma unroll
              for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int k = 0; k < NT; ++k) {
                  const f32x4 t = sum[m][k] + acc[m][k];
                  acc[m][k] -= t - sum[m][k];
                  sum[m][k] = t;
                }
            }
          }
        }
      }
    }
    if (part == 1) continue;
    wave_lds_fence();                                          // (the tiles have been read)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) s_wave[w][(16 * m + 4 * q + r) * (NC + 1) + 16 * k + n] = sum[m][k][r] + acc[m][k][r];
    lds_barrier();
    // ---- increments: lane = candidate, the slots dealt to the 256 / NC groups of lanes ----
    whole |= part > 0;
    far = false; again = 0;
    LOADED(me);                                                // (or the lane's candidate is kept in registers through the products)
    candidate(cc, c, id);
#pragma unroll 1
    for (int j0 = 0; j0 + first < Wb; j0 += SLOTS) {
      const int j = j0 + tid / NC, js = min(j, Wb - 1);
      const int at = js * (NC + 1) + cc;
      const float v = (s_wave[0][at] + s_wave[1][at]) + (s_wave[2][at] + s_wave[3][at]);
      const bool mine = j < Wb && c < K && s_live[js], rep = id == s_last[js];
      float inc = v < 3.0e38f ? add_log(s_m[js], v) : v;
      inc = rep ? s_rep[js] : inc;
      far |= mine && !rep && !(v > s_low[js]);
      again |= mine && !rep && !(v > DENSE_RANGE) ? 1u << (j0 / SLOTS) : 0u;
      if (mine) *(float*)((char*)inc_u + 4u * (uint32_t)(js * Kr + c)) = canon0(inc);
      scored(j0, mine, js, canon0(inc), cc, c, id);
    }
    if (whole) break;
    const bool any = __ballot(far) != 0ull;                    // (rare)
    if (lane == 0) s_far[w] = any;
    lds_barrier();                                             // (the sums have been read too)
    if ((s_far[0] | s_far[1] | s_far[2] | s_far[3]) == 0) break;   // (then no sum is below the product's range either, see s_low)
  }
  // a sum below the range of the product, every product far below M or none finite: again, frame by frame
  unsigned long long todo = __ballot(again != 0u);             // (rare)
  const unsigned long long redone = todo;
  while (todo != 0ull) {                                       // (uniform)
    const int who = __ffsll((long long)todo) - 1;
    todo &= todo - 1ull;
    const int idw = __builtin_amdgcn_readlane(id, who);
    for (uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)again, who); bits != 0u; bits &= bits - 1u) {
      const int j = SLOTS * (__ffs((int)bits) - 1) + (64 * w + who) / NC;
      const size_t h = h0 + j;
      const DenseSlot g = slots[h];
      const float* gphi = p.gphi[cur] + h * Tp;
      const double* Bu = p.Bcum + (size_t)u * Tp;
      const double Bref = Bu[checked(p, g.ref, 0, T, ERR_TIME_INDEX)];
      const float* col = xu + (size_t)idw * Tp;
      Lse a;
      a.m = LOG0F; a.s = 0.0f;
      for (int t = g.f_lo + lane; t <= g.f_hi; t += 64) {
        Lse v;
        v.m = dense_f(gphi, Bu, Bref, t) + col[t]; v.s = 1.0f;
        a = lse_join(a, v);
      }
      const float r = lse_finish<64>(a);
      if (lane == who) *(float*)((char*)inc_u + 4u * (uint32_t)(j * Kr + c)) = canon0(r);
    }
  }
  if (redone != 0ull)                                          // (uniform: the wave holds whole chunks)
#pragma unroll 1
    for (int j0 = 0; j0 + first < Wb; j0 += SLOTS) {
      const int j = j0 + tid / NC, js = min(j, Wb - 1);
      const bool mine = j < Wb && c < K && s_live[js];
      scored(j0, mine, js, mine ? FETCH(inc_u + (size_t)js * Kr + c) : LOG0F, cc, c, id);
    }
}
