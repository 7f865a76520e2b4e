// Scoring when every id but blank and eos is a candidate (the paper's Eq. (3) as it stands, no pre-selection).
// The sum over frames of exp(f_t(g) + x_t(c)) is a product of two matrices -- exp(f_t(g)), beam slots by frames, and
// exp(x_t(c)) = p^c(z_t = c), frames by candidates -- so that one exp2 per (candidate, frame) serves all beam slots of an
// utterance and the rest is fp32 MFMA.  What is left is the time it takes to read the posteriors.
//   k_dense_prep   per (utterance, slot): window, F_t = exp(f_t - M) over it (M the largest f term; 0 outside) and the
//                  frames between its first and its last F that is not 0, eos scores, and the one candidate the product does not fit: the repeat of the slot's last label (blank
//                  variable only, third alignment rule of Sec. 2.1);
//   k_dense_scores per (utterance, chunk of candidates): the product, i.e. the prefix-score increments;
//   k_list_top     per (utterance, slot): joint scores (Eq. (1)) and the group's best-first list.
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

typedef float f32x4 __attribute__((__vector_size__(16)));

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

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_dense_prep(Params p, const float* __restrict__ att, int l, int cur) {
  extern __shared__ __align__(16) unsigned char dense_smem[];
  float* dense_f_lds = (float*)dense_smem;                     // [Tp]
  __shared__ float s_red[BLOCK / 64], s_rs[BLOCK / 64];
  const int tid = threadIdx.x, w = uni(tid >> 6);
  const int Wb = p.Wb, Tp = p.Tp, u = blockIdx.y, j = blockIdx.x;
  const size_t h = (size_t)u * Wb + j;
  const HypRec r = p.rec[cur][h];
  const UttInfo ui = p.uinfo[u];
  if (h == 0 && w == BLOCK / 64 - 1) publish_progress(p.host_progress, p.n_finished, l);
  const int T = ui.T;
  DenseSlot* slot = p.dense_slot + h;
  if (p.finished[u] || !r.live) {
    if (tid == 0) {
      p.grp[h] = GroupOut{0, 0, 0, -1, LOG0D, LOG0D, 0, {0, 0, 0, 0, 0, 0}};
      slot->live = 0; slot->s = 0x7fffffff; slot->e = -1;
    }
    return;
  }
  int s = l > 1 ? l : 1, e = T;
  if (p.win_m1 >= 0) s = max(s, r.tau - p.win_m1);
  if (p.win_m2 >= 0) e = min(e, r.tau_end + p.win_m2);
  s = checked(p, s, 1, T + 1, ERR_WINDOW);
  e = checked(p, e, -1, T, ERR_WINDOW);
  const float* gphi = p.gphi[cur] + h * Tp;
  const float* gb = p.gb[cur] + h * Tp;
  const double* Bu = p.Bcum + (size_t)u * Tp;
  const double Bref = r.bref;
  const int lo = max(s, r.rs + 1), hi = min(e, r.re + 1);      // frames that have an f term
  const bool rep_ok = r.last >= 0 && r.last != p.blank_id && r.last != p.eos_id && r.last < p.V;
  const float* xr = p.xT + ((size_t)u * p.V + (rep_ok ? r.last : 0)) * Tp;
  float m = LOG0F;
  Lse a;                                                       // the repeated label's sum
  a.m = LOG0F; a.s = 0.0f;
  // frames per lane and round, their loads in flight together (one by one: 7.8 -> 6.9 us a launch at 1500 frames)
  constexpr int R = 3;
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
  float* F = p.dense_F + h * Tp;
  __shared__ int s_lo[BLOCK / 64], s_hi[BLOCK / 64];
  int f_lo = 0x7fffffff, f_hi = -1;                            // (scalar: a wave's lanes hold 64 frames in a row)
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
    }
  }
  if ((tid & 63) == 0) { s_lo[w] = f_lo; s_hi[w] = f_hi; }
  lds_barrier();
  if (tid == 0) {
    Lse c;
    c.m = s_am[0]; c.s = s_rs[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) { Lse d; d.m = s_am[i]; d.s = s_rs[i]; c = lse_join(c, d); }
    DenseSlot q;
    q.live = 1; q.last = rep_ok ? r.last : -1; q.win_s = s; q.win_e = e;
    q.mref = M; q.inc_rep = c.m < LOG0_CLASS ? LOG0F : c.m + fast_logf(c.s);
    q.rs = r.rs; q.re = r.re; q.ref = r.ref; q.pad = 0;
    q.s = s_lo[0]; q.e = s_hi[0];
#pragma unroll
    for (int i = 1; i < BLOCK / 64; ++i) { q.s = min(q.s, s_lo[i]); q.e = max(q.e, s_hi[i]); }
    q.offr = r.off + Bref;
    q.jbase = (1.0 - p.lambda) * r.att + p.beta * (double)l;
    *slot = q;
    const bool has = r.rs <= T && r.re >= T;
    const float ce = has ? gphi[T] : LOG0F;
    const bool v = ce > LOG0_CLASS;
    const double ctc = v ? q.offr + (ui.BT - Bref) + (double)ce : LOG0D;
    const int W = e >= s ? e - s + 1 : 0;
    p.grp[h] = GroupOut{0, 0, s, e, ctc, v ? p.lambda * ctc + (1.0 - p.lambda) * (double)att[h * p.V + p.eos_id] + q.jbase : LOG0D,
                        (long long)p.K * (long long)W, {0, 0, 0, 0, 0, 0}};
  }
}

// Grid: (chunks of 16 * NT candidates, U), four waves that share the frames of the window: each takes every fourth
// block of 16 frames (together they walk along the columns) for all the work-group's candidates and slots (no operand is shared between waves, so none goes through LDS),
// and their sums meet in LDS at the end.  MFMA 16x16x4: lane (n, q) = (lane & 15, lane >> 4) holds four consecutive
// frames of candidate n (of slot n): its float4 serves four products whose frame index runs over the four q.
// Only the frames between the first and the last F of any slot that is not 0 are read: where F underflows its products are
// exactly 0.  Peaked posteriors leave a few hundred frames round the slots' last labels (a label missed costs nats, F is 0
// from 87 on), 3 to 4 in 16 at 16 utterances of 1500 frames, 5000 ids: 115 -> 33 us a launch; flat ones leave them all.
// Bound: the posteriors of those frames (4 V T bytes per utterance if all: 480 MB).  MFMA:
// 32 cycles for 16 x 16 x 4, two slot tiles beyond 16 slots: half the time the bytes take.  Half a block is fetched ahead:
// 114 us a launch with all frames, 116.5 with one accumulator per tile and the loads where the compiler put them; with the two
// accumulators the sums need and the loads left to it a decode of 27.1 ms took 37.5.  159 registers, three waves per
// SIMD, for four candidate and two slot tiles; held to fewer the form of one slot tile spills (12.4 -> 13.7 ms a decode).
template <int NT, int MT>
__global__ __launch_bounds__(256, 3) void k_dense_scores(const float* __restrict__ xT, const float* __restrict__ F,
                                                         const DenseSlot* __restrict__ slots,
                                                         int Wb, int Tp, int V, int K, Params p, int l, int cur) {
  constexpr int NC = 16 * NT;
  __shared__ float s_acc[4][16 * MT][NC + 1];
  __shared__ int s_last[MAX_BEAM], s_live[MAX_BEAM];
  __shared__ float s_m[MAX_BEAM], s_rep[MAX_BEAM];
  const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6), n = lane & 15, q = lane >> 4;
  const int u = blockIdx.y, c0 = (int)blockIdx.x * NC;
  const size_t h0 = (size_t)u * Wb;
  if (p.finished[u]) return;
  const int T = p.uinfo[u].T;
  int smin, emax;                                              // the frames that any slot has an F for
  {
    DenseSlot d;
    d.live = 0; d.s = 0x7fffffff; d.e = -1;
    if (lane < Wb) d = slots[h0 + lane];
    if (tid < Wb) { s_last[tid] = d.last; s_live[tid] = d.live; s_m[tid] = d.mref; s_rep[tid] = d.inc_rep; }
    int a = d.live ? d.s : 0x7fffffff, b = d.live ? d.e : -1;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { a = min(a, __shfl_xor(a, o)); b = max(b, __shfl_xor(b, o)); }
    smin = uni(min(max(a, 1), T)); emax = uni(min(b, T));
  }
  const int lo_ex = min(p.blank_id, p.eos_id), hi_ex = max(p.blank_id, p.eos_id);
  const float* xu = xT + (size_t)u * V * Tp;
  const int b0 = smin >> 5, nb = emax >= smin ? (emax >> 5) - b0 + 1 : 0;      // blocks of 32 frames: whole lines of xT
  const int bw = b0 + w, ew = b0 + nb;
  const float* bp[NT];
  const float* ap[MT];
#pragma unroll
  for (int k = 0; k < NT; ++k) bp[k] = xu + (size_t)full_v_id(min(c0 + 16 * k + n, K - 1), lo_ex, hi_ex) * Tp + 4 * q;
#pragma unroll
  for (int k = 0; k < MT; ++k) ap[k] = F + (h0 + min(16 * k + n, Wb - 1)) * Tp + 4 * q;
  f32x4 acc[MT][NT], sum[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int k = 0; k < NT; ++k) acc[i][k] = sum[i][k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // half a block (16 frames) is on its way while the half before it is worked on
  auto fetch = [&](int b, int hf, float4 (&x)[NT], float4 (&f)[MT]) {
#pragma unroll
    for (int k = 0; k < NT; ++k) x[k] = *(const float4*)(bp[k] + 32 * b + 16 * hf);
#pragma unroll
    for (int k = 0; k < MT; ++k) f[k] = *(const float4*)(ap[k] + 32 * b + 16 * hf);
    SCHED_FENCE();
  };
  auto products = [&](const float4 (&x)[NT], const float4 (&f)[MT]) {
    float ex[NT][4], fa[MT][4];
#pragma unroll
    for (int k = 0; k < NT; ++k) { ex[k][0] = exp_exact(x[k].x); ex[k][1] = exp_exact(x[k].y); ex[k][2] = exp_exact(x[k].z); ex[k][3] = exp_exact(x[k].w); }
#pragma unroll
    for (int k = 0; k < MT; ++k) { fa[k][0] = f[k].x; fa[k][1] = f[k].y; fa[k][2] = f[k].z; fa[k][3] = f[k].w; }
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int k = 0; k < NT; ++k)
#pragma unroll
        for (int i = 0; i < MT; ++i) acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[i][c], ex[k][c], acc[i][k], 0, 0, 0);
  };
  float4 x0[NT], f0[MT], x1[NT], f1[MT];
  if (bw < ew) {
    fetch(bw, 0, x0, f0);
    int b = bw;
    for (; b + 4 < ew; b += 4) {
      fetch(b, 1, x1, f1);
      products(x0, f0);
      fetch(b + 4, 0, x0, f0);
      products(x1, f1);
      // the block's 32 frames join the sum; what that rounds away starts the next block's
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int k = 0; k < NT; ++k) {
          const f32x4 t = sum[i][k] + acc[i][k];
          acc[i][k] -= t - sum[i][k];
          sum[i][k] = t;
        }
    }
    fetch(b, 1, x1, f1);                                       // (the wave's last block)
    products(x0, f0);
    products(x1, f1);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int k = 0; k < NT; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_acc[w][16 * i + 4 * q + r][16 * k + n] = sum[i][k][r] + acc[i][k][r];
  lds_barrier();
  // ---- increments: lane = candidate, the slots dealt to 256 / NC groups of lanes ----
  const int cc = tid & (NC - 1), c = c0 + cc;
  const int id = full_v_id(min(c, K - 1), lo_ex, hi_ex);
  for (int j0 = 0; j0 < Wb; j0 += 256 / NC) {
    const int j = j0 + tid / NC, js = min(j, Wb - 1);
    const bool mine = j < Wb && c < K && s_live[js];
    const float sum = (s_acc[0][js][cc] + s_acc[1][js][cc]) + (s_acc[2][js][cc] + s_acc[3][js][cc]);
    float inc = sum < 3.0e38f ? add_log(s_m[js], sum) : sum;
    const bool rep = id == s_last[js];
    if (rep) inc = s_rep[js];
    const bool redo = mine && !rep && !(sum > 1.0e-30f);
    unsigned long long todo = __ballot(redo);
    while (todo != 0ull) {                                     // (uniform) every product far below M, or none finite
      const int who = __ffsll((long long)todo) - 1;
      todo &= todo - 1ull;
      const int jr = __builtin_amdgcn_readlane(js, who), idr = __builtin_amdgcn_readlane(id, who);
      const size_t h = h0 + jr;
      const DenseSlot d = slots[h];
      const float* gphi = p.gphi[cur] + h * Tp;
      const double* Bu = p.Bcum + (size_t)u * Tp;
      const double Bref = Bu[checked(p, d.ref, 0, T, ERR_TIME_INDEX)];
      const float* col = xu + (size_t)idr * Tp;
      Lse a;
      a.m = LOG0F; a.s = 0.0f;
      for (int t = max(d.win_s, d.rs + 1) + lane; t <= min(d.win_e, d.re + 1); t += 64) {
        Lse v;
        v.m = dense_f(gphi, Bu, Bref, t) + col[t]; v.s = 1.0f;
        a = lse_join(a, v);
      }
      const float r = lse_finish<64>(a);
      if (lane == who) inc = r;
    }
    if (mine) p.cand_inc[(h0 + j) * (size_t)K + c] = canon0(inc);
  }
}
