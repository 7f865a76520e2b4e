// Select kernels (k_select: one work-group per utterance; k_select_split, further down: one per
// new beam slot).  Algorithm 2 from TopB on:
//   - merge the groups' best-first lists into the utterance's new beam (TopB / GatherB),
//     total order (joint desc, parent slot asc, token asc);
//   - the "p > best_score" test that moves g.<eos> into the ended set, forced ending at the
//     step cap, the eos-run stops;
//   - ENDDETECT: Eq. (4), then Algorithm 3's tau count;
//   - forward variables of the new hypotheses over their parent's window (a part of a wave, a wave or four waves each,
//     the recurrence evaluated as two scans of affine maps in the (logaddexp, +)
//     semiring), their time indices tau / tau~ (first argmax from the parent's tau on);
//   - back-pointer record and the step's outputs.
// Everything the decisions need is fetched in one round of independent loads at the top
// (old slots' records and the group lists); the only dependent second round is the
// survivors' state and posterior columns.
#pragma once
#include "common.h"
#include "k_score.h"

struct Aff { float a, b; };   // v -> (v + a) (+) b   in the log semiring

__device__ __forceinline__ Aff aff_then(Aff first, Aff second) {
  Aff r; r.a = first.a + second.a; r.b = lae(first.b + second.a, second.b); return r;
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ Aff aff_stage(Aff v) {
  Aff left;                                 // lanes without a source get the identity map
  left.a = dpp_f<CTRL, ROW_MASK>(0.0f, v.a);
  left.b = dpp_f<CTRL, ROW_MASK>(LOG0F, v.b);
  return aff_then(left, v);
}

struct ArgMax { float v; int t; };

// largest value, earliest frame among equals, over LPS lanes; result in all of them.  The largest value first, then the
// smallest frame among the lanes that hold it: each step of either is one instruction, which on pairs took nine (the
// three maxima of a step together: 1.3 -> 0.6 us at a batch of 512).
template <int LPS>
__device__ __forceinline__ ArgMax lanes_argmax(ArgMax x) {
  float m = row16_max(x.v);
  if (LPS == 64) {                          // (lanes hold ascending frames: the first of them)
    ArgMax r;
    r.v = fmaxf(fmaxf(lane_f(m, 0), lane_f(m, 16)), fmaxf(lane_f(m, 32), lane_f(m, 48)));
    r.t = __builtin_amdgcn_readlane(x.t, __ffsll((long long)__ballot(x.v == r.v)) - 1);
    return r;
  }
  const bool hi = (threadIdx.x & 32) != 0;
  if (LPS == 32) {
    const float a = fmaxf(lane_f(m, 0), lane_f(m, 16)), b = fmaxf(lane_f(m, 32), lane_f(m, 48));
    m = hi ? b : a;
  }
  int t = row16_min_i(x.v == m ? x.t : 0x7fffffff);
  if (LPS == 32) {
    const int a = min(__builtin_amdgcn_readlane(t, 0), __builtin_amdgcn_readlane(t, 16));
    const int b = min(__builtin_amdgcn_readlane(t, 32), __builtin_amdgcn_readlane(t, 48));
    t = hi ? b : a;
  }
  x.v = m; x.t = t;
  return x;
}

// Forward variables of new hypotheses (parent slot `par` extended by `tok`) over the
// parent's window: two scans of affine maps in the (logaddexp, +) semiring (each lane
// owns FPL consecutive frames, composes their maps, the lanes scan the composed maps, and each
// lane then replays its own frames).
// LPS lanes share a survivor, 64 / LPS survivors a wave: 16 lanes x 8 frames cost a wave about 1.6 times the instructions
// of 64 lanes x 2 frames and do four survivors instead of one, which is what counts once there are more survivors than
// idle SIMDs; NWV = 4: the four waves of a work-group share one survivor (long windows of small batches).  NEAR: the frames that
// matter for the new hypothesis's sums are looked for (HypRec::near_frames).
// The recurrence runs on the stored form of the variables (per-frame reference B_t taken out,
// see Params::Bcum): with x'_t(c) = x_t(c) - max(x_t(blank), floor) and d_t = x_t(blank) -
// max(x_t(blank), floor) (zero unless the floor cut),
//   n_t = (n_{t-1} (+) f_t) + x'_t(c),     phi_t = (phi_{t-1} + d_t) (+) n_t,     b_t = phi_{t-1} + d_t,
// so that staying in blank costs nothing and values do not drift with t.  The child's state is
// re-based by delta = inc + (B_r - B_r'), r the parent's reference frame and r' = the parent's
// tau the child's: its values are then near zero around its own tau.  Writes the new state into
// slot n of the other buffer and returns delta and tau / tau~ (first argmax of the true variables,
// stored + B_t, from the parent's tau on; the parent's values if nothing is finite).
// Lanes own frames from a multiple of four on, so that state, posteriors and B go as 16-byte accesses (8, two frames per lane); what
// such an access holds outside the window is written as log0 and never read (the stored range says so).
struct SurvivorIn {
  int par, tok, s, en, rs, re, ptau, ptau_end, plast, pref;
  float inc;
  int T;            // frames of the utterance (bounds of every time index)
  int above0;       // (see UttInfo)
};

// inclusive scan of affine maps over LPS lanes: lane t ends with map_0 then ... then map_t
template <int LPS>
__device__ __forceinline__ Aff scan_aff(Aff v) {
  v = aff_stage<0x111, 0xf>(v);
  v = aff_stage<0x112, 0xf>(v);
  v = aff_stage<0x114, 0xf>(v);
  v = aff_stage<0x118, 0xf>(v);
  if (LPS >= 32) v = aff_stage<0x142, 0xa>(v);
  if (LPS >= 64) v = aff_stage<0x143, 0xc>(v);
  return v;
}
struct SurvivorLds {                                       // NWV > 1
  Aff tot[2][4];                                           // the waves' composed maps (n, phi)
  float last_n, last_p;                                    // the values of the pass's last frame
  ArgMax best[2][4];
  int near_lo[4], near_hi[4];
};
// smallest lo, largest hi over LPS lanes that hold ascending frames (lo > hi: none); result in all of them
template <int LPS>
__device__ __forceinline__ void lanes_range(int& lo, int& hi) {
  if (LPS == 64) {
    const unsigned long long m = __ballot(lo <= hi);
    const int a = __builtin_amdgcn_readlane(lo, (__ffsll((long long)m) - 1) & 63), b = __builtin_amdgcn_readlane(hi, 63 - (__clzll((long long)m) & 63));
    lo = m != 0ull ? a : 0x7fffffff; hi = m != 0ull ? b : -1;
    return;
  }
  lo = row16_min_i(lo); hi = -row16_min_i(-hi);
  if (LPS == 32) {
    const bool up = (threadIdx.x & 32) != 0;
    const int a = min(__builtin_amdgcn_readlane(lo, 0), __builtin_amdgcn_readlane(lo, 16)), b = min(__builtin_amdgcn_readlane(lo, 32), __builtin_amdgcn_readlane(lo, 48));
    const int c = max(__builtin_amdgcn_readlane(hi, 0), __builtin_amdgcn_readlane(hi, 16)), d = max(__builtin_amdgcn_readlane(hi, 32), __builtin_amdgcn_readlane(hi, 48));
    lo = up ? b : a; hi = up ? d : c;
  }
}

template <int LPS, int FPL, int NWV, bool NEAR>
__device__ __forceinline__ void survivor(const SelectArgs& p, int Wb, int u, int n, bool active, const SurvivorIn& in,
                                         SurvivorLds* sx, int& arg_n, int& arg_b, uint32_t& near_out, float& delta_out, double& bref_out) {
  static_assert((FPL == 2 || FPL % 4 == 0) && (NWV == 1 || LPS == 64), "float4 (float2) per lane; waves share a survivor as wholes");
  constexpr int N = FPL == 2 ? 2 : 4, NQ = FPL / N, SPAN = LPS * FPL * NWV;      // frames per pass
  const int lane = threadIdx.x & 63, w = NWV > 1 ? uni(threadIdx.x >> 6) : 0;
  const int li = lane & (LPS - 1), lf = (w * 64 + li) * FPL;   // lane's place, its first frame's
  const size_t h0 = (size_t)u * Wb;
  int bad = 0;
  const size_t hp = h0 + clamped(in.par, 0, Wb - 1, ERR_LIST_ENTRY, bad);
  const float* xu = p.xT + (size_t)u * p.V * p.Tp;
  const float* x0p = xu + (size_t)p.blank_id * p.Tp;
  const float* xcp = xu + (size_t)clamped(in.tok, 0, p.V - 1, ERR_TOKEN, bad) * p.Tp;
  const double* Bu = p.Bcum + (size_t)u * p.Tp;
  const float* pgp = p.gphi + hp * p.Tp;
  const float* pgb = p.gb + hp * p.Tp;
  float* cgp = p.gphi_new + (h0 + n) * p.Tp;
  float* cgb = p.gb_new + (h0 + n) * p.Tp;
  const int T = in.T;
  const int s = clamped(in.s, 1, T, ERR_WINDOW, bad), en = clamped(in.en, s, T, ERR_WINDOW, bad), rs = in.rs, re = in.re;
  // (the child's reference frame is the parent's tau; both values are first needed after the recurrence)
  double Bnew = Bu[clamped(in.ptau, 0, T, ERR_TIME_INDEX, bad)], Bold = Bu[clamped(in.pref, 0, T, ERR_TIME_INDEX, bad)];
  report(p, bad);
  const bool rep = (in.tok == in.plast);
  const int lo = max(s, in.ptau);
  float carry_n = LOG0F, carry_p = LOG0F;
  ArgMax best_n, best_b;
  best_n.v = best_b.v = LOG0F; best_n.t = best_b.t = 0;
  int near_lo = 0x7fffffff, near_hi = -1;
  for (int base = s & ~3; __ballot(base <= en) != 0ull; base += SPAN) {
    float gp[FPL], gb[FPL], x0[FPL], xc[FPL];
    double Bt[FPL];
    const int t0 = base + lf;
    const int tm = min(max(base - 1, 0), T);               // the frame before the pass
    const float gp_m = pgp[tm], gb_m = pgb[tm];
#pragma unroll
    for (int k = 0; k < NQ; ++k) {                         // (clamped into the row; rows are whole multiples of four)
      const int t4 = min(t0 + N * k, p.Tp - N);
      struct __align__(4 * N) F { float v[N]; };
      struct __align__(16) D { double v[2]; };
      const F a = *(const F*)(pgp + t4), b = *(const F*)(pgb + t4), c = *(const F*)(x0p + t4), d = *(const F*)(xcp + t4);
#pragma unroll
      for (int i = 0; i < N; ++i) { gp[N * k + i] = a.v[i]; gb[N * k + i] = b.v[i]; x0[N * k + i] = c.v[i]; xc[N * k + i] = d.v[i]; }
#pragma unroll
      for (int i = 0; i < N; i += 2) { const D e = *(const D*)(Bu + t4 + i); Bt[N * k + i] = e.v[0]; Bt[N * k + i + 1] = e.v[1]; }
    }
    float tw_p = 0.0f, tw_b = 0.0f;                        // the frame before the wave's
    if (NWV > 1) { const int tw = min(max(base + w * 64 * FPL - 1, 0), T); tw_p = pgp[tw]; tw_b = pgb[tw]; }
#pragma unroll
    for (int k = 0; k < FPL; ++k) { LOADED(gp[k]); LOADED(gb[k]); }
    // the previous frame's state: the lane before holds it for the lane's first frame
    float pp = dpp_f<0x138, 0xf>(0.0f, gp[FPL - 1]), pb = dpp_f<0x138, 0xf>(0.0f, gb[FPL - 1]);
    if (li == 0) { pp = NWV > 1 ? tw_p : gp_m; pb = NWV > 1 ? tw_b : gb_m; }
    Aff mn[FPL];                                           // n_t = (n_{t-1} (+) f_t) + x'_t(c)
    float d[FPL];
    bool v[FPL];
#pragma unroll
    for (int k = 0; k < FPL; ++k) {
      const int t = t0 + k;
      v[k] = t >= s && t <= en;
      const float gpp = k == 0 ? pp : gp[k > 0 ? k - 1 : 0], gbp = k == 0 ? pb : gb[k > 0 ? k - 1 : 0];
      const float x0f = fmaxf(x0[k], BLANK_FLOOR), x = xc[k] - x0f;
      d[k] = x0[k] - x0f;
      float f = LOG0F;
      if (t - 1 >= rs && t - 1 <= re) f = rep ? gbp : gpp;
      mn[k].a = v[k] ? x : 0.0f; mn[k].b = v[k] ? f + x : LOG0F;
    }
    // (mp: the frames' maps on entry; composed from the lane's first frame on as soon as they are read, so that the
    // lane's values then follow from v_in each for itself, not one after the other)
    auto run = [&](Aff (&mp)[FPL], float carry, int which, float& v_in, float (&out)[FPL]) {
#pragma unroll
      for (int k = 1; k < FPL; ++k) mp[k] = aff_then(mp[k - 1], mp[k]);
      const Aff P = scan_aff<LPS>(mp[FPL - 1]);
      Aff E;                                               // maps of all earlier lanes
      E.a = dpp_f<0x138, 0xf>(0.0f, P.a); E.b = dpp_f<0x138, 0xf>(LOG0F, P.b);
      if (li == 0) { E.a = 0.0f; E.b = LOG0F; }
      if (NWV > 1) {
        if (lane == 63) sx->tot[which][w] = P;
        lds_barrier();
#pragma unroll
        for (int i = 0; i < NWV - 1; ++i)                  // through the earlier waves' maps
          if (i < w) { const Aff W = sx->tot[which][i]; carry = lae(carry + W.a, W.b); }
      }
      v_in = lae(E.a + carry, E.b);
#pragma unroll
      for (int k = 0; k < FPL; ++k) out[k] = lae(v_in + mp[k].a, mp[k].b);
    };
    float n_in, p_in, nv[FPL], pv[FPL];
    run(mn, carry_n, 0, n_in, nv);
    Aff mp[FPL];                                           // phi_t = (phi_{t-1} + d_t) (+) n_t
#pragma unroll
    for (int k = 0; k < FPL; ++k) { mp[k].a = v[k] ? d[k] : 0.0f; mp[k].b = v[k] ? nv[k] : LOG0F; }
    run(mp, carry_p, 1, p_in, pv);
    const float delta = in.inc + (float)(Bold - Bnew);
    // re-base, store, and the lane's own first argmax over t >= lo of the true variables
    // (stored + B_t; B relative to the child's reference)
    ArgMax xn, xb;
    xn.v = LOG0F; xn.t = t0; xb.v = LOG0F; xb.t = t0;
    float rp[FPL], rb[FPL], near_v[FPL];
#pragma unroll
    for (int k = 0; k < FPL; ++k) {
      const int t = t0 + k;
      const float bv = (k == 0 ? p_in : pv[k > 0 ? k - 1 : 0]) + d[k];
      const float rn = (!v[k] || nv[k] < LOG0_CLASS) ? LOG0F : nv[k] - delta;
      rp[k] = (!v[k] || pv[k] < LOG0_CLASS) ? LOG0F : pv[k] - delta;
      rb[k] = (!v[k] || bv < LOG0_CLASS) ? LOG0F : bv - delta;
      const bool ok = t >= lo;
      const float bt = (float)(Bt[k] - Bnew);
      near_v[k] = v[k] ? rp[k] + bt : LOG0F;
      // (bt <= 0 from the child's reference frame on: what is log0 stays in its class)
      const float cn = ok ? rn + bt : LOG0F, cb = ok ? rb[k] + bt : LOG0F;
      if (cn > xn.v) { xn.v = cn; xn.t = t; }              // (strict: the earlier frame keeps a tie)
      if (cb > xb.v) { xb.v = cb; xb.t = t; }
    }
    if (active) {
#pragma unroll
      for (int k = 0; k < NQ; ++k)
        if (t0 + N * k <= en && t0 + N * k + N - 1 >= s) {
          struct __align__(4 * N) F { float v[N]; } a, b;
#pragma unroll
          for (int i = 0; i < N; ++i) { a.v[i] = rp[N * k + i]; b.v[i] = rb[N * k + i]; }
          *(F*)(cgp + t0 + N * k) = a;
          *(F*)(cgb + t0 + N * k) = b;
        }
    }
    xn = lanes_argmax<LPS>(xn); xb = lanes_argmax<LPS>(xb);
    if (NEAR && (NWV > 1 || p.want_near)) {                // (uniform)
      int pass_lo = 0x7fffffff, pass_hi = -1;
#pragma unroll
      for (int k = FPL - 1; k >= 0; --k)
        if (near_v[k] >= -NEAR_DEPTH) { pass_lo = t0 + k; pass_hi = max(pass_hi, t0 + k); }
      lanes_range<LPS>(pass_lo, pass_hi);
      near_lo = min(near_lo, pass_lo); near_hi = max(near_hi, pass_hi);
    }
    if (xn.v > LOG0_CLASS && xn.v > best_n.v) best_n = xn;
    if (xb.v > LOG0_CLASS && xb.v > best_b.v) best_b = xb;
    if (__ballot(base + SPAN <= en) != 0ull) {             // (uniform) another pass: hand on the last frame's values
      if (NWV > 1) {
        if (threadIdx.x == 64 * NWV - 1) { sx->last_n = nv[FPL - 1]; sx->last_p = pv[FPL - 1]; }
        lds_barrier();
        carry_n = sx->last_n; carry_p = sx->last_p;
        lds_barrier();
      } else {
        carry_n = __shfl(nv[FPL - 1], (lane & ~(LPS - 1)) + LPS - 1);
        carry_p = __shfl(pv[FPL - 1], (lane & ~(LPS - 1)) + LPS - 1);
      }
    }
  }
  if (NWV > 1) {
    if (lane == 0) { sx->best[0][w] = best_n; sx->best[1][w] = best_b; sx->near_lo[w] = near_lo; sx->near_hi[w] = near_hi; }
    lds_barrier();
    best_n = sx->best[0][0]; best_b = sx->best[1][0];      // (waves hold ascending frames within a pass, not across passes)
#pragma unroll
    for (int i = 0; i < NWV; ++i) { near_lo = min(near_lo, sx->near_lo[i]); near_hi = max(near_hi, sx->near_hi[i]); }
#pragma unroll
    for (int i = 1; i < NWV; ++i) {
      const ArgMax a = sx->best[0][i], b = sx->best[1][i];
      if (a.v > best_n.v || (a.v == best_n.v && a.t < best_n.t)) best_n = a;
      if (b.v > best_b.v || (b.v == best_b.v && b.t < best_b.t)) best_b = b;
    }
  }
  arg_n = best_n.v > LOG0_CLASS ? best_n.t : in.ptau;
  arg_b = best_b.v > LOG0_CLASS ? best_b.t : in.ptau_end;
  near_out = in.above0 ? near_pack(0, T) : near_pack(near_lo, near_hi);
  delta_out = in.inc + (float)(Bold - Bnew);
  bref_out = Bnew;
}

// The form of least latency for windows of up to 128 frames: one wave, two frames per lane (any start; longer windows
// in several passes).
template <bool NEAR>
__device__ __forceinline__ void wave_survivor(const SelectArgs& p, int Wb, int u, int n, const SurvivorIn& in,
                                                  int& arg_n, int& arg_b, uint32_t& near_out, float& delta_out, double& bref_out) {
  constexpr int FPL = 2;
  const int lane = threadIdx.x & 63;
  const size_t h0 = (size_t)u * Wb;
  int bad = 0;
  const size_t hp = h0 + clamped(in.par, 0, Wb - 1, ERR_LIST_ENTRY, bad);
  const float* xu = p.xT + (size_t)u * p.V * p.Tp;
  const float* x0 = xu + (size_t)p.blank_id * p.Tp;
  const float* xc = xu + (size_t)clamped(in.tok, 0, p.V - 1, ERR_TOKEN, bad) * p.Tp;
  const double* Bu = p.Bcum + (size_t)u * p.Tp;
  const float* pgp = p.gphi + hp * p.Tp;
  const float* pgb = p.gb + hp * p.Tp;
  float* cgp = p.gphi_new + (h0 + n) * p.Tp;
  float* cgb = p.gb_new + (h0 + n) * p.Tp;
  const int T = in.T;
  const int s = clamped(in.s, 1, T, ERR_WINDOW, bad), en = clamped(in.en, s, T, ERR_WINDOW, bad), rs = in.rs, re = in.re;
  // (the child's reference frame is the parent's tau; both values are first needed after the recurrence)
  double Bnew = Bu[clamped(in.ptau, 0, T, ERR_TIME_INDEX, bad)], Bold = Bu[clamped(in.pref, 0, T, ERR_TIME_INDEX, bad)];
  report(p, bad);
  const bool rep = (in.tok == in.plast);
  const int lo = max(s, in.ptau);
  float carry_n = LOG0F, carry_p = LOG0F;
  float best_n = LOG0F, best_b = LOG0F;
  int near_lo = 0x7fffffff, near_hi = -1;
  arg_n = in.ptau; arg_b = in.ptau_end;
  for (int base = s; base <= en; base += 64 * FPL) {
    int t[FPL]; bool v[FPL]; double Bt[FPL];
    float g_p[FPL], g_b[FPL], x0v[FPL], xcv[FPL];
    Aff mn[FPL];                                         // n_t = (n_{t-1} (+) f_t) + x'_t(c)
    float d[FPL];
#pragma unroll
    for (int k = 0; k < FPL; ++k) {                      // one round of loads
      t[k] = base + FPL * lane + k;
      v[k] = t[k] <= en;
      const int tc = min(t[k], en);                      // clamped: loads are unconditional
      g_p[k] = pgp[tc - 1]; g_b[k] = pgb[tc - 1]; x0v[k] = x0[tc]; xcv[k] = xc[tc];   // (tc >= s >= 1)
      Bt[k] = Bu[tc];
    }
#pragma unroll
    for (int k = 0; k < FPL; ++k) { LOADED(g_p[k]); LOADED(g_b[k]); }
#pragma unroll
    for (int k = 0; k < FPL; ++k) {
      const float x = xcv[k] - fmaxf(x0v[k], BLANK_FLOOR);
      d[k] = x0v[k] - fmaxf(x0v[k], BLANK_FLOOR);
      float f = rep ? g_b[k] : g_p[k];
      f = t[k] - 1 >= rs && t[k] - 1 <= re ? f : LOG0F;
      mn[k].a = v[k] ? x : 0.0f; mn[k].b = v[k] ? f + x : LOG0F;
    }
    Aff C = mn[0];
#pragma unroll
    for (int k = 1; k < FPL; ++k) C = aff_then(C, mn[k]);
    Aff P = scan_aff<64>(C);
    Aff E;                                               // maps of all earlier lanes
    E.a = dpp_f<0x138, 0xf>(0.0f, P.a); E.b = dpp_f<0x138, 0xf>(LOG0F, P.b);
    const float n_in = lae(E.a + carry_n, E.b);
    float nv[FPL];
    nv[0] = lae(n_in + mn[0].a, mn[0].b);
#pragma unroll
    for (int k = 1; k < FPL; ++k) nv[k] = lae(nv[k - 1] + mn[k].a, mn[k].b);
    Aff mp[FPL];                                         // phi_t = (phi_{t-1} + d_t) (+) n_t
#pragma unroll
    for (int k = 0; k < FPL; ++k) { mp[k].a = v[k] ? d[k] : 0.0f; mp[k].b = v[k] ? nv[k] : LOG0F; }
    C = mp[0];
#pragma unroll
    for (int k = 1; k < FPL; ++k) C = aff_then(C, mp[k]);
    P = scan_aff<64>(C);
    E.a = dpp_f<0x138, 0xf>(0.0f, P.a); E.b = dpp_f<0x138, 0xf>(LOG0F, P.b);
    const float p_in = lae(E.a + carry_p, E.b);
    float pv[FPL];
    pv[0] = lae(p_in + mp[0].a, mp[0].b);
#pragma unroll
    for (int k = 1; k < FPL; ++k) pv[k] = lae(pv[k - 1] + mp[k].a, mp[k].b);
    carry_n = lane_f(nv[FPL - 1], 63); carry_p = lane_f(pv[FPL - 1], 63);
    const float delta = in.inc + (float)(Bold - Bnew);
    // re-base, store, and the lane's own first argmax over t >= lo of the true variables
    // (stored + B_t; B relative to the child's reference)
    ArgMax xn, xb;
    xn.v = LOG0F; xn.t = t[0]; xb.v = LOG0F; xb.t = t[0];
    float near_v[FPL];
#pragma unroll
    for (int k = 0; k < FPL; ++k) {
      const float bv = (k == 0 ? p_in : pv[k > 0 ? k - 1 : 0]) + d[k];   // b_t = phi_{t-1} + d_t
      const float rn = (nv[k] < LOG0_CLASS) ? LOG0F : nv[k] - delta;
      const float rp = (pv[k] < LOG0_CLASS) ? LOG0F : pv[k] - delta;
      const float rb = (bv < LOG0_CLASS) ? LOG0F : bv - delta;
      if (v[k]) { cgp[t[k]] = rp; cgb[t[k]] = rb; }
      const bool ok = v[k] && t[k] >= lo;
      const float bt = (float)(Bt[k] - Bnew);
      near_v[k] = v[k] ? rp + bt : LOG0F;
      const float cn = ok ? rn + bt : LOG0F, cb = ok ? rb + bt : LOG0F;   // (bt <= 0, as in `survivor`)
      if (cn > xn.v) { xn.v = cn; xn.t = t[k]; }           // (strict: the earlier frame keeps a tie)
      if (cb > xb.v) { xb.v = cb; xb.t = t[k]; }
    }
    xn = lanes_argmax<64>(xn); xb = lanes_argmax<64>(xb);
    if (NEAR) {
      int pass_lo = 0x7fffffff, pass_hi = -1;
#pragma unroll
      for (int k = FPL - 1; k >= 0; --k)
        if (near_v[k] >= -NEAR_DEPTH) { pass_lo = t[k]; pass_hi = max(pass_hi, t[k]); }
      lanes_range<64>(pass_lo, pass_hi);
      near_lo = min(near_lo, pass_lo); near_hi = max(near_hi, pass_hi);
    }
    if (xn.v > LOG0_CLASS && xn.v > best_n) { best_n = xn.v; arg_n = xn.t; }
    if (xb.v > LOG0_CLASS && xb.v > best_b) { best_b = xb.v; arg_b = xb.t; }
  }
  near_out = in.above0 ? near_pack(0, T) : near_pack(near_lo, near_hi);
  delta_out = in.inc + (float)(Bold - Bnew);
  bref_out = Bnew;
}

// The lists' sort keys: the score as an order-preserving integer whose 10 lowest mantissa bits are replaced by the
// entry's position i = j * Wb + r (group j's r-th best; earlier position = larger key).  One integer comparison then
// gives a strict total order: joint score descending and, among scores equal to within 2^-42 relative (far inside the
// tolerance to which scores are meaningful), parent slot, then token, ascending.  Entries past a list's length: 0.
__device__ __forceinline__ unsigned long long entry_key(double J, int i, bool in) {
  const long long b = __double_as_longlong(J);
  const unsigned long long k = (unsigned long long)(b ^ ((b >> 63) | (long long)0x8000000000000000ull));
  return ((k & ~1023ull) | (unsigned long long)(1023 - i)) & (in ? ~0ull : 0ull);
}
__device__ __forceinline__ int key_entry(unsigned long long key) { return 1023 - (int)(key & 1023ull); }

// The Wb largest of the lists' entries in order, by one wave.  The lists are sorted, so few of the Wb * Wb entries can
// be among them: a lower bound on the Wb-th largest is the Wb-th largest of the first two of every list (compared by the
// upper halves of their keys; no bound if there are fewer), found with one comparison per list entry on values that
// readlane makes scalar; the entries that reach the bound, about 1.3 Wb, are packed into s_ck ([NP + 4], 16-byte
// aligned) and ranked in the same way.  put(rank, entry, valid) is called by all lanes together.  Returns how many were
// packed: at least Wb if there are that many entries at all.  s_key: NP entries, a multiple of 64, zeros behind the lists'.
// One wave needs no barrier: 100 entries all against all by four waves, keys broadcast from LDS, took 1.3 us, the
// packing of the entries above the smallest head through atomics and a ranking by the whole work-group 1.9 us (beam 10,
// 512 utterances) and 2.6 us (beam 20).
template <class F>
__device__ __forceinline__ int rank_lists(const unsigned long long* s_key, unsigned long long* s_ck, int NP, int Wb, F&& put) {
  const int lane = threadIdx.x & 63;
  // (a lane per entry, list lane / 2; the low six bits make the values unique, below 64: no entry)
  const bool in2 = (lane >> 1) < Wb && (lane & 1) < Wb;
  uint32_t hi = (uint32_t)(s_key[min(lane >> 1, Wb - 1) * Wb + min(lane & 1, Wb - 1)] >> 32);
  LOADED(hi);                                              // (no branch round the load)
  const uint32_t k1 = in2 ? (hi & ~63u) | (uint32_t)(63 - lane) : 0u;
  uint32_t bound = 64u;                                    // (an entry's upper half is above that)
  if (__popcll(__ballot(k1 >= 64u)) >= Wb) {
    const int above = lanes_above<8>(k1, 2 * Wb);
    const int at = (__ffsll((long long)__ballot(above == Wb - 1)) - 1) & 63;
    bound = (uint32_t)__builtin_amdgcn_readlane((int)k1, at) & ~63u;
  }
  int n = 0;
  unsigned long long next = s_key[lane];
  for (int i0 = 0; i0 < NP; i0 += 64) {
    const unsigned long long key = next;
    next = s_key[min(i0 + 64, NP - 64) + lane];
    const unsigned long long m = __ballot((uint32_t)(key >> 32) >= bound);
    if ((uint32_t)(key >> 32) >= bound)
      s_ck[n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u))] = key;
    n += __popcll(m);
  }
  __builtin_amdgcn_wave_barrier();
  if (n <= 64) {
    const unsigned long long at = s_ck[lane], me = lane < n ? at : 0ull;
    const int above = lanes_above<8>(me, n);
    put(above, key_entry(me), lane < n);
  } else {                                                 // (beams of about 30 and more, scores that agree in 26 bits)
    const int quads = (n + 3) >> 2;
    if (lane < 4) s_ck[n + lane] = 0ull;
    __builtin_amdgcn_wave_barrier();
    const ulonglong2* s_k2 = (const ulonglong2*)s_ck;
    for (int e0 = 0; e0 < n; e0 += 64) {
      const unsigned long long me = e0 + lane < n ? s_ck[e0 + lane] : 0ull;
      int above = 0;
#pragma unroll 4
      for (int q = 0; q < quads; ++q) {
        const ulonglong2 v = s_k2[2 * q], v2 = s_k2[2 * q + 1];
        above += (int)(v.x > me) + (int)(v.y > me) + (int)(v2.x > me) + (int)(v2.y > me);
      }
      put(above, key_entry(me), e0 + lane < n);
    }
  }
  return n;
}

// Every id a candidate: the Wb best of all (slot, candidate) pairs of an utterance, joint score descending (compared as the fp64 it is),
// then slot, then place = token id ascending.  The scores are not in memory: k_dense_scores leaves increments and attention
// values, and the best score that each slot has in each chunk of 16 or 32 candidates, chunk by chunk (SelectArgs::pitch entries each).
// The Wb-th largest of 64 maxima over those is a pivot that at least Wb scores reach; then the chunks that reach it, their candidates'
// scores, those that reach it, ranked by quads of lanes.  How many chunks reach it depends on how the best ones share
// the 64 maxima (an entry's is its place modulo 64): the slots of a beam have their best candidates in the same few chunks, which an odd
// pitch puts into maxima of their own.  Measured (decodes of 130 to 9001 ids, peaked and flat rows, beams 3 to 32): 1.0 to 1.2 Wb chunks on
// average, at most 2 Wb.  With the slots one after the other and a pivot known to 14 bits of the maxima's range: 1.5 Wb and 9 Wb
// at beam 32, and where a slot's number of chunks was a multiple of 64 the rounds below in many steps: a decode of 4 utterances of 700 frames,
// 4096 ids, beam 32, 9450 -> 3180 us, 16 at beam 20 7570 -> 4760, 16 of 500, 1024 ids, beam 32, 4240 -> 2260; 16 of 1500, 5000 ids, beam 20,
// 8740 -> 8480; maxima past those that the lanes hold eight at a time: one utterance of 300, 20000 ids, beam 32, 2760 -> 1840.
// More than CHUNKS chunks or 32 Wb scores at the pivot (scores equal in their upper halves, to 2^-20 relative): the Wb best chunks exactly, in
// Wb rounds of a block-wide maximum, whose candidates are all that can be among the best.  (Figures: k_dense_scores.)
template <int BLOCK>
struct DenseTopLds {
  static constexpr int CHUNKS = 128;
  uint32_t chunk[CHUNKS];                                  // slot in the upper 5 bits, the chunk's first place
  double base[MAX_BEAM];
  double r_key[2][16];
  uint32_t r_at[2][16];
  uint32_t all_max[BLOCK];
  uint32_t kmax[64], rank[64];
  int n_chunks, n;
};
// The scores that reach the pivot, 32 for each new hypothesis (as many as Wb chunks hold), in dynamic LDS behind the 20 * NP bytes of the
// select kernels' entries: 20 bytes each.
struct DenseTopList {
  double* key;
  uint32_t* at;                                            // slot in the upper 5 bits, place
  float *inc, *att;
  int cap;
  static constexpr int BYTES = 20 * 32;
  __device__ __forceinline__ DenseTopList(unsigned char* lds, int Wb) : key((double*)lds), cap(32 * Wb) {
    at = (uint32_t*)(key + cap); inc = (float*)(at + cap); att = inc + cap;
  }
};
template <bool DENSE, int BLOCK> struct DenseLds { int none; };
template <int BLOCK> struct DenseLds<true, BLOCK> { DenseTopLds<BLOCK> top; };
template <bool DENSE> struct DenseNext { int none; };
template <> struct DenseNext<true> : HypRec {};             // the new hypothesis
constexpr int DENSE_KEYS = 16;                             // best scores of chunks that a lane holds

template <int BLOCK>
__device__ __forceinline__ void dense_fetch(const SelectArgs& p, int u, double (&key)[DENSE_KEYS]) {
  const int total = p.n_chunks * p.pitch;
  const double* best = p.best + (size_t)u * total;
#pragma unroll
  for (int k = 0; k < DENSE_KEYS; ++k) {
    key[k] = LOG0D;
    if (k * BLOCK < total) key[k] = FETCH(best + min((int)threadIdx.x + k * BLOCK, total - 1));   // (uniform)
  }
}
// put(rank, score, slot, place, inc, att) by one lane for each of the best.  Returns how many there are (Wb or more: all).
template <int BLOCK, class F>
__device__ __forceinline__ int dense_top(const SelectArgs& p, DenseTopLds<BLOCK>& t, const DenseTopList& list, int u, int Wb, const double (&key)[DENSE_KEYS], F&& put) {
  constexpr int NW = BLOCK / 64;
  int tid = threadIdx.x;
  const int lane = tid & 63, w = uni(tid >> 6);
  const size_t h0 = (size_t)u * Wb;
  const int total = p.n_chunks * p.pitch, bits = p.chunk_bits;
  const double* best = p.best + (size_t)u * total;
  auto each = [&](auto&& f) {                              // f(place among the utterance's best, its score)
#pragma unroll
    for (int k = 0; k < DENSE_KEYS; ++k)
      if (tid + k * BLOCK < total) f(tid + k * BLOCK, key[k]);
    constexpr int R = 8;                                   // loads in flight
#pragma unroll 1
    for (int i0 = DENSE_KEYS * BLOCK; i0 < total; i0 += R * BLOCK) {
      double more[R];
#pragma unroll
      for (int k = 0; k < R; ++k) more[k] = FETCH(best + min(i0 + k * BLOCK + tid, total - 1));
#pragma unroll
      for (int k = 0; k < R; ++k)
        if (i0 + k * BLOCK + tid < total) f(i0 + k * BLOCK + tid, more[k]);
    }
  };
  double most = LOG0D;
  each([&](int, double k) { most = fmax(most, k); });      // (the pitch's spare entries are NaN)
  // The 64 maxima, and the rank of each: a quarter of the comparisons by each of four waves (lanes turned by a quarter, see take_k; all by
  // every wave, 13 cycles a value: 100 utterances of 60 to 200 frames, 800 ids, beam 20, 1727 -> 1617 us a decode, 256 of 400 to 700, 1000 ids 13490 -> 13290; bit by bit with ballots, until just Wb are left: 128 utterances, 100 ids,
  // beam 20, 2785 -> 2850).
  t.all_max[tid] = (uint32_t)(joint_image(most) >> 32);
  if (tid == 0) { t.n_chunks = 0; t.n = 0; }
  lds_barrier();
  if (w < 4) {
    const int turned = (lane + 16 * w) & 63;
    uint32_t v = t.all_max[turned];
#pragma unroll
    for (int i = 1; i < NW; ++i) v = max(v, t.all_max[64 * i + turned]);
    int n = 0;
    above8<0>(v, n); above8<8>(v, n);
    ((uint8_t*)t.rank)[4 * turned + w] = (uint8_t)n;
    if (w == 0) t.kmax[lane] = v;
  }
  lds_barrier();
  const uint32_t kmax = t.kmax[lane];
  const int above = (int)((t.rank[lane] * 0x01010101u) >> 24);
  uint32_t L = 0u;
#pragma unroll 1
  for (int r = Wb - 1; r >= 0; --r) {                      // (equal maxima: the rank before)
    const unsigned long long m = __ballot(above == r);
    if (m != 0ull) { L = (uint32_t)__builtin_amdgcn_readlane((int)kmax, __ffsll((long long)m) - 1); break; }
  }
  const double low = L != 0u ? image_joint((unsigned long long)L << 32) : (double)LOG0_CLASS;   // (the least score with that upper half; fewer maxima than Wb: all scores)
  auto chunk_at = [&](int i) { const int c = i / p.pitch; return (uint32_t)(i - c * p.pitch) << 27 | (uint32_t)c << bits; };
  LOADED(tid);                                             // (or the places stay in registers from the first pass on)
  each([&](int i, double k) {
    if (k >= low) {
      const int pos = atomicAdd(&t.n_chunks, 1);
      if (pos < DenseTopLds<BLOCK>::CHUNKS) t.chunk[pos] = chunk_at(i);
    }
  });
  lds_barrier();
  // the candidates of n chunks that reach `least`
  auto candidates = [&](int n, double least) {
    constexpr int R = 4;                                   // loads in flight
#pragma unroll 1
    for (int e0 = 0; e0 < n << bits; e0 += R * BLOCK) {
      float inc[R], att[R];
      uint32_t at[R];
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int e = e0 + k * BLOCK + tid;
        at[k] = t.chunk[min(e >> bits, n - 1)] + (uint32_t)(e & ((1 << bits) - 1));
        const size_t g = (h0 + (at[k] >> 27)) * (size_t)dense_row(p.K) + min((int)(at[k] & 0x7ffffffu), p.K - 1);
        inc[k] = FETCH(p.inc + g); att[k] = FETCH(p.att + g);
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int e = e0 + k * BLOCK + tid, slot = (int)(at[k] >> 27);
        const double J = dense_joint(p.lambda, t.base[slot], inc[k], att[k]);
        if (e < n << bits && (int)(at[k] & 0x7ffffffu) < p.K && J > (double)LOG0_CLASS && J >= least) {   // (false for NaN)
          const int pos = atomicAdd(&t.n, 1);
          if (pos < list.cap) { list.key[pos] = J; list.at[pos] = at[k]; list.inc[pos] = inc[k]; list.att[pos] = att[k]; }
        }
      }
    }
  };
  int nc = uni(t.n_chunks);
  if (nc <= DenseTopLds<BLOCK>::CHUNKS) candidates(nc, low);
  lds_barrier();
  if (nc > DenseTopLds<BLOCK>::CHUNKS || uni(t.n) > list.cap) {   // (uniform, rare)
    double last = 0.0;
    uint32_t last_at = 0u;
    nc = 0;
#pragma unroll 1
    for (int rd = 0; rd < Wb; ++rd) {                      // the best behind the one taken last: by score, slot, place
      double m = LOG0D;
      uint32_t at = ~0u;
#pragma unroll 1
      for (int i = tid; i < total; i += BLOCK) {
        const double k = best[i];
        if (k > (double)LOG0_CLASS && k >= m && (rd == 0 || k <= last)) {
          const uint32_t a = chunk_at(i);
          if ((rd == 0 || k < last || a > last_at) && (k > m || a < at)) { m = k; at = a; }
        }
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        const double om = __shfl_xor(m, o);
        const uint32_t oa = __shfl_xor(at, o);
        if (om > m || (om == m && oa < at)) { m = om; at = oa; }
      }
      if (lane == 0) { t.r_key[rd & 1][w] = m; t.r_at[rd & 1][w] = at; }
      lds_barrier();                                       // (two buffers: one barrier per round is enough)
      m = t.r_key[rd & 1][0]; at = t.r_at[rd & 1][0];
#pragma unroll
      for (int i = 1; i < NW; ++i) {
        const double om = t.r_key[rd & 1][i];
        const uint32_t oa = t.r_at[rd & 1][i];
        if (om > m || (om == m && oa < at)) { m = om; at = oa; }
      }
      if (!(m > (double)LOG0_CLASS)) break;                // (uniform)
      if (tid == 0) { t.chunk[rd] = at; t.n = 0; }
      last = m; last_at = at; ++nc;
    }
    lds_barrier();
    candidates(nc, last);
    lds_barrier();
  }
  const int n = min(uni(t.n), list.cap);
#pragma unroll 1
  for (int e0 = 0; e0 < n; e0 += BLOCK / 4) {
    const int e = e0 + (tid >> 2);
    const double me = e < n ? list.key[e] : 0.0;
    const uint32_t at = e < n ? list.at[e] : 0u;
    int rank = 0, equal = 0;                               // (its own entry among the equal ones)
#pragma unroll 2
    for (int i = tid & 3; i < n; i += 4) {
      const double o = list.key[i];
      rank += o > me ? 1 : 0; equal += o == me ? 1 : 0;
    }
    rank += dpp_i<0xB1, 0xf>(0, rank);                     // quad_perm [1,0,3,2]
    rank += dpp_i<0x4E, 0xf>(0, rank);                     // quad_perm [2,3,0,1]
    equal += dpp_i<0xB1, 0xf>(0, equal);
    equal += dpp_i<0x4E, 0xf>(0, equal);
    if (__ballot(e < n && equal > 1) != 0ull)              // (uniform, rare: equal scores go by slot and place)
#pragma unroll 1
      for (int i = 0; i < n; ++i) rank += (int)(list.key[i] == me) & (int)(list.at[i] < at);
    if ((tid & 3) == 0 && e < n && rank < Wb) put(rank, me, (int)(at >> 27), (int)(at & 0x7ffffffu), list.inc[e], list.att[e]);
  }
  return n;
}

// Ended set and ENDDETECT of one utterance, by one wave (lane j = old slot j).  `mine`: slot j
// held a live hypothesis; je / stp / tau_j / cells_j: its eos joint score, eos-run stop, tau and
// prefix-score terms of this step.  st_* / ring_*: the utterance's state as loaded by lane 0
// (scalars) and lanes m < M (ring entries).  Writes the state back, the two per-old-slot
// outputs and the work counters; returns whether the utterance finishes at this step.
__device__ __forceinline__ bool wave_ended_set(const SelectArgs& p, int Wb, int u, UttState* us, int l, int T, int lmax_u, bool has_best,
                                               double best, int n_new, bool mine, double je_in, int stp_in,
                                               int tau_j, long long cells_j, double st_best, int st_n,
                                               int st_cnt, double ring_sc, int ring_tag) {
  const int lane = threadIdx.x & 63;
  const size_t h0 = (size_t)u * Wb, UW = (size_t)p.U * Wb;
  const bool forced = (l >= lmax_u);
  const double je = mine ? je_in : LOG0D;
  const int stp = mine ? stp_in : 0;
  const bool je_ok = je > (double)LOG0_CLASS;
  const bool added = mine && (forced || stp || (je_ok && (!has_best || je > best)));
  long long cells = mine ? cells_j : 0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cells += __shfl_xor(cells, o);
  const int ngroups = __popcll(__ballot(mine));
  const int n_add = __popcll(__ballot(added));
  const int n_tauT = __popcll(__ballot(added && tau_j == T));
  // best newly ended entry: largest score, lowest slot among equals (the one added first)
  double bje = added ? je : -1.0e300; int bj = added ? lane : 0x7fffffff;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const double ov = __shfl_xor(bje, o); const int oj = __shfl_xor(bj, o);
    const bool up = ov > bje || (ov == bje && oj < bj);
    bje = up ? ov : bje; bj = up ? oj : bj;
  }
  if (lane < Wb) { p.out8[UW + h0 + lane] = (uint8_t)added; p.out8[2 * UW + h0 + lane] = (uint8_t)stp; }
  const int n_before = __shfl(st_n, 0);
  const int n_ended = n_before + n_add;
  const int cnt = __shfl(st_cnt, 0) + n_tauT;
  double ybest = __shfl(st_best, 0);
  const bool new_best = n_add > 0 && (n_before == 0 || bje > ybest);
  if (new_best) ybest = bje;
  // ring of the best ended score per length (slot = length % M)
  const int M = p.end_m;
  const bool ring_upd = (lane == (l % M)) && n_add > 0;
  if (ring_upd) { ring_tag = l; ring_sc = bje; }
  bool fin = forced || n_new == 0;
  if (!fin && n_ended > 0) {
    if (p.end_flags & 1) {                       // Eq. (4)
      const bool counts = lane < M && ring_tag >= 1 && ring_tag > l - M && ring_tag <= l &&
                          (ring_sc - ybest < (double)p.end_d);
      if (__popcll(__ballot(counts)) == M) fin = true;
    }
    if (!fin && (p.end_flags & 2) && cnt > p.end_c) fin = true;   // Algorithm 3
  }
  if (ring_upd) { us->ring_tag[lane] = ring_tag; us->ring_score[lane] = ring_sc; }
  if (lane == 0) {
    us->n_ended = n_ended; us->cnt_tau_T = cnt;
    if (new_best) { us->best_score = ybest; us->best_step = l; us->best_slot = bj; }
    if (fin) {
      us->finished_step = l;
      p.finished[u] = 1;
      atomicAdd(p.n_finished, 1);
    }
    p.cells[u] += (unsigned long long)cells;
    p.groups[u] += (unsigned long long)ngroups;
  }
  return fin;
}

// Wave 0 ranks the lists and takes the ended set, the others 64 / LPS new hypotheses each at a time.
// Wb_m: the beam, in the bits from 8 on 65536 / Wb + 1 (a position i < 1024 is of list (i * that) >> 16).
// Dynamic LDS: 36 * NP + 32 bytes, NP = Wb * Wb rounded up to whole waves (the list entries and the packed keys); every id a candidate:
// 20 * NP (no keys: with them a beam of 32 would take more than 64 KB) and DenseTopList::BYTES * Wb.
template <int BLOCK, int LPS, int FPL, bool DENSE>
__global__ __launch_bounds__(BLOCK, DENSE ? 4 : 1) void k_select(const HypRec* __restrict__ rec_now, UttState* __restrict__ utt,
                                                  const GroupOut* __restrict__ grp, const ListEntry* __restrict__ grp_list,
                                                  const UttInfo* __restrict__ uinfo, int Wb_m, int l, int U, SelectArgs p) {
  constexpr int NW = BLOCK / 64;
  extern __shared__ __align__(16) unsigned char sel_smem[];
  const int Wb = Wb_m & 255, div_m = Wb_m >> 8;
  const int NE = Wb * Wb;
  const int NP = (NE + 63) & ~63;
  unsigned long long* s_key = (unsigned long long*)sel_smem;          // [NP]
  unsigned long long* s_ck = s_key + NP;                              // [NP + 4] keys of the entries that can reach the new beam
  double* s_J = DENSE ? (double*)sel_smem : (double*)(s_ck + NP + 4); // [NP]
  int* s_tok = (int*)(s_J + NP);                                      // [NP] each
  float* s_inc = (float*)(s_tok + NP);
  float* s_att = s_inc + NP;
  using TopLds = DenseLds<DENSE, BLOCK>;
  __shared__ TopLds s_top;
  __shared__ int s_sel[MAX_BEAM];          // entry index of the new beam's slot n
  __shared__ int s_n;                      // entries ranked
  // old slots' records
  __shared__ int o_live[MAX_BEAM], o_stp[MAX_BEAM], o_tau[MAX_BEAM], o_tau_end[MAX_BEAM];
  __shared__ int o_rs[MAX_BEAM], o_re[MAX_BEAM], o_last[MAX_BEAM], o_ws[MAX_BEAM], o_we[MAX_BEAM], o_ref[MAX_BEAM];
  __shared__ long long o_cells[MAX_BEAM];
  __shared__ double o_je[MAX_BEAM], o_hatt[MAX_BEAM], o_off[MAX_BEAM];
  __shared__ int s_fin;
  __shared__ int s_ntau[MAX_BEAM], s_ntau_end[MAX_BEAM];   // time indices of the new hypotheses
  __shared__ uint32_t s_near[MAX_BEAM];                    // the frames that matter for their sums (HypRec)
  __shared__ float s_delta[MAX_BEAM];                      // by how much each new hypothesis was re-based
  __shared__ double s_bref[MAX_BEAM];                      // B at each new hypothesis's reference frame

  const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6);
  const int u = blockIdx.x;
  const size_t h0 = (size_t)u * Wb;
  TRACE_POINT(p, (size_t)u * Wb, 8);

  // ---- first round of loads: everything that depends on nothing --------------------------------
  // (loads first, with indices clamped instead of branches, all of their uses behind them)
  UttState* us = utt + u;
  const int fs = us->finished_step;
  const int hj = min(tid, Wb - 1);
  const HypRec r = rec_now[h0 + hj];
  const GroupOut g = grp[h0 + hj];
  const UttInfo ui = uinfo[u];
  const int T = ui.T, lmax_u = ui.lmax;
  // utterance state, wave 0: the scalars, lanes m < M the ring entries
  double st_best = LOG0D, ring_sc = LOG0D;
  int st_n = 0, st_cnt = 0, ring_tag = -1;
  if (w == 0) {
    st_best = us->best_score; st_n = us->n_ended; st_cnt = us->cnt_tau_T;
    ring_sc = us->ring_score[min(lane, MAX_END_M - 1)]; ring_tag = us->ring_tag[min(lane, MAX_END_M - 1)];
  }
  // group lists: entry i = j * Wb + r of this utterance (group j's r-th best; Wb * Wb <= 1024 entries)
  auto load_entry = [&](int i, ListEntry& le, int& nj) {
    const int ic = min(i, NE - 1);
    le = grp_list[h0 * Wb + ic];
    nj = grp[h0 + ((ic * div_m) >> 16)].n;
  };
  auto keep_entry = [&](int i, const ListEntry& le, int nj) {
    s_tok[i] = le.tok; s_inc[i] = le.inc; s_att[i] = le.att;
    s_J[i] = le.J;
    s_key[i] = entry_key(le.J, i, (i < NE) & (i - ((i * div_m) >> 16) * Wb < nj));
  };
  ListEntry le;
  int nj;
  double best[DENSE_KEYS];
  double d_base = 0.0;
  if constexpr (DENSE) { d_base = dense_base(p.lambda, p.slots[h0 + hj]); dense_fetch<BLOCK>(p, u, best); }
  else load_entry(tid, le, nj);
  // (scalar loads: on their way together and waited for once, beside the vector loads)
  PIN4(fs, T, lmax_u, p.err);
  PIN4(p.xT, p.Bcum, p.gphi, p.gb);
  PIN4(p.gphi_new, p.gb_new, p.rec_new, p.trie);
  PIN4(p.out, p.out8, p.trie_stride, p.V);
  PIN4(p.Tp, p.blank_id, p.end_flags, p.end_m);
  PIN4(p.end_c, p.end_d, p.win_union, p.win_m2);
  PIN4(p.finished, p.n_finished, p.cells, p.groups);
  if (fs != 0 && fs < l) return;           // outputs of a finished utterance were settled when it finished
  if constexpr (DENSE) { if (tid < Wb) s_top.top.base[tid] = d_base; }
  else {
    if (64 * w < NP) keep_entry(tid, le, nj);              // (whole waves)
    for (int i = tid + BLOCK; i < NP; i += BLOCK) { load_entry(i, le, nj); keep_entry(i, le, nj); }
  }
  if (tid < Wb) {
    o_live[tid] = r.live; o_stp[tid] = g.stopped;
    o_tau[tid] = r.tau; o_tau_end[tid] = r.tau_end;
    o_rs[tid] = r.rs; o_re[tid] = r.re; o_last[tid] = r.last;
    o_ws[tid] = g.win_s; o_we[tid] = g.win_e; o_ref[tid] = r.ref;
    o_cells[tid] = g.cells;
    o_je[tid] = g.joint_eos; o_hatt[tid] = r.att; o_off[tid] = r.off;
  }
  if (tid < MAX_BEAM) s_sel[tid] = -1;
  lds_barrier();
  TRACE_POINT(p, (size_t)u * Wb, 9);
  if constexpr (DENSE) {
    const int n = dense_top<BLOCK>(p, s_top.top, DenseTopList((unsigned char*)s_J + 20 * NP, Wb), u, Wb, best, [&](int rank, double J, int slot, int place, float inc, float att) {
      const int e = slot * Wb + rank;                      // (an entry of that slot's list, see div_m)
      s_sel[rank] = e; s_J[e] = J; s_inc[e] = inc; s_att[e] = att;
      s_tok[e] = full_v_id(place, min(p.blank_id, p.eos_id), max(p.blank_id, p.eos_id));
    });
    if (tid == 0) s_n = n;
  } else if (w == 0) {
    const int n = rank_lists(s_key, s_ck, NP, Wb, [&](int rank, int e, bool valid) { if (valid && rank < Wb) s_sel[rank] = e; });
    if (lane == 0) s_n = n;
  }
  lds_barrier();
  const int ne = s_n;

  TRACE_POINT(p, (size_t)u * Wb, 10);
  // ---- ended set, end detection: wave 0, lane j = old slot j ---------------------------------
  const int n_new = min(ne, Wb);
  if (w == 0) {
    const bool has_best = ne > 0;
    const double best = has_best ? s_J[checked(p, s_sel[0], 0, NE - 1, ERR_LIST_ENTRY)] : LOG0D;
    const int j = lane < Wb ? lane : 0;
    const bool mine = lane < Wb && o_live[j];
    const bool fin = wave_ended_set(p, Wb, u, us, l, T, lmax_u, has_best, best, n_new, mine, o_je[j], o_stp[j], o_tau[j],
                                    o_cells[j], st_best, st_n, st_cnt, ring_sc, ring_tag);
    if (lane == 0) s_fin = fin ? 1 : 0;
  }
  TRACE_POINT(p, (size_t)u * Wb, 11);

  TRACE_POINT(p, (size_t)u * Wb, 12);
  // ---- forward variables of the new hypotheses --------------------------------------------
  // (wave 0 is busy with the ended set above; the other waves take the survivors at once.  A
  // finished utterance's new state is computed too but never used: its slots are marked dead.)
  const size_t UW = (size_t)p.U * Wb;
  float* out_score = (float*)(p.out + 2 * UW);
  constexpr int PER = 64 / LPS;
  const int wu = uni(w), nu = uni(n_new);
  for (int n0 = (wu - 1) * PER; n0 >= 0 && n0 < nu; n0 += (NW - 1) * PER) {
    const int n = n0 + lane / LPS;
    const bool active = n < nu;
    const int e = active ? checked(p, s_sel[n], 0, NE - 1, ERR_LIST_ENTRY) : 0, par = (e * div_m) >> 16;
    SurvivorIn in;
    in.par = par; in.T = T; in.above0 = ui.above0;
    if (active) {
      in.tok = s_tok[e]; in.inc = s_inc[e];
      in.s = o_ws[par]; in.en = o_we[par]; in.rs = o_rs[par]; in.re = o_re[par];
      in.ptau = o_tau[par]; in.ptau_end = o_tau_end[par]; in.plast = o_last[par]; in.pref = o_ref[par];
    } else {                                               // (lanes without a hypothesis go through the motions)
      in.tok = p.blank_id; in.inc = 0.0f; in.s = in.en = 1; in.rs = in.re = in.ptau = in.ptau_end = in.plast = in.pref = 0;
    }
    int arg_n, arg_b;
    uint32_t near;
    float delta;
    double bref;
    survivor<LPS, FPL, 1, (LPS > 16)>(p, Wb, u, active ? n : 0, active, in, nullptr, arg_n, arg_b, near, delta, bref);
    if (active && (lane & (LPS - 1)) == LPS - 1) {
      p.out[3 * UW + h0 + n] = arg_n; p.out[4 * UW + h0 + n] = arg_b;
      p.trie[(size_t)2 * p.trie_stride + h0 + n] = arg_n;
      s_ntau[n] = arg_n; s_ntau_end[n] = arg_b; s_near[n] = near; s_delta[n] = delta; s_bref[n] = bref;
    }
  }
  lds_barrier();                       // (the survivors' state stores stay in flight)
  const bool fin = s_fin != 0;
  // ---- new beam: records, outputs, back-pointers ------------------------------------------
  for (int n = tid; n < Wb; n += BLOCK) {
    const size_t h = h0 + n;
    if (n < n_new) {
      const int e = checked(p, s_sel[n], 0, NE - 1, ERR_LIST_ENTRY), par = (e * div_m) >> 16, tok = s_tok[e];
      p.out[h] = par; p.out[UW + h] = tok; out_score[h] = (float)s_J[e];
      p.out8[h] = fin ? 0 : 1;
      p.trie[h] = par; p.trie[p.trie_stride + h] = tok;
      HypRec r;
      r.live = fin ? 0 : 1; r.last = tok; r.rs = o_ws[par]; r.re = o_we[par];
      r.tau = s_ntau[n]; r.tau_end = s_ntau_end[n]; r.ref = o_tau[par]; r.near_frames = s_near[n];
      r.off = o_off[par] + (double)s_delta[n];
      r.att = o_hatt[par] + (double)s_att[e];
      r.joint = s_J[e];
      r.bref = s_bref[n];
      p.rec_new[h] = r;
      if (p.win_union && !fin) {                 // this hypothesis's share of the next step's window
        atomicMin(&p.union_win[2 * ((l + 1) & 1)], s_ntau[n]);
        atomicMax(&p.union_win[2 * ((l + 1) & 1) + 1], min(s_ntau_end[n] + p.win_m2, T));
      }
    } else {
      p.out[h] = -1; p.out[UW + h] = -1; out_score[h] = LOG0F; p.out8[h] = 0;
      p.out[3 * UW + h] = 0; p.out[4 * UW + h] = 0;
      p.trie[h] = -1; p.trie[p.trie_stride + h] = -1; p.trie[(size_t)2 * p.trie_stride + h] = 0;
      p.rec_new[h].live = 0;
    }
  }

  TRACE_POINT(p, (size_t)u * Wb, 13);
}

// Split form of the select kernel: one work-group per (utterance, new beam slot n), used up to 2048 groups (see the
// host's rule; with the batch-wide window every utterance's share of it lies apart).  Every work-group of
// an utterance ranks the utterance's Wb * Wb list entries itself (the lists are small, the
// ranking is cheaper than a second launch), evaluates the forward variables of
// new hypothesis n and writes its record; the work-group of slot number Wb meanwhile
// updates the ended set, runs ENDDETECT and writes what belongs to the utterance as a whole
// (finished flag, live flags of all slots, the per-old-slot outputs, work counters).  The
// survivors of one utterance so run on Wb compute units instead of sharing one.
// Within a launch the work-groups of an utterance only read what the others do not write:
// the utterance state is read by the last slot's work-group alone, and "finished before this step"
// is taken from the step number at which the utterance finished (0 or the current step both
// mean no).
// One wave does all of it (BLOCK = 64), with no barrier to wait at.  Where windows beyond 128 frames are common (the
// host knows from the window margins), and for beams above 12 (one wave holds 192 list entries), it is four: all of them
// load, the first one ranks, and all share the recurrence of a window of more than 128 frames.  (Per launch, windows of
// 101 frames, one wave / four: beam 4, 64 utterances 7.0 / 7.4 us, beam 12, 64 utterances 7.8 / 8.1, 128 9.0 / 10.2.)
// NEAR: where the score kernel looks at near_frames (one wave: never; found everywhere it cost 1.3 % of a decode at margins of 80).
// Dynamic LDS: 36 * NP + 32 bytes, NP = Wb * Wb rounded up to whole waves (the list entries and the packed keys); every id a candidate:
// 20 * NP + DenseTopList::BYTES * Wb, and 4 * Tp at least (dense_terms).
// The arguments in front of the block are what the first round of loads needs: plain leading arguments reach the wave
// in registers when it starts (kernel-argument preload), so that those loads do not wait for a load of the arguments.
// Grid: (1 << sh, Wb, ceil(U / (1 << sh))), sh = l >> 28: utterance z * 2^sh + x, new slot y (as in k_score).
template <int BLOCK, bool NEAR, bool DENSE>
__global__ __launch_bounds__(BLOCK, DENSE ? 4 : 1) void k_select_split(const HypRec* __restrict__ rec_now, UttState* __restrict__ utt,
                                                        const GroupOut* __restrict__ grp, const ListEntry* __restrict__ grp_list,
                                                        const UttInfo* __restrict__ uinfo, int Wb_m, int l_sh, int U, SelectArgs p) {
  constexpr bool WIDE = BLOCK > 64;
  extern __shared__ __align__(16) unsigned char split_smem[];
  const int Wb = Wb_m & 255, div_m = Wb_m >> 8;                       // (see k_select)
  const int NE = Wb * Wb;
  const int NP = (NE + 63) & ~63;
  unsigned long long* s_key = (unsigned long long*)split_smem;        // [NP]
  unsigned long long* s_ck = s_key + NP;                              // [NP + 4]
  double* s_J = DENSE ? (double*)split_smem : (double*)(s_ck + NP + 4);   // [NP]
  int* s_tok = (int*)(s_J + NP);                                      // [NP] each
  float* s_inc = (float*)(s_tok + NP);
  float* s_att = s_inc + NP;
  using TopLds = DenseLds<DENSE, BLOCK>;
  __shared__ TopLds s_top;
  __shared__ DenseNext<DENSE> s_next;
  __shared__ int s_sel[DENSE ? MAX_BEAM : 1];
  __shared__ SurvivorLds s_sx;
  __shared__ int o_live[MAX_BEAM], o_stp[MAX_BEAM], o_tau[MAX_BEAM];
  __shared__ int o_par[MAX_BEAM][8];       // what a survivor needs of its parent: window, range, tau, tau~, last label, reference frame
  __shared__ long long o_cells[MAX_BEAM];
  __shared__ double o_je[MAX_BEAM], o_hatt[MAX_BEAM], o_off[MAX_BEAM];
  __shared__ int s_pick[3];                // entry ranked n, entry ranked 0, number of entries ranked

  const int tid = threadIdx.x, lane = tid & 63, w = BLOCK == 64 ? 0 : uni(tid >> 6);
  const int l = l_sh & 0xfffffff, sh = l_sh >> 28;
  const int u = (int)((blockIdx.z << sh) + blockIdx.x), n = (int)blockIdx.y;
  if (u >= U) return;                    // (the grid is whole eights of utterances)
  UttState* us = utt + u;
  const int fs = us->finished_step;        // (tested after the first round of loads is on its way)
  const size_t h0 = (size_t)u * Wb;
  const bool lead = n == Wb;
  if (lead) TRACE_POINT(p, (size_t)u * Wb, 8);

  // ---- first round of loads: everything that depends on nothing --------------------------------
  // (as in k_select)
  const int hj = min(tid, Wb - 1);
  const HypRec r = rec_now[h0 + hj];
  const GroupOut g = grp[h0 + hj];
  constexpr int CH = BLOCK == 64 ? 3 : 1024 / BLOCK;       // (NE <= 144 for one wave)
  ListEntry le[CH];
  int nj[CH];
  double best[DENSE_KEYS];
  double d_base = 0.0;
  if constexpr (DENSE) { d_base = dense_base(p.lambda, p.slots[h0 + hj]); dense_fetch<BLOCK>(p, u, best); }
#pragma unroll
  for (int k = 0; !DENSE && k < CH; ++k) {
    const int i = min(tid + k * BLOCK, NE - 1);
    if (BLOCK == 64 || k == 0 || k * BLOCK < NE) { le[k] = grp_list[h0 * Wb + i]; nj[k] = grp[h0 + ((i * div_m) >> 16)].n; }
  }
  const UttInfo ui = uinfo[u];
  const int T = ui.T, lmax_u = ui.lmax;
  double st_best = LOG0D, ring_sc = LOG0D;
  int st_n = 0, st_cnt = 0, ring_tag = -1;
  if (lead && w == 0) {
    st_best = us->best_score; st_n = us->n_ended; st_cnt = us->cnt_tau_T;
    ring_sc = us->ring_score[min(lane, MAX_END_M - 1)]; ring_tag = us->ring_tag[min(lane, MAX_END_M - 1)];
  }
  // (scalar loads: on their way together and waited for once, beside the vector loads)
  PIN4(fs, T, lmax_u, p.err);
  PIN4(p.xT, p.Bcum, p.gphi, p.gb);
  PIN4(p.gphi_new, p.gb_new, p.rec_new, p.trie);
  PIN4(p.out, p.out8, p.trie_stride, p.V);
  PIN4(p.Tp, p.blank_id, p.end_flags, p.end_m);
  PIN4(p.end_c, p.end_d, p.win_union, p.win_m2);
  PIN4(p.finished, p.n_finished, p.cells, p.groups);
  if constexpr (DENSE) { if (tid < Wb) s_top.top.base[tid] = d_base; }
#pragma unroll
  for (int k = 0; !DENSE && k < CH; ++k) {
    const int i = tid + k * BLOCK;
    if (k * BLOCK + 64 * w < NP) {         // (whole waves)
      s_tok[i] = le[k].tok; s_inc[i] = le[k].inc; s_att[i] = le[k].att;
      s_J[i] = le[k].J;
      s_key[i] = entry_key(le[k].J, i, (i < NE) & (i - ((i * div_m) >> 16) * Wb < nj[k]));
    }
  }
  if (tid < Wb) {
    o_live[tid] = r.live; o_stp[tid] = g.stopped;
    o_tau[tid] = r.tau;
    o_par[tid][0] = g.win_s; o_par[tid][1] = g.win_e; o_par[tid][2] = r.rs; o_par[tid][3] = r.re;
    o_par[tid][4] = r.tau; o_par[tid][5] = r.tau_end; o_par[tid][6] = r.last; o_par[tid][7] = r.ref;
    o_cells[tid] = g.cells;
    o_je[tid] = g.joint_eos; o_hatt[tid] = r.att; o_off[tid] = r.off;
  }
  if (fs != 0 && fs < l) return;           // outputs of a finished utterance were settled when it finished
  lds_barrier();
  if (lead) TRACE_POINT(p, (size_t)u * Wb, 9);

  int pick_n = -1, pick_0 = -1, ne = 0;                    // entry ranked n, entry ranked 0 (all scalar)
  if constexpr (DENSE) {
    ne = dense_top<BLOCK>(p, s_top.top, DenseTopList((unsigned char*)s_J + 20 * NP, Wb), u, Wb, best, [&](int rank, double J, int slot, int place, float inc, float att) {
      const int e = slot * Wb + rank;                      // (an entry of that slot's list, see div_m)
      s_sel[rank] = e; s_J[e] = J; s_inc[e] = inc; s_att[e] = att;
      s_tok[e] = full_v_id(place, min(p.blank_id, p.eos_id), max(p.blank_id, p.eos_id));
    });
  } else if (w == 0) {
    ne = rank_lists(s_key, s_ck, NP, Wb, [&](int rank, int e, bool) {   // (ranks below ne are of entries)
      const unsigned long long mn = __ballot(rank == n), m0 = __ballot(rank == 0);
      const int en = __builtin_amdgcn_readlane(e, (__ffsll((long long)mn) - 1) & 63), e0 = __builtin_amdgcn_readlane(e, (__ffsll((long long)m0) - 1) & 63);
      pick_n = mn != 0ull ? en : pick_n;
      pick_0 = m0 != 0ull ? e0 : pick_0;
    });
    if (WIDE && lane == 0) { s_pick[0] = pick_n; s_pick[1] = pick_0; s_pick[2] = ne; }
  }
  if constexpr (DENSE) {
    lds_barrier();
    pick_n = n < min(ne, Wb) ? uni(s_sel[n]) : -1; pick_0 = ne > 0 ? uni(s_sel[0]) : -1;
  } else if (WIDE) {
    lds_barrier();
    pick_n = uni(s_pick[0]); pick_0 = uni(s_pick[1]); ne = uni(s_pick[2]);
  }
  const int n_new = min(ne, Wb);
  if (lead) TRACE_POINT(p, (size_t)u * Wb, 10);

  const size_t UW = (size_t)p.U * Wb;
  float* out_score = (float*)(p.out + 2 * UW);
  const bool hyp = n < Wb && n < n_new;
  int bad = 0;
  const int e_n = clamped(hyp ? pick_n : 0, 0, NE - 1, ERR_LIST_ENTRY, bad), par = (e_n * div_m) >> 16;
  report(p, bad);
  // (a lane each, then into scalar registers: the recurrence below then runs on scalar bases and bounds)
  const int pv = o_par[par][lane & 7];
  const int par_s = __builtin_amdgcn_readlane(pv, 0), par_e = __builtin_amdgcn_readlane(pv, 1);
  const bool shared = WIDE && hyp && par_e - par_s >= 128;                   // all waves take part (uniform)
  if (n < Wb && (w == 0 || shared)) {
    // ---- new hypothesis n: forward variables, record, outputs, back-pointer -----------------
    const size_t h = h0 + n;
    if (hyp) {
      const int e = e_n;
      SurvivorIn in;
      in.par = par; in.tok = uni(s_tok[e]); in.inc = s_inc[e]; in.T = T; in.above0 = ui.above0;
      in.s = par_s; in.en = par_e;
      in.rs = __builtin_amdgcn_readlane(pv, 2); in.re = __builtin_amdgcn_readlane(pv, 3);
      in.ptau = __builtin_amdgcn_readlane(pv, 4); in.ptau_end = __builtin_amdgcn_readlane(pv, 5);
      in.plast = __builtin_amdgcn_readlane(pv, 6); in.pref = __builtin_amdgcn_readlane(pv, 7);
      int arg_n, arg_b;
      uint32_t near;
      float delta;
      double bref;
      if (WIDE && shared) {                                // (uniform: two frames per lane while one pass holds the window, 16
                                                           // whole utterances 1549 -> 1515 us a decode with both forms instead of four always; eight
                                                           // where it takes them to need no second pass, 16 x 1500 frames 11889 -> 11659)
        if (par_e - (par_s & ~3) < 128 * (BLOCK / 64)) survivor<64, 2, BLOCK / 64, NEAR>(p, Wb, u, n, true, in, &s_sx, arg_n, arg_b, near, delta, bref);
        else if (par_e - (par_s & ~3) < 256 * (BLOCK / 64)) survivor<64, 4, BLOCK / 64, NEAR>(p, Wb, u, n, true, in, &s_sx, arg_n, arg_b, near, delta, bref);
        else survivor<64, 8, BLOCK / 64, NEAR>(p, Wb, u, n, true, in, &s_sx, arg_n, arg_b, near, delta, bref);
      }
      else wave_survivor<NEAR>(p, Wb, u, n, in, arg_n, arg_b, near, delta, bref);
      if (tid == 0) {
        p.out[3 * UW + h] = arg_n; p.out[4 * UW + h] = arg_b;
        p.trie[(size_t)2 * p.trie_stride + h] = arg_n;
        p.out[h] = par; p.out[UW + h] = in.tok; out_score[h] = (float)s_J[e];
        p.trie[h] = par; p.trie[p.trie_stride + h] = in.tok;
        // (the record's live flag belongs to the utterance's lead work-group, see below)
        HypRec* r = p.rec_new + h;
        r->last = in.tok; r->rs = in.s; r->re = in.en; r->tau = arg_n; r->tau_end = arg_b; r->ref = in.ptau;
        if (NEAR) r->near_frames = near;
        r->off = o_off[par] + (double)delta;
        r->att = o_hatt[par] + (double)s_att[e];
        r->joint = s_J[e];
        r->bref = bref;
        if constexpr (DENSE) {
          s_next.last = in.tok; s_next.rs = in.s; s_next.re = in.en; s_next.tau = arg_n; s_next.tau_end = arg_b; s_next.ref = in.ptau;
          s_next.off = o_off[par] + (double)delta; s_next.att = o_hatt[par] + (double)s_att[e]; s_next.bref = bref;
        }
        if (p.win_union) {                       // the utterance's share of the next step's window (ignored if it finishes)
          int32_t* sh = p.union_win + 2 * ((size_t)((l + 1) & 1) * p.U + u);
          atomicMin(&sh[0], arg_n);
          atomicMax(&sh[1], min(arg_b + p.win_m2, T));
        }
      }
    } else if (lane == 0) {
      p.out[h] = -1; p.out[UW + h] = -1; out_score[h] = LOG0F;
      p.out[3 * UW + h] = 0; p.out[4 * UW + h] = 0;
      p.trie[h] = -1; p.trie[p.trie_stride + h] = -1; p.trie[(size_t)2 * p.trie_stride + h] = 0;
    }
  } else if (lead && w == 0) {
    // ---- the utterance as a whole: ended set, end detection, live flags ----------------------
    const bool has_best = ne > 0;
    const double best = has_best ? s_J[checked(p, pick_0, 0, NE - 1, ERR_LIST_ENTRY)] : LOG0D;
    const int j = lane < Wb ? lane : 0;
    const bool mine = lane < Wb && o_live[j];
    const bool fin = wave_ended_set(p, Wb, u, us, l, T, lmax_u, has_best, best, n_new, mine, o_je[j], o_stp[j], o_tau[j],
                                    o_cells[j], st_best, st_n, st_cnt, ring_sc, ring_tag);
    if (lane < Wb) {
      const int lv = (lane < n_new && !fin) ? 1 : 0;
      p.out8[h0 + lane] = (uint8_t)lv;
      p.rec_new[h0 + lane].live = lv;
    }
  }
  if (lead) TRACE_POINT(p, (size_t)u * Wb, 13);
  if constexpr (DENSE) {
    // ---- what the product of the next step needs of the new hypothesis (should the utterance have finished, that step looks at
    // nothing of it)
    if (n < Wb && hyp) {                                   // (uniform)
      __syncthreads();                                     // (the forward variables are written, the arrays read)
      dense_terms<BLOCK>(p, (float*)split_smem, u, ui, l + 1, s_next, p.gphi_new + (h0 + n) * p.Tp, p.gb_new + (h0 + n) * p.Tp,
                         p.dense_F + (h0 + n) * p.Tp, p.slots_next + h0 + n, p.eos_next + h0 + n);
    } else if (n < Wb && tid == 0) dense_no_slot(p.slots_next + h0 + n);
  }
}
