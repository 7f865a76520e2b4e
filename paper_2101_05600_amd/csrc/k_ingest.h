// Batch ingest: Algorithm 2's initialisation on the device.
#pragma once
#include "common.h"

// What the host sets up for a batch -- lengths, step caps, the first batch-wide window -- from pinned host memory
// into device memory, and the batch-wide counters.  set[0..3]: the window words, set[4..]: lengths, then step caps.
__global__ __launch_bounds__(256) void k_setup(Params p, const int32_t* set, int n_empty) {
  const int u = blockIdx.x * 256 + threadIdx.x;
  if (u < p.U) { p.lens[u] = set[4 + u]; p.lmax[u] = set[4 + p.U + u]; p.uinfo[u].above0 = 0; }
  if (p.union_utt) {                                       // step 1: every hypothesis is empty, tau = tau~ = 0
    if (u < p.U) {
      int32_t* sh = p.union_win + 2 * ((size_t)p.U + u);   // (the first step's parity is 1)
      const int T = set[4 + u];
      p.union_win[2 * u] = 0x7fffffff; p.union_win[2 * u + 1] = -1;
      sh[0] = 0; sh[1] = p.win_m2 < T ? p.win_m2 : T;
    }
  } else if (u < 4) p.union_win[u] = set[u];
  if (u == 0) { *p.n_finished = n_empty; *p.err = 0; }
}

// Per-frame reference and empty-prefix state, one work-group per utterance.  z_0 = blank (first alignment rule of
// Sec. 2.1), so the blank variable of the empty hypothesis at frame t is the running sum of the blank
// log-posteriors and the label variable is log0.  That running sum (fp64, each term floored at
// BLANK_FLOOR) is also the reference B_t every stored forward variable is taken relative to: the
// empty hypothesis's stored blank variable is therefore 0 at every frame (minus whatever the
// floor cut off: log0 from the first frame on whose blank probability is zero).
// The blank column is read from the caller's posteriors, not from xT: it then depends on nothing that the
// transposition writes and runs beside it (in a launch of its own, one wave per utterance: 13 us at cfg2, 23 us at
// 1500 frames, after the transposition).  The frames of a round of 2048 are all requested before the first is used.
// An utterance of no frames is an unused slot of the batch: it counts as finished from the start (counted by the
// host), holds no hypothesis and takes part in nothing.
__device__ __forceinline__ void init_state(const Params& p, const float* __restrict__ x, int u) {
  __shared__ double s_v[2][4], s_c[2][4];                // per wave: totals of the pass
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int T = p.lens[u];
  const size_t hyp0 = (size_t)u * p.Wb;
  float* gphi = p.gphi[0] + hyp0 * p.Tp;
  float* gb = p.gb[0] + hyp0 * p.Tp;
  double* Bu = p.Bcum + (size_t)u * p.Tp;
  const float* xb = x + (size_t)u * p.t_max * p.V + p.blank_id;   // row t - 1 holds frame t
  double carry = 0.0, carry_cut = 0.0;
  if (tid == 0) { gphi[0] = 0.0f; gb[0] = 0.0f; Bu[0] = 0.0; }
  constexpr int R = 8;
  for (int base = 1; base <= T; base += 256 * R) {
    float x0[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int t = base + 256 * k + tid;
      x0[k] = t <= T ? fmaxf(xb[(size_t)(t - 1) * p.V], LOG0F) : 0.0f;
    }
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (base + 256 * k > T) break;                     // (uniform)
      const int t = base + 256 * k + tid;
      double v = (double)fmaxf(x0[k], BLANK_FLOOR);      // floored term of B_t
      double c = (double)x0[k] - v;                      // what the floor cut off (0 or negative)
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const double n = __shfl_up(v, o), nc = __shfl_up(c, o);
        if (lane >= o) { v += n; c += nc; }
      }
      if (lane == 63) { s_v[k & 1][w] = v; s_c[k & 1][w] = c; }
      lds_barrier();                                     // (two buffers: the next pass writes the other one)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const double a = s_v[k & 1][i], b = s_c[k & 1][i];
        if (i < w) { v += a; c += b; }
      }
      v += carry; c += carry_cut;
      if (t <= T) { Bu[t] = v; gb[t] = gphi[t] = fmaxf((float)c, LOG0F); }
#pragma unroll
      for (int i = 0; i < 4; ++i) { carry += s_v[k & 1][i]; carry_cut += s_c[k & 1][i]; }
    }
  }
  for (int t = T + 1 + tid; t < p.Tp; t += 256) Bu[t] = carry;   // (never weighted: keeps reads defined)
  if (tid < p.Wb) {
    const size_t h = hyp0 + tid;
    const bool first = tid == 0 && T > 0;
    HypRec r;
    r.live = first; r.last = -1; r.rs = 0; r.re = T; r.tau = 0; r.tau_end = 0; r.ref = 0; r.near_frames = near_pack(0, T);
    r.off = 0.0; r.att = 0.0; r.joint = 0.0; r.bref = 0.0;
    p.rec[0][h] = r;
    // the other buffer: dead until the first selection fills it, but never left holding what the
    // allocation happened to contain (a kernel may load a dead slot's record before it looks at its flag)
    r.live = 0;
    p.rec[1][h] = r;
    p.grp[h] = GroupOut{0, 0, 0, -1, LOG0D, LOG0D, 0, {0, 0, 0, 0, 0, 0}};
    p.out_live[h] = first; p.out_parent[h] = 0; p.out_token[h] = -1; p.out_score[h] = 0.0f;
    p.out_tau[h] = 0; p.out_tau_end[h] = 0; p.out_eos_added[h] = 0; p.out_stopped[h] = 0;
    p.trie_parent[h] = 0; p.trie_token[h] = -1; p.trie_tau[h] = 0;   // level 0: the empty hypothesis
  }
  if (tid == 64) {
    UttInfo& ui = p.uinfo[u];                              // (not above0: the tiles' work-groups set it meanwhile)
    ui.T = T; ui.lmax = p.lmax[u]; ui.BT = carry;          // (B_T: the running sum after the last frame; 0 for T = 0)
    UttState s;
    s.best_score = LOG0D; s.fb_score = LOG0D;
    for (int i = 0; i < MAX_END_M; ++i) { s.ring_score[i] = LOG0D; s.ring_tag[i] = -1; }
    s.n_ended = 0; s.best_step = 0; s.best_slot = 0; s.cnt_tau_T = 0; s.finished_step = T > 0 ? 0 : -1; s.pad = 0;
    p.utt[u] = s;
    p.finished[u] = T > 0 ? 0 : 1;
    p.cells[u] = 0ull;
    p.groups[u] = 0ull;
  }
}

// CTC log-posteriors [U][t_max][V] (frame-major, as an encoder emits them) -> token-major
// xT[u][k][t], t = 1..T_u, so that one candidate's frames are contiguous.  A work-group moves a
// tile of 128 tokens x 32 stored frames through LDS: 512 bytes contiguous per frame on the way in
// (float4 per lane when rows are 16-byte aligned: VEC), whole aligned 128-byte lines per token on
// the way out (rows of xT start on line boundaries, and the tile is cut in STORED frame indices,
// which are one more than the 0-based input frame).  Frames at and beyond T_u are never read.
// Index 0 and the entries after T_u up to the end of their tile (at least four) are set to zero:
// aligned float4 loads of a window may touch them (their terms are masked through the f array,
// which needs finite values there).  Work-groups go round-robin over the eight XCDs; tiles are
// numbered so that each XCD walks through one contiguous eighth of the utterance's tiles, token
// tiles of a 32-frame band one after the other: the lines two neighbouring tiles share are then
// fetched into one L2 instead of two, and each XCD streams through its own region of memory.
// Which eighth an XCD takes rotates with the utterance, so that short utterances (whose last
// eighths are empty) do not leave the same XCDs idle.
// Bound by memory (each value read and written once).  Four float4 per lane and 17 KB per work-group keep more
// work-groups at different points of load and store than eight and 33 KB do: 512 utterances of 250..875 frames, 5000 ids,
// 2397 -> 2280 us, 5.1 TB/s, where a plain copy of the same form reaches 5.7.  64 tokens or 64 frames per tile
// are not faster, nor is a bound on the registers.
// Grid: (8 + 8 * per_xcd, U).  The first column of work-groups sets up the utterances' initial state instead
// (seven idle columns beside it keep the tiles' order over the XCDs).
#define INGEST_TOK 128    // tokens of a tile

template <bool VEC>
__global__ __launch_bounds__(256) void k_ingest(Params p, const float* __restrict__ x, int nvt, int n_tiles,
                                                   int per_xcd) {
  __shared__ __attribute__((aligned(16))) float tile[32][INGEST_TOK + 4];
  constexpr int N4 = INGEST_TOK / 32;                      // float4 per thread: the tile's 32 frames in this many rounds
  constexpr int LPF = INGEST_TOK / 4;                      // lanes per frame

  const int u = blockIdx.y;
  const int bx = (int)blockIdx.x - 8;
  if (bx < 0) {
    if (bx == -8) init_state(p, x, u);
    return;
  }
  const int T = p.lens[u];
  const int g = ((bx - u) & 7) * per_xcd + (bx >> 3);
  if (g >= n_tiles) return;
  const int jt = g / nvt, vt = g - jt * nvt;
  const int d0 = jt * 32;                                // first stored frame index of the tile
  if (d0 > T + 4) return;
  const int v0 = vt * INGEST_TOK;
  const int lane = threadIdx.x % LPF, w = threadIdx.x / LPF;   // (lane of the frame, frames of a round)
  const float* src = x + (size_t)u * p.t_max * p.V;
  float4 r[N4];
  const int v = v0 + 4 * lane;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    const int tt = d0 - 1 + w + (256 / LPF) * i;                   // 0-based input frame of stored index tt + 1
    r[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (tt >= 0 && tt < T) {
      const float* row = src + (size_t)tt * p.V + v;
      if (VEC) {
        if (v < p.V) r[i] = *(const float4*)row;         // V is a multiple of 4 here
      } else {
        if (v + 0 < p.V) r[i].x = row[0];
        if (v + 1 < p.V) r[i].y = row[1];
        if (v + 2 < p.V) r[i].z = row[2];
        if (v + 3 < p.V) r[i].w = row[3];
      }
    }
  }
  float top = 0.0f;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    float4 c;
    c.x = fmaxf(r[i].x, LOG0F); c.y = fmaxf(r[i].y, LOG0F); c.z = fmaxf(r[i].z, LOG0F); c.w = fmaxf(r[i].w, LOG0F);
    top = fmaxf(fmaxf(fmaxf(top, c.x), fmaxf(c.y, c.z)), c.w);
    const int t = w + (256 / LPF) * i;
    *(float4*)&tile[t][(4 * lane) ^ (((t >> 3) & 3) << 2)] = c;   // (swizzle: see the reads below)
  }
  // not a log-posterior: a plain store of the one value that anyone stores.  (An atomic per wave meets all XCDs at one address: 64
  // utterances whose posteriors lie 30 higher, 266 us a launch without the flag, 524 to 579 with the atomic, 273 now.)
  if (__ballot(top > NEAR_X_MAX) != 0ull && (threadIdx.x & 63) == 0) STORE_FLAG(1, &p.uinfo[u].above0);
  __syncthreads();
  float* dst = p.xT + (size_t)u * p.V * p.Tp;
#pragma unroll
  for (int i = 0; i < N4; ++i) {
    const int q = i * 256 + threadIdx.x;
    const int vl = q >> 3, t4 = (q & 7) * 4;             // eight lanes cover one token's 32 frames
    // a wave reads 8 tokens x 8 groups of 4 frames; with rows of 132 floats, frames 8 apart would
    // share banks, so each band of 8 rows keeps its float4 columns in a different order: the lanes
    // of a wave (of a half wave too) fall on distinct banks
    const int vs = vl ^ ((t4 >> 3) << 2);
    const int d = d0 + t4;
    if (v0 + vl < p.V && d < p.Tp) {                     // Tp is a multiple of 4
      float4 o;
      o.x = (d + 0 >= 1 && d + 0 <= T) ? tile[t4 + 0][vs] : 0.0f;
      o.y = (d + 1 <= T) ? tile[t4 + 1][vs] : 0.0f;
      o.z = (d + 2 <= T) ? tile[t4 + 2][vs] : 0.0f;
      o.w = (d + 3 <= T) ? tile[t4 + 3][vs] : 0.0f;
      *(float4*)(dst + (size_t)(v0 + vl) * p.Tp + d) = o;
    }
  }
}
