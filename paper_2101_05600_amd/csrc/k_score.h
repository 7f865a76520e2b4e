// Score kernel: one work-group per (utterance, beam slot) hypothesis g.
//   1. candidate pre-selection: the K ids with the largest attention log-prob, ties to the
//      smaller id.  The row never goes through LDS: every lane keeps its float4 loads in
//      registers.  A pivot that is provably not above the K-th largest value (K of the lanes' maxima
//      reach it; for log-probabilities from counts of the maxima, else found by bisection with ballots), then
//      a short list of the few values that reach it (about 1.2 K), then the K largest of these: up to
//      64 entries are ranked one per lane, up to 128 two per lane, the waves sharing the comparisons; more, or equal
//      values at the K-th place, by quads of lanes.  Rows that do not fit the registers, or with so many values at the
//      pivot that the short list overflows (heavy ties), take a radix select that re-reads the row.
//   2. window [s, e] from g's time indices (the two equations after Eq. (5));
//   3. prefix score of every extension g.c: log-sum over t in [s, e] of
//      f_t + log p^c(z_t = c), f_t = blank variable of g at t-1 if c repeats g's last label,
//      else phi_{t-1}(g)  (Eq. (3) / Eq. (5)); frames run along lanes (16 lanes per
//      candidate, float4 per lane), all of a lane's column loads of a round are issued before the first
//      is consumed; their sums and the largest over the candidate's lanes are taken, then one fused
//      multiply-add and one exp2 per term.  In wide windows over the frames near g's last label first, and over others
//      only where a sum does not outweigh what they could add;
//   4. eos score phi_T(g), joint scores (Eq. (1)), the eos-run test, and the group's
//      best-first list of at most Wb candidates for the per-utterance selection.
// The candidate list of a group is in no particular order and no result depends on it; wherever
// equal scores must be ordered the token id decides.
#pragma once
#include "common.h"

// (every id a candidate, see k_dense.h) one beam slot: its frames,
struct DenseRange {
  int32_t s, e;              // first and last frame whose F is not 0 (none: s > e)
  int32_t far_s, far_e;      // frames at either end of s .. e that the product leaves out at first (far_s -1: no hypothesis)
  __device__ __forceinline__ bool live() const { return far_s >= 0; }
};
struct __align__(64) DenseSlot : DenseRange {
  float low;                 // the sum from which on they cannot count
  int32_t last;
  float mref, inc_rep;       // largest f term M; increment of the candidate that repeats the last label
  double offr, jbase;        // off' + B_r; joint score without this step's terms
  int32_t ref;               // reference frame (HypRec)
  int32_t f_lo, f_hi;        // first and last frame that has an f term
};

// and what its eos extension and its window are
struct DenseEos { double ctc; int32_t s, e; };

// and what its candidates' scores are formed from, beside increments and attention values
struct DenseLeft { double offr, jbase; };

// Joint score (Eq. (1)) of a candidate from its increment and its attention value: the same to the last bit wherever it is formed
template <class S>
__host__ __device__ __forceinline__ double dense_base(double lambda, const S& d) { return fma(lambda, d.offr, d.jbase); }
__host__ __device__ __forceinline__ double dense_sum(double lambda, double base, float inc, float att) { return fma(lambda, (double)inc, fma(1.0 - lambda, (double)att, base)); }
__host__ __device__ __forceinline__ double dense_joint(double lambda, double base, float inc, float att) {
  return inc > LOG0_CLASS ? dense_sum(lambda, base, inc, att) : LOG0D;
}

#define PIVOT_CAP 512     // entries of the short list (all waves together)
#define RADIX_BITS 10

__device__ __forceinline__ float key_to_att(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// base[i], base the same for all lanes and i < 2^30: the byte offset stays in 32 bits, beside a scalar base (an index that
// may be negative costs a lane four instructions for its 64-bit address)
template <class T>
__device__ __forceinline__ T at32(const T* base, int i) { return *(const T*)((const char*)base + (uint32_t)i * (uint32_t)sizeof(T)); }

// ---- candidate selection -----------------------------------------------------------------
// An attention row in the registers of a work-group: 16-byte granules of it (granule g = ids head + 4 g ..
// + 3, g = tid + k * BLOCK), and the at most six ids before the first and after the last whole granule of
// a row that does not start or end on a 16-byte boundary (ex, of id ex_id, in the first lanes; -inf in the others).
// Granules past the row's end hold the last one again.
template <int NV4>
struct RowRegs {
  float4 v[NV4];
  float ex;
  int ex_id, head, n_ex;
};

// The short list: wave w's entries at s_ent[w * WCAP ..], each region padded with zeros to a multiple of four.
// Entries are 64-bit: order-preserving key in the upper word, ~id in the lower, so that one
// integer comparison orders by (value descending, id ascending).
struct ShortList {
  static constexpr int WCAP = PIVOT_CAP / 4;
  static constexpr int GCAP = 64;                          // granules per wave
  int n, n0, n1, n2, n3;     // entries: all, of each wave
  __device__ __forceinline__ int at(int e) const {         // where entry e lies
    return e + (e >= n0 ? WCAP - n0 : 0) + (e >= n0 + n1 ? WCAP - n1 : 0) + (e >= n0 + n1 + n2 ? WCAP - n2 : 0);
  }
  __device__ __forceinline__ int of(int w) const { return w == 0 ? n0 : (w == 1 ? n1 : (w == 2 ? n2 : n3)); }
};

// The pivot: a value that at least K of the lanes' maxima reach (s_mx, complete), found by every wave for itself.
// Bisection on the distance below the row's largest value, in sixteenths up to 32: nine steps of compare, count,
// choose (a way out of the loop when the answer is exact costs more than it saves, and on the upper half of the
// float's bits it would take sixteen steps).  A maximum counts as reaching M - (d + 1) / 16 if floor(16 (M -
// maximum)) <= d; subtraction is monotone and M - that is exact enough for the maximum to be >= the pivot then.
// Where the K-th value lies further down, or is not finite: bisection on the float's upper 16 bits.
// (Pivots of the waves on their own, a quarter of K each, cost less, but the smallest of the four lets 60 values
// through instead of 47 for K = 40, in every fourth row more than the 64 that one wave ranks: one utterance with 40
// candidates 1259 -> 1249 us per decode, a batch of 256 at beam 20 15710 -> 15135 us together with the form below
// that holds three float4 per lane.)
__device__ __forceinline__ float pivot_by_bits(float4 m, int K) {
  const float ninf = -__builtin_huge_valf();
  const int some = (__popcll(__ballot(m.x > ninf)) + __popcll(__ballot(m.y > ninf))) + (__popcll(__ballot(m.z > ninf)) + __popcll(__ballot(m.w > ninf)));
  if (some < K) return ninf;                               // (few ids)
  const uint32_t k0 = att_key(m.x, -1, -2, -2), k1 = att_key(m.y, -1, -2, -2), k2 = att_key(m.z, -1, -2, -2), k3 = att_key(m.w, -1, -2, -2);
  uint32_t thr = 0;
#pragma unroll 1
  for (int bit = 31; bit >= 16; --bit) {
    const uint32_t t = thr | (1u << bit);
    const int c = (__popcll(__ballot(k0 >= t)) + __popcll(__ballot(k1 >= t))) + (__popcll(__ballot(k2 >= t)) + __popcll(__ballot(k3 >= t)));
    if (c >= K) thr = t;
  }
  return thr <= att_key(ninf, -1, -2, -2) ? ninf : key_to_att(thr);
}
template <int BLOCK>
__device__ __forceinline__ float find_pivot(const float* s_mx, int K, float& M) {
  static_assert(BLOCK == 256, "four maxima per lane");
  const float4 m = ((const float4*)s_mx)[threadIdx.x & 63];
  M = row16_max(fmaxf(fmaxf(m.x, m.y), fmaxf(m.z, m.w)));
  M = fmaxf(fmaxf(lane_f(M, 0), lane_f(M, 16)), fmaxf(lane_f(M, 32), lane_f(M, 48)));
  // (a lane without a value: past the end of the scale)
  auto scale = [&](float v) { const float d16 = (M - v) * 16.0f; return d16 < 511.0f ? (int)d16 : 511; };
  const int q0 = scale(m.x), q1 = scale(m.y), q2 = scale(m.z), q3 = scale(m.w);
  int lim = 511;                                           // smallest d found so that K lanes have q <= d
#pragma unroll
  for (int bit = 256; bit > 0; bit >>= 1) {
    const int t = lim - bit;
    const int c = (__popcll(__ballot(q0 <= t)) + __popcll(__ballot(q1 <= t))) + (__popcll(__ballot(q2 <= t)) + __popcll(__ballot(q3 <= t)));
    lim = c >= K ? t : lim;
  }
  return lim < 511 ? M - (float)(lim + 1) * 0.0625f : pivot_by_bits(m, K);   // (uniform, rare)
}

// The same for log-probabilities, whose scale needs no row maximum: sixteenths below zero, counted in LDS by all lanes at once (two
// counts a word, s_hist zeroed), so that a prefix sum over the 512 counts takes the place of nine dependent rounds, and of the row maximum.
// 64 utterances 2760 -> 2699 us a decode, 512 8423 -> 8312, 16 whole utterances 1506 -> 1479; one utterance the same.
// Scores on another scale: values above zero count as zero, and three probabilities above 0.94 there are not, so that K values in the
// first count, or less than K in all of them, send the row to the bisection, which has its scale from the row's maximum (64 utterances
// whose rows lie 20 higher: 8530 us a decode with a list of all that lies above zero, 2868 with bisection alone, 2843 now).
__device__ __forceinline__ void pivot_count(uint32_t* s_hist, float mx) {
  const int q = (int)fmaxf(fminf(-16.0f * mx, 511.0f), 0.0f);
  if (q < 511) atomicAdd(&s_hist[q >> 1], (q & 1) ? 0x10000u : 1u);
}
template <int BLOCK>
__device__ __forceinline__ float find_pivot_hist(const uint32_t* s_hist, const float* s_mx, int K) {
  const int lane = threadIdx.x & 63;
  const uint4 h = ((const uint4*)s_hist)[lane];             // counts 8 * lane .. 8 * lane + 7
  const uint32_t s2 = (h.x + h.y) + (h.z + h.w);
  const int all = (int)((s2 & 0xffffu) + (s2 >> 16));
  const int upto = (int)wave_incl_scan_u32((uint32_t)all, lane);
  const unsigned long long reach = __ballot(upto >= K);
  int n = upto - all, below = 0;                            // (the lane's counts one by one: how many until K are reached)
  auto count = [&](uint32_t w) {
    n += (int)(w & 0xffffu); below += n < K ? 1 : 0;
    n += (int)(w >> 16); below += n < K ? 1 : 0;
  };
  count(h.x); count(h.y); count(h.z); count(h.w);
  const int first = (__ffsll((long long)reach) - 1) & 63, lim = 8 * first + __builtin_amdgcn_readlane(below, first);
  float M;
  if (reach != 0ull && lim > 0) return (float)(lim + 1) * -0.0625f;   // (uniform)
  return find_pivot<BLOCK>(s_mx, K, M);
}

// This wave's part of the short list.  Its granules whose maximum reaches L are packed into LDS (one ballot per
// register; hits are rare: 1 % of a row), then their values are looked at with a lane each.  Returns how many
// values reach L; a region that would overflow stores no more (WCAP + 1 is returned if granules overflowed).
template <int BLOCK, int NV4>
__device__ __forceinline__ int collect_hits(const RowRegs<NV4>& r, const float (&m4)[NV4], float L, int blank_id, int eos_id,
                                            float4* gran, int32_t* gid, unsigned long long* ent) {
  const int tid = threadIdx.x, lane = tid & 63;
  int ngr = 0;                                             // (scalar, like n below: counts of ballots)
  auto pack = [&](bool hit, float4 v, int id) {
    const unsigned long long b = __ballot(hit);
    if (hit) {
      const int pos = ngr + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
      gran[min(pos, ShortList::GCAP - 1)] = v; gid[min(pos, ShortList::GCAP - 1)] = id;
    }
    ngr += __popcll(b);
  };
#pragma unroll
  for (int k = 0; k < NV4; ++k) pack(m4[k] >= L, r.v[k], r.head + 4 * (tid + k * BLOCK));
  if (r.n_ex > 0) {                                        // (uniform)
    const float none = __builtin_nanf("");                 // (never a hit; -inf was one wherever the pivot is -inf)
    pack(tid < r.n_ex && r.ex >= L, make_float4(r.ex, none, none, none), r.ex_id);
  }
  wave_lds_fence();
  const bool linf = (L == -__builtin_huge_valf());         // then blank and eos are hits too (there may be no K candidates)
  int n = 0;
  const int nv = 4 * min(ngr, ShortList::GCAP);
  for (int i0 = 0; i0 < nv; i0 += 64) {
    const int i = i0 + lane;
    const float val = i < nv ? ((const float*)gran)[i] : 0.0f;
    const int id = i < nv ? gid[i >> 2] + (i & 3) : 0;
    const bool none = id == blank_id || id == eos_id;      // not a candidate
    const bool hit = i < nv && val >= L && (linf || !none);
    const unsigned long long b = __ballot(hit);
    if (hit) {
      const int pos = n + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
      const uint32_t u = __float_as_uint(val);
      uint32_t key = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
      if (none) key = 0u;                                  // below a genuine -inf
      if (pos < ShortList::WCAP) ent[pos] = ((unsigned long long)key << 32) | (uint32_t)~id;
    }
    n += __popcll(b);
  }
  if (lane < 3 && n + lane < ((n + 3) & ~3) && n + lane < ShortList::WCAP) ent[n + lane] = 0ull;
  return ngr > ShortList::GCAP ? ShortList::WCAP + 1 : n;
}

// The K largest of a short list of at most 64 entries.  In every wave each lane holds an entry; a wave broadcasts a quarter of
// the entries one after the other (readlane), every lane counts those above its own, and the quarters' counts meet in LDS
// (s_part: a byte per wave and entry).  Each wave for itself over all of them, without the exchange and its barrier, takes a
// tenth more instructions per work-group: decodes of 64 utterances 2842 -> 2797 us, of 512 8546 -> 8438, of one the same.  (A bisection with ballots until exactly K entries are left takes twice as
// long.)  ids: this wave's copy of their ids; s_av: their values, by the first wave.  False (in all waves alike) if equal
// values straddle the K-th place.
__device__ __forceinline__ bool take_k(int w, const unsigned long long* s_ent, const ShortList& sl, int K, uint32_t* s_part, int32_t* ids, float* s_av) {
  const int lane = threadIdx.x & 63, turned = (lane + 16 * w) & 63;   // (the wave's quarter: its lanes 0 to 15)
  const unsigned long long me = s_ent[sl.at(min(lane, sl.n - 1))];
  const uint32_t v = ((const uint32_t*)s_ent)[2 * sl.at(min(turned, sl.n - 1)) + 1];
  const int above = lanes_above<16>(turned < sl.n ? v : 0u, 16);
  ((uint8_t*)s_part)[4 * turned + w] = (uint8_t)above;
  lds_barrier();
  const int rank = (int)((s_part[lane] * 0x01010101u) >> 24);   // (the bytes' sum, at most 63)
  const bool take = lane < sl.n && rank < K;
  const unsigned long long b = __ballot(take);
  if (__popcll(b) != K) return false;                      // (equal values have equal ranks)
  const int pos = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u));
  if (take) {
    ids[pos] = (int)~(uint32_t)me;
    if (w == 0) s_av[pos] = key_to_att((uint32_t)(me >> 32));
  }
  return true;
}

// The same of 65 to 128 entries, two per lane (60 candidates: about 73 entries), whose ranking by quads of lanes, each reading the whole
// list from LDS, took 2.1 of a work-group's 10.4 us (256 utterances, beam 20, 60 candidates: a decode 13840 -> 13570 us).  Rows of
// 50 candidates have that many now and then.
__device__ __forceinline__ bool take_k_of_128(int w, const unsigned long long* s_ent, const ShortList& sl, int K, uint32_t* s_part, int32_t* ids, float* s_av) {
  const int lane = threadIdx.x & 63, turned = (lane + 16 * w) & 63;
  const uint32_t* hi = (const uint32_t*)s_ent + 1;
  const uint32_t a = hi[2 * sl.at(turned)], b1 = hi[2 * sl.at(min(64 + turned, sl.n - 1))], b = 64 + turned < sl.n ? b1 : 0u;
  int na = 0, nb = 0;
  above8<0>(a, a, b, na, nb); above8<8>(a, a, b, na, nb);
  if (64 + 16 * w < sl.n) {                                // (uniform)
    above8<0>(b, a, b, na, nb);
    if (72 + 16 * w < sl.n) above8<8>(b, a, b, na, nb);
  }
  ((uint8_t*)s_part)[4 * turned + w] = (uint8_t)na;
  ((uint8_t*)s_part)[256 + 4 * turned + w] = (uint8_t)nb;
  lds_barrier();
  auto rank = [&](int e) { return (int)((s_part[e] * 0x01010101u) >> 24); };   // (at most 127)
  const bool ta = rank(lane) < K, tb = 64 + lane < sl.n && rank(64 + lane) < K;
  const unsigned long long ba = __ballot(ta), bb = __ballot(tb);
  if (__popcll(ba) + __popcll(bb) != K) return false;      // (equal values have equal ranks)
  auto put = [&](int pos, int e) {
    const unsigned long long me = s_ent[sl.at(e)];
    ids[pos] = (int)~(uint32_t)me;
    if (w == 0) s_av[pos] = key_to_att((uint32_t)(me >> 32));
  };
  auto before = [&](unsigned long long m) { return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)); };
  const int pa = before(ba), pb = __popcll(ba) + before(bb);
  if (ta) put(pa, lane);
  if (tb) put(pb, 64 + lane);
  return true;
}

// How many entries of the short list exceed `me`, the quad's lanes together.
__device__ __forceinline__ int list_rank_quad(const unsigned long long* s_ent, const ShortList& sl, unsigned long long me,
                                              int part) {
  int rank = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const ulonglong2* e2 = (const ulonglong2*)(s_ent + w * ShortList::WCAP);
    const int q = (sl.of(w) + 3) >> 2;
    for (int i = part; i < q; i += 4) {
      const ulonglong2 a = e2[2 * i], b = e2[2 * i + 1];
      rank += ((int)(a.x > me) + (int)(a.y > me)) + ((int)(b.x > me) + (int)(b.y > me));
    }
  }
  rank += dpp_i<0xB1, 0xf>(0, rank);                       // quad_perm [1,0,3,2]
  rank += dpp_i<0x4E, 0xf>(0, rank);                       // quad_perm [2,3,0,1]
  return rank;
}

// Radix select on the order-preserving keys (10 + 10 + 10 + 2 bits) straight from the row in
// global memory, then an ordered compaction (ascending ids).
template <int BLOCK>
__device__ __forceinline__ void select_radix(const float* __restrict__ arow, int V, int K, int blank_id, int eos_id,
                                          uint32_t* s_hist, uint32_t* s_scan, uint32_t* s_sel,
                                          bool use_lds, int32_t* out_lds, float* out_att_lds, int32_t* out_g) {
  const int tid = threadIdx.x;
  uint32_t prefix = 0, pmask = 0, krem = (uint32_t)K;
#pragma unroll 1
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = pass == 0 ? 22 : (pass == 1 ? 12 : (pass == 2 ? 2 : 0));
    const int bits = pass == 3 ? 2 : RADIX_BITS;
    const uint32_t bmask = (1u << bits) - 1u;
    const int nb = 1 << bits;
    __syncthreads();
    for (int i = tid; i < nb; i += BLOCK) s_hist[i] = 0;
    __syncthreads();
    for (int i = tid; i < V; i += BLOCK) {
      uint32_t k = att_key(arow[i], i, blank_id, eos_id);
      if ((k & pmask) == prefix) atomicAdd(&s_hist[(k >> shift) & bmask], 1u);
    }
    __syncthreads();
    // find the bin in which the count of larger-or-equal keys reaches krem
    const int per = nb / BLOCK > 0 ? nb / BLOCK : 1;
    uint32_t local = 0;
    const int b_lo = tid * per;
    if (b_lo < nb)
      for (int b = 0; b < per; ++b) local += s_hist[b_lo + b];
    uint32_t total;
    uint32_t excl = block_excl_scan_u32<BLOCK>(local, s_scan, &total);
    uint32_t above = total - excl - local;                   // keys in bins owned by higher threads
    if (b_lo < nb && above < krem && above + local >= krem) {
      uint32_t run = above;
      for (int b = per - 1; b >= 0; --b) {
        uint32_t h = s_hist[b_lo + b];
        if (run + h >= krem) { s_sel[0] = (uint32_t)(b_lo + b); s_sel[1] = krem - run; break; }
        run += h;
      }
    }
    __syncthreads();
    prefix |= s_sel[0] << shift;
    pmask |= bmask << shift;
    krem = s_sel[1];
  }
  // prefix = key of the K-th best; krem = how many of the keys equal to it are taken
  // (those with the smallest ids).  Ordered compaction, contiguous id chunk per thread; the
  // two counts are scanned separately (either can be as large as the row).
  const int chunk = (V + BLOCK - 1) / BLOCK;
  const int i0 = min(V, tid * chunk), i1 = min(V, i0 + chunk);
  uint32_t gt = 0, eq = 0;
  for (int i = i0; i < i1; ++i) {
    uint32_t k = att_key(arow[i], i, blank_id, eos_id);
    gt += (k > prefix); eq += (k == prefix);
  }
  uint32_t total;
  const uint32_t gt_before = block_excl_scan_u32<BLOCK>(gt, s_scan, &total);
  uint32_t eq_before = block_excl_scan_u32<BLOCK>(eq, s_scan, &total);
  uint32_t pos = gt_before + min(eq_before, krem);
  for (int i = i0; i < i1; ++i) {
    const float a = arow[i];
    uint32_t k = att_key(a, i, blank_id, eos_id);
    bool take = (k > prefix) || (k == prefix && eq_before < krem);
    if (k == prefix) ++eq_before;
    if (take && pos < (uint32_t)K) {
      if (use_lds) { out_lds[pos] = i; out_att_lds[pos] = a; }
      else out_g[pos] = i;
      ++pos;
    }
  }
}

// ---- log-sum-exp pieces -----------------------------------------------------------------------
// Natural units throughout: a term is f + x, rounded once, and the largest term M goes into the result as it is.  (With
// f and x scaled to units of log 2 a term was rounded twice and M a third time on the way back: 1.3 to 1.4 times the
// rounding error, for the same number of instructions and the same time: 50.6 / 50.9 us a launch at beam 20, 256 utterances.)
#define L2E 1.4426950408889634f
#define LN2 0.6931471805599453f

template <int LPC>
__device__ __forceinline__ float chain_max(float m) {
  static_assert(LPC == 16 || LPC == 64, "a candidate's lanes are one DPP row or one wave");
  m = row16_max(m);
  if (LPC == 64) m = fmaxf(fmaxf(lane_f(m, 0), lane_f(m, 16)), fmaxf(lane_f(m, 32), lane_f(m, 48)));
  return m;
}
template <int LPC>
__device__ __forceinline__ float chain_sum(float s) {
  s = row16_sum(s);
  if (LPC == 64) s = (lane_f(s, 0) + lane_f(s, 16)) + (lane_f(s, 32) + lane_f(s, 48));
  return s;
}

// The sum of a candidate's terms over its LPC lanes: M the largest term so far (of all lanes), s this lane's share of the
// sum of 2^(term log2 e - c), c = M log2 e as fp32 rounds it (chain_ref).  One addition, one maximum, one fused multiply-add, one exp2
// and one addition per term.  The fused multiply-add rounds only the distance from M; what c lacks of M log2 e is known
// exactly and taken out once, in chain_finish.  A reference below -2^28 is not used (c = 0, s = 0): there what c lacks
// would leave the range of exp2, and neighbouring floats lie 32 apart, so that M is the sum; log0 is of that kind.
#define LSE_DEEP (-268435456.0f)
struct ChainSum { float M, s; };
__device__ __forceinline__ float chain_ref(float M) { return (M < LSE_DEEP ? 0.0f : M) * L2E; }

template <int N>
__device__ __forceinline__ float terms(const float4 (&x)[N], const float4 (&f)[N], float (&v)[4 * N]) {   // their maximum
#pragma unroll
  for (int i = 0; i < N; ++i) {
    v[4 * i] = x[i].x + f[i].x; v[4 * i + 1] = x[i].y + f[i].y;
    v[4 * i + 2] = x[i].z + f[i].z; v[4 * i + 3] = x[i].w + f[i].w;
  }
  float m = v[0];
#pragma unroll
  for (int i = 1; i < 4 * N; ++i) m = fmaxf(m, v[i]);
  return m;
}
template <int N>
__device__ __forceinline__ float exp_sum(const float (&v)[N], float c) {
  float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
  for (int i = 0; i < N; i += 2) {
    s0 += __builtin_amdgcn_exp2f(fmaf(v[i], L2E, -c));
    s1 += __builtin_amdgcn_exp2f(fmaf(v[i + 1], L2E, -c));
  }
  return s0 + s1;
}
// N float4 of a column against the f terms
template <int LPC, int N>
__device__ __forceinline__ ChainSum chain_first(const float4 (&x)[N], const float4 (&f)[N]) {
  float v[4 * N];
  ChainSum a;
  a.M = chain_max<LPC>(terms<N>(x, f, v));
  a.s = exp_sum(v, chain_ref(a.M));
  return a;
}
template <int LPC, int N>
__device__ __forceinline__ void chain_more(ChainSum& a, const float4 (&x)[N], const float4 (&f)[N]) {
  float v[4 * N];
  const float c0 = chain_ref(a.M);
  a.M = fmaxf(a.M, chain_max<LPC>(terms<N>(x, f, v)));
  const float c = chain_ref(a.M);
  a.s = a.s * __builtin_amdgcn_exp2f(fminf(c0 - c, 0.0f)) + exp_sum(v, c);   // (c falls only from an unused 0, with s = 0)
}
template <int LPC>
__device__ __forceinline__ float chain_finish(const ChainSum& a) {
  const float s = chain_sum<LPC>(a.s);
  float r = a.M + (__builtin_amdgcn_logf(s) - fmaf(a.M, L2E, -chain_ref(a.M))) * LN2;
  r = a.M < LSE_DEEP ? a.M : r;
  return (a.M < LOG0_CLASS) ? LOG0F : r;
}

// The same where lanes go their own ways (sums in two parts, sums redone frame by frame): m the largest term of the lane
// so far, s the sum of e^(term - m).
struct Lse { float m, s; };
__device__ __forceinline__ Lse lse_block(float4 x, float4 f) {
  const float t0 = x.x + f.x, t1 = x.y + f.y, t2 = x.z + f.z, t3 = x.w + f.w;
  Lse r;
  r.m = fmaxf(fmaxf(t0, t1), fmaxf(t2, t3));
  r.s = (__builtin_amdgcn_exp2f((t0 - r.m) * L2E) + __builtin_amdgcn_exp2f((t1 - r.m) * L2E)) +
        (__builtin_amdgcn_exp2f((t2 - r.m) * L2E) + __builtin_amdgcn_exp2f((t3 - r.m) * L2E));
  return r;
}
__device__ __forceinline__ Lse lse_join(Lse a, Lse b) {
  Lse r;
  r.m = fmaxf(a.m, b.m);
  r.s = a.s * __builtin_amdgcn_exp2f((a.m - r.m) * L2E) + b.s * __builtin_amdgcn_exp2f((b.m - r.m) * L2E);
  return r;
}
// all lanes of a candidate together
template <int LPC>
__device__ __forceinline__ float lse_finish(Lse a) {
  const float M = chain_max<LPC>(a.m);
  const float s = chain_sum<LPC>(a.s * __builtin_amdgcn_exp2f((a.m - M) * L2E));
  return (M < LOG0_CLASS) ? LOG0F : M + fast_logf(s);      // (s >= 1: the largest term contributes 1)
}

// Block-wide maximum / sum (logits mode: log-sum-exp of a whole attention row).  The per-lane
// partials are floats; partial sums are added in fp64.
template <int BLOCK>
__device__ __forceinline__ float block_max_f(float m, float* s_red /*[BLOCK / 64]*/) {
  constexpr int NW = BLOCK / 64;
  m = row16_max(m);
  m = fmaxf(fmaxf(lane_f(m, 0), lane_f(m, 16)), fmaxf(lane_f(m, 32), lane_f(m, 48)));
  lds_barrier();
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = m;
  lds_barrier();
  float M = s_red[0];
#pragma unroll
  for (int i = 1; i < NW; ++i) M = fmaxf(M, s_red[i]);
  return M;
}
template <int BLOCK>
__device__ __forceinline__ double block_sum_d(float sum, double* s_d /*[BLOCK / 64]*/) {
  constexpr int NW = BLOCK / 64;
  sum = row16_sum(sum);
  const double ws = ((double)lane_f(sum, 0) + (double)lane_f(sum, 16)) +
                    ((double)lane_f(sum, 32) + (double)lane_f(sum, 48));
  lds_barrier();
  if ((threadIdx.x & 63) == 0) s_d[threadIdx.x >> 6] = ws;
  lds_barrier();
  double tot = 0.0;
#pragma unroll
  for (int i = 0; i < NW; ++i) tot += s_d[i];
  return tot;
}

// Order-preserving 64-bit image of a joint score whose lowest mantissa bits (`mask`) hold `low` instead: one integer
// comparison then orders by (score descending, low descending).  0 = not a competitor.
__device__ __forceinline__ unsigned long long joint_key(double J, unsigned long long mask, int low, bool valid) {
  if (!valid) return 0ull;
  const unsigned long long b = (unsigned long long)__double_as_longlong(J);
  const unsigned long long k = (b >> 63) ? ~b : (b | 0x8000000000000000ull);
  return (k & ~mask) | (unsigned long long)low;
}

// Grid: (1 << sh, Wb, ceil(U / (1 << sh))), sh = bits 4-7 of flags: utterance z * 2^sh + x, beam slot y.  With sh = 3 the
// work-groups of an utterance share an XCD (work-groups go round-robin over the eight), and with it the L2 in
// which a column that several beam slots score is fetched once.
// flags bit 0: the whole row can be held in registers (NV4 * BLOCK granules); bit 1: rows are fetched before it is known whether the
// utterance has finished (up to a work-group per compute unit: the dead slots' rows cost nobody's bandwidth then; one
// utterance 1021 -> 1011 us a decode, 21 with a batch-wide window 1443 -> 1432, 16 whole utterances within the noise), and the four
// waves share the ranking of the group's list, with one more barrier (one utterance 965 -> 942, 21 with a batch-wide window 1448 -> 1432,
// 16 whole utterances 1397 -> 1368; 384 to 1280 groups within half a per cent either way, 5120 slower by that).
// The arguments in front of the parameter block are what the first loads of a work-group need (the records
// of the current buffer = p.rec[cur], p.uinfo, p.finished as words, the attention rows, Wb, p.V): as plain
// leading arguments they are handed to the wave in registers when it starts (kernel-argument preload),
// so that the record's load does not have to wait for a load of the argument block first.
// CB candidates per chain of 16 lanes and round, IT float4 of each in flight.  Windows of up to 128 frames: 3 x 2, up to 192:
// 2 x 3, both with a loop per candidate for what lies beyond; the same registers, and one more frame round costs what one
// more candidate round does.  Wider windows, whole utterances: 3 x 2 for 33 to 48 candidates, rounds of all three together, 2 x 3 for other
// numbers, which would leave places of three empty (create_impl).  NEAR, all but the first: at first over the frames near g's last label only (HypRec::near_frames).  500 frames, 16 utterances, beam 10, 40
// candidates, peaked posteriors: 11.5 -> 9.0 us a launch against 2 x 4 over all frames; flat ones: the same to 2 %, and against one
// candidate per wave (4 float4 per lane) at 1500 frames a decode of 16 utterances 9.4 -> 7.2 ms.  Margins of 80 (256 utterances of
// 1500 frames, beam 20, 60 candidates): a decode 14362 -> 14167 us; with 3 x 2 there 14530.  The first form has nothing to gain.
// Whole utterances with the eos-run rule are armed at every step; summed over all frames they took up to a quarter longer than
// with one candidate per wave (498 utterances of 663 to 1007 frames, beam 4: 6.6 -> 8.3 ms; near frames first 6.5; 122 of 590 to
// 1484, beam 19, 59 candidates: 17.4 -> 18.0 and 11.2).
// More than 64 candidates: 3 x 2, 2 x 3 as above, wider windows 2 x 4 in rounds of both candidates together, all frames (16 whole utterances
// of 200 to 500 frames, 256 candidates: 8900 us a decode with 3 x 2, whose last round is two thirds empty, 8470; of 1500 frames, 128
// candidates 4890 -> 4270, one candidate per wave 5540).  With the eos-run rule armed the two parts of the sums run together too:
// candidate by candidate, a round's loads after the other's, 1500 frames and 100 candidates take 7260 us a decode, together 4600.
// NV4: granules of the row per lane.  BIGK: more candidates per hypothesis than one wave ranks (K > 64, or ids
// beyond 65535).  Only that form of the
// kernel carries the paths for it: candidate arrays in global memory when K exceeds the work-group, the exact
// ranking by the whole work-group, the eos-run rule's work-group-wide path (a second sum beside the first in
// the column pass, the test across all waves).  They cost registers that the common form does without.
template <int BLOCK, int CB, int IT, int NV4, bool NEAR, bool BIGK>
__global__ __launch_bounds__(BLOCK, (BIGK || NV4 > 10 ? 4 : (NV4 <= 5 ? (NEAR && IT == 2 ? 6 : 7) : 5))) void k_score(const HypRec* __restrict__ rec_now,
                                                 const UttInfo* __restrict__ uinfo, const uint32_t* __restrict__ fin_words,
                                                 const float* __restrict__ att, int Wb, int V, int flags, int l, int U,
                                                 ScoreArgs p, ScoreLate late_args) {
  constexpr int LPC = 16;                                  // lanes per candidate: a DPP row
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(16) float s_mx[BLOCK];              // the lanes' maxima
  __shared__ int s_cnt[BLOCK / 64];                        // short list: entries per wave
  __shared__ __align__(16) int32_t s_wid[BIGK ? 1 : BLOCK];              // the K candidates, each wave's own copy
  __shared__ uint32_t s_scan[BLOCK / 64 + 1];
  __shared__ uint32_t s_sel[2];
  __shared__ float s_e2w[(BLOCK / 64) * MAX_EOS_RUN + 1];
  __shared__ int s_nvalid;
  __shared__ __align__(8) float s_red[4 * (BLOCK / 64)];   // per wave: floats (a row's maxima), then doubles (its sums)
  __shared__ float s_lse;                                  // raw scores in: the row's log-sum-exp
  __shared__ double s_eos[5];                              // eos scores, jbase, offr and 1 - lambda, computed early, needed again at the end
  __shared__ float s_e2f[2 * MAX_EOS_RUN];                 // eos-run rule: f terms of the last R frames (both kinds)

  const int tid = threadIdx.x, w = uni(tid >> 6);
  const int sh = (flags >> 4) & 15;
  const int u = (int)((blockIdx.z << sh) + blockIdx.x);
  const int grp = u * Wb + (int)blockIdx.y;
  // (the utterance's finished byte is fetched as part of its aligned word: a uniform word load
  // can take the scalar path, a byte load cannot)
  uint32_t fin_word = fin_words[u >> 2];
  TRACE_DECL;
  // ---------------- the attention row -----------------------------------------------------------
  // A running utterance's rows are fetched before the records are there, all loads in flight together: nearly all of its slots hold
  // hypotheses, and a work-group's time is 2 us until its record is there and 1.8 until its row is (256 utterances, beam 20, 13570 ->
  // 13449 us a decode, eight instead of seven work-groups on a compute unit among them; 48 utterances of 10000 ids 2395 -> 2335).  In
  // small batches without asking for the flag either.  Not rows of up to 3072 ids, which are soon there: the record first, a live slot's row once it
  // is there (2300 ids: 128 utterances 1997 -> 1980 us a decode, 512 4593 -> 4561, 256 at beam 20 4176 -> 4139, 64 the same); nor, with more than 64
  // candidates, rows of up to 5120 (100 of 2300 ids, 128 utterances 4310 -> 4250, 200 of 3000 11530 -> 11440, 100 of 5000 4940 -> 4900; longer rows
  // 5575 -> 5535 the other way).  With one candidate per hypothesis the first slot alone ever holds one (the last slot that can is in flags from bit 8 on: 256 utterances, beam 20, 5000 ids,
  // 3080 -> 2480); a row that no registers hold is not waited for (48 of 20000 ids 18460 -> 18210 to 18410, by the build).  Whole
  // 16-byte granules by the lanes in turn; what a row that is not aligned has before and after them by the first lanes.
  const float* arow = att + (size_t)grp * V;
  const bool in_regs = (flags & 1) != 0;
  RowRegs<NV4> row;
  row.head = (int)((0u - (unsigned)((uintptr_t)arow >> 2)) & 3u);
  const int ng = (V - row.head) >> 2;                      // whole granules
  const int tail = V - row.head - 4 * ng;
  row.n_ex = row.head + tail;
  row.ex_id = tid < row.head ? tid : row.head + 4 * ng + (tid - row.head);
  row.ex = -__builtin_huge_valf();
  // (each row is read once: past the L2, whose lines the columns and the state need again.  512 utterances 29.2 -> 27.9 us a launch,
  // 256 of 1500 frames at beam 20 46.6 -> 45.9, 64 utterances the same.  Not long rows with many candidates, which mostly end in the
  // radix selection that reads them again: 26 utterances, 11520 ids, 141 candidates 23050 -> 21130 us a decode; up to 5120 ids 2 % more
  // for 200 candidates, 2 % less for 100)
  auto fetch_row = [&]() {
    const char* a4 = (const char*)(arow + row.head);
#pragma unroll
    for (int k = 0; k < NV4; ++k) {
      const f32x4* at = (const f32x4*)(a4 + 16u * (uint32_t)min(tid + k * BLOCK, ng - 1));
      const f32x4 v = BIGK && NV4 > 5 ? *at : LOAD_ASIDE(at);
      row.v[k] = make_float4(v[0], v[1], v[2], v[3]);
    }
    if (tid < row.n_ex) row.ex = at32(arow, row.ex_id);
  };
  const bool early = (flags & 2) != 0;
  constexpr bool AHEAD = NV4 > (BIGK ? 5 : 3);
  int rec_at = grp, ui_at = u;                             // (OPAQUE: loads that are not waited for together with the flag)
  if (AHEAD) {
    int go = in_regs && u < U && (int)blockIdx.y <= flags >> 8;
    if (!early && (NV4 < 16 || in_regs)) { OPAQUE(fin_word); go &= ((fin_word >> (8 * (u & 3))) & 0xffu) == 0u; }   // (up to 10240 ids: always there)
    if (go) fetch_row();
    OPAQUE(rec_at); OPAQUE(ui_at);
  }
  // g's record and the utterance's constants: one 64-byte line and one 32-byte entry
  // through the scalar path (uniform addresses, nothing in this kernel writes them)
  const HypRec rec = rec_now[rec_at];
  const UttInfo ui = uinfo[ui_at];
  if (!AHEAD && in_regs && early && u < U) fetch_row();
  PIN4(rec.live, rec.off, ui.BT, fin_word);
  PIN4(p.xT, p.Bcum, p.gphi, p.gb);
  PIN4(p.lambda, p.beta, p.off_f, p.mode);
  PIN4(p.Tp, p.K, p.win_m1, p.eos_run);
  // (not all of the block: with four more the scalar registers run out and part of it is loaded twice, 35 -> 36.6 us
  // a launch at 512 utterances)
  const int dead = (int)((fin_word >> (8 * (u & 3))) & 0xffu) | (rec.live == 0);
  const int K = p.K;
  const bool smallk = !BIGK || (K <= BLOCK);
  const int T = ui.T;
  const int tau = rec.tau, tau_end = rec.tau_end;
  const int rs = rec.rs, re = rec.re, last = rec.last;
  const double off = rec.off, acum = rec.att;
  if (grp == 0 && w == BLOCK / 64 - 1) {                   // (not in wave 0, which finishes last)
    const ScoreLatePtr q = score_late(late_args);
    publish_progress(q->host_progress, q->n_finished, l);
    // batch-wide window: clear the slot the select kernel of this step will fill for the next one
    if (!(p.mode & SC_UNION_UTT) && tid == BLOCK - 1) {
      q->union_win[2 * ((l + 1) & 1)] = 0x7fffffff;
      q->union_win[2 * ((l + 1) & 1) + 1] = -1;
    }
  }
  if ((p.mode & SC_UNION_UTT) && blockIdx.y == 0 && tid == BLOCK - 1 && u < U) {
    int32_t* sh_u = score_late(late_args)->union_win + 2 * ((size_t)((l + 1) & 1) * U + u);
    sh_u[0] = 0x7fffffff; sh_u[1] = -1;
  }
  if (dead) {
    // (the grid is whole eights of utterances; those past the last are dead here too)
    if (tid == 0 && u < U) score_late(late_args)->grp[grp] = GroupOut{0, 0, 0, -1, LOG0D, LOG0D, 0, {0, 0, 0, 0, 0, 0}};
    return;
  }
  if (!AHEAD && in_regs && !early) fetch_row();

  TRACE_MARK(0);
  uint32_t* s_work = (uint32_t*)(smem);
  // (the radix histogram, or) the short list, and the granules that hold its values
  unsigned long long* s_ent = (unsigned long long*)s_work;
  float4* s_gran = (float4*)(smem + p.off_f);             // (the f terms are staged when these are done with)
  int32_t* s_gid = (int32_t*)(s_gran + 4 * ShortList::GCAP);
  float* s_F = (float*)(smem + p.off_f);                  // f terms
  float* s_Fb = s_F + p.wp_max;
  // per-candidate arrays of the group (K <= BLOCK): sort key and joint score (8 bytes each), then
  // id, prefix-score increment, attention value, eos-run scratch (4 bytes each)
  const int Ks = BIGK ? (smallk ? K : 0) : 64;
  unsigned long long* s_key = (unsigned long long*)(smem + p.off_small);
  double* s_J = (double*)(s_key + Ks);                     // joint score as computed (NaN kept)
  int32_t* s_cid = (int32_t*)(s_J + Ks);                   // only touched when smallk
  float* s_inc = (float*)(s_cid + Ks);
  float* s_av = s_inc + Ks;
  float* s_pre = s_av + Ks;                                // BIGK: prefix score without the last R frames
  int32_t* g_cid = BIGK ? score_late(late_args)->cand_id + (size_t)grp * K : nullptr;   // (many candidates, like the others below)

  // raw scores in: the row holds unnormalised scores; log_softmax is folded in here (the order of
  // the ids is the same, only the values the scores use are shifted by the row's log-sum-exp)
  const bool logits = (p.mode & SC_LOGITS) != 0;
  float row_lse = 0.0f;
  const float x_eos = arow[p.eos_id];
  if (logits && !in_regs) {
    float m = -3.0e38f, sum = 0.0f;
    for (int i = tid; i < V; i += BLOCK) m = fmaxf(m, arow[i]);
    const float M = block_max_f<BLOCK>(m, s_red);
    for (int i = tid; i < V; i += BLOCK) sum += __expf(arow[i] - M);
    row_lse = (float)((double)M + log(block_sum_d<BLOCK>(sum, (double*)(s_red + BLOCK / 64))));
    if (tid == 0) s_lse = row_lse;                         // (read after further barriers)
  }

  // the pivot's counts (in the place of the candidates' ids, which come later), cleared while the row is on its way
  const bool hist = !BIGK && in_regs && !logits;
  if (hist) { s_wid[tid] = 0; lds_barrier(); }

  // ---------------- window (needs only g's record) ----------------------------------------
  int s = l > 1 ? l : 1, e = T;
  if (p.mode & SC_UNION) {            // s^l = min_ij s_ij, e^l = max_ij e_ij (last two equations of Sec. 3.2.3)
    int lo = 0x7fffffff, hi = -1;
    if (p.mode & SC_UNION_UTT) {                           // the unfinished utterances' shares together
      const int32_t* shares = score_late(late_args)->union_win + 2 * (size_t)(l & 1) * U;
      for (int i = tid; i < U; i += BLOCK)
        if (((fin_words[i >> 2] >> (8 * (i & 3))) & 0xffu) == 0u) { lo = min(lo, shares[2 * i]); hi = max(hi, shares[2 * i + 1]); }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) { lo = min(lo, __shfl_xor(lo, o)); hi = max(hi, __shfl_xor(hi, o)); }
      if ((tid & 63) == 0) { s_cnt[w] = lo; s_scan[w] = (uint32_t)hi; }
      lds_barrier();
#pragma unroll
      for (int i = 0; i < BLOCK / 64; ++i) { lo = min(lo, s_cnt[i]); hi = max(hi, (int)s_scan[i]); }
      lo = uni(lo); hi = uni(hi);
      lds_barrier();                                       // (both arrays serve the selection below)
    } else { const int32_t* share = score_late(late_args)->union_win + 2 * (l & 1); lo = share[0]; hi = share[1]; }
    if (p.win_m1 >= 0) s = max(s, lo - p.win_m1);
    if (p.win_m2 >= 0) e = min(e, hi);
  } else {
    if (p.win_m1 >= 0) s = max(s, tau - p.win_m1);
    if (p.win_m2 >= 0) e = min(e, tau_end + p.win_m2);
  }
  int bad = 0;
  s = clamped(s, 1, T + 1, ERR_WINDOW, bad);               // (an empty window is e < s; its loads stay inside the row)
  e = clamped(e, -1, T, ERR_WINDOW, bad);
  report(p, bad);
  const int W = e >= s ? e - s + 1 : 0;
  const int t0 = s & ~3;                                   // column loads start on a 16-byte boundary
  const int n4 = W > 0 ? ((e - t0) >> 2) + 1 : 0;
  auto eos_run_armed = [&]() {
    return (p.end_flags & 4) && p.eos_run > 0 && T >= p.eos_run && W > 0 && e == T && re == T && max(s, rs) <= T - p.eos_run + 1;
  };
  // NEAR: the float4 of the window that the sums run over at first, j0 .. j1 - 1, those with frames near g's last label (HypRec),
  // and the sum from which on the others cannot count.  With the eos-run rule armed the sums stop short of the last frames: where
  // less than NEAR_ENOUGH of the frames behind g's last label come before those, most sums would fall below the bound, and all frames
  // are summed at once.  Where they fill half of their rounds of loads or less, posteriors are sharp: the rest of the rounds goes to the frames on
  // both sides, and often no sum is left that the others could count for (margins of 80, three times as sharp: 2260 -> 2020 us a decode;
  // always, the bytes cost more: long recordings at beam 20 13810 -> 14170)
  int j0 = 0, j1 = n4;
  float sum_low = -3.0e38f;
  if (NEAR && n4 > 0) {
    const int a = max(s, (int)(rec.near_frames & 0xffffu) + 1), b = min(e, (int)(rec.near_frames >> 16) + 1);
    if (a <= b && (!eos_run_armed() || tau + NEAR_ENOUGH <= T - p.eos_run)) { j0 = (a - t0) >> 2; j1 = ((b - t0) >> 2) + 1; }
    const int m = (j1 - j0 + LPC * IT - 1) / (LPC * IT) * (LPC * IT);
    if (2 * (j1 - j0) <= m) { j0 = max(0, min(j0 - (m - (j1 - j0)) / 2, n4 - m)); j1 = min(j0 + m, n4); }
    if (j1 - j0 < n4) sum_low = NEAR_MARGIN - NEAR_DEPTH + fast_logf((float)(4 * (n4 - (j1 - j0))));
  }
  const float* gphi = p.gphi + (size_t)grp * p.Tp;
  const float* gb = p.gb + (size_t)grp * p.Tp;
  // Stored forward variables have the per-frame reference B_t taken out (see Params::Bcum); all
  // increments of this step are relative to off'(g) + B_r, r = g's reference frame
  const double* Bu = p.Bcum + (size_t)u * p.Tp;
  const double Bref = rec.bref;
  const double offr = off + Bref;
  const double BT = ui.BT - Bref;                          // B_T - B_r

  // What the f terms, the eos score and the eos-run rule need of g's state is requested here, behind the row, and
  // used after the candidate selection: nothing waits for it before.
  auto in_range = [&](int t) { return t >= s && t <= e && t - 1 >= rs && t - 1 <= re; };   // frame t has an f term
  const int pr0 = min(max(t0 + tid - 1, 0), T);
  const float f0_p = at32(gphi, pr0), f0_b = at32(gb, pr0);
  const double f0_B = at32(Bu, pr0);
  float eos_p = LOG0F;
  if (rs <= T && re >= T) eos_p = gphi[T];

  TRACE_MARK(1);
  const int R = p.eos_run;
  const bool e2 = eos_run_armed();
  constexpr bool wave_rank = !BIGK;                        // the group's list is ranked by one wave on 64-bit keys
  // eos-run rule with few candidates: the f terms of the last R frames are kept apart (and left out of the
  // window's arrays), so that the sums below stop at frame T - R; the first wave completes them at the end
  const bool e2w = e2 && wave_rank;
  const bool e2g = BIGK && e2 && !wave_rank;               // the rule by the whole work-group (many candidates)
  // the arrays hold whole rounds of LPC * IT float4 from j0 on (log0 past the window's end), so that the sums need no bounds
  const int n4r = j0 + max(1, (n4 - j0 + LPC * IT - 1) / (LPC * IT)) * (LPC * IT);   // (not NEAR: j0 = 0)
  const double lam = p.lambda, jbase = (1.0 - lam) * acum + p.beta * (double)l;
  // eos-run rule: E_t = phi_t(g) of frame t = T-R+1+tid
  float e2_Et = LOG0F, e2_p = LOG0F;
  double e2_B = 0.0;
  if (e2 && tid < R) { const int t = T - R + 1 + tid; e2_p = at32(gphi, t); e2_B = at32(Bu, t); }
  // The f terms of the window into LDS:
  // gamma_{t-1}(g) - off' - B_r = stored_{t-1} + (B_{t-1} - B_r); far from r the second part is
  // large and coarse in fp32, and the term is then negligible by that same factor
  auto stage_state = [&]() {
    float ph = f0_p, b = f0_b;
    double B = f0_B;

    for (int i = tid; i < 4 * n4r; i += BLOCK) {
      const int t = t0 + i;
      if (i >= BLOCK) { const int pr = min(max(t - 1, 0), T); ph = at32(gphi, pr); b = at32(gb, pr); B = at32(Bu, pr); }
      float f = LOG0F, fb = LOG0F;
      if (in_range(t)) {
        const float bt = (float)(B - Bref);
        f = canon0(ph + bt); fb = canon0(b + bt);
      }
      const int k = t - (T - R + 1);
      if (e2w && k >= 0 && k < R) { s_e2f[k] = f; s_e2f[MAX_EOS_RUN + k] = fb; f = LOG0F; fb = LOG0F; }
      s_F[i] = f; s_Fb[i] = fb;
    }
    if (e2 && tid < R) e2_Et = canon0(e2_p + (float)(e2_B - Bref));
    if (tid == 0) {
      // eos: phi_T(g) = off' + B_T + stored  (raw scores: the joint score still lacks the row's log-sum-exp)
      const float ce = eos_p;
      const bool v = ce > LOG0_CLASS;
      const double ctc = v ? offr + BT + (double)ce : LOG0D;
      s_eos[0] = ctc;
      s_eos[1] = v ? lam * ctc + (1.0 - lam) * (double)x_eos + jbase : LOG0D;
      s_eos[2] = jbase; s_eos[3] = offr; s_eos[4] = 1.0 - lam;   // (held in registers through the sums they were spilled)
    }
  };
  TRACE_MARK(2);

  // ---------------- 1. candidates -----------------------------------------------------------
  // direct: the K ids lie in s_wid (a copy per wave) and s_av, else in s_cid / s_av (or, K > BLOCK, in global memory)
  bool direct = false;
  if (p.mode & SC_RESTRICTED) {
    bool ok = false;
    if (in_regs) {
      // The granules' maxima, the lane's.  Blank and eos are among them: the pivot is one that two lanes more reach, and the
      // list leaves them out (taken out here, they cost ten branches: a short launch, one utterance, 8.0 -> 7.6 us).
      float m4[NV4], fmx = row.ex;
#pragma unroll
      for (int k = 0; k < NV4; ++k) {
        m4[k] = fmaxf(fmaxf(row.v[k].x, row.v[k].y), fmaxf(row.v[k].z, row.v[k].w));
        if (tid + k * BLOCK >= ng) m4[k] = __builtin_nanf("");   // (past the row's end: never a hit, whatever the pivot)
        fmx = fmaxf(fmx, m4[k]);
      }
      TRACE_MARK(6);
      s_mx[tid] = fmx;
      if (hist) pivot_count((uint32_t*)s_wid, fmx);
      lds_barrier();
      // at least K values of candidates are >= L (-inf if there are not K + 2 lanes with finite maxima)
      float M = 0.0f;
      const float L = hist ? find_pivot_hist<BLOCK>((const uint32_t*)s_wid, s_mx, K + 2) : find_pivot<BLOCK>(s_mx, min(K + 2, BLOCK), M);   // (256 candidates: of nearly all lanes)
      TRACE_MARK(7);
      const int nh = collect_hits<BLOCK, NV4>(row, m4, L, p.blank_id, p.eos_id, s_gran + w * ShortList::GCAP,
                                              s_gid + w * ShortList::GCAP, s_ent + w * ShortList::WCAP);
      if ((tid & 63) == 0) s_cnt[w] = nh;
      TRACE_MARK(14);
      if (logits) {
        M = fmaxf(M, -3.0e38f);
        float sum = __expf(row.ex - M);
        int t = tid;
        LOADED(t);                                         // (or the lanes within the row are kept from above, in scalar registers)
#pragma unroll
        for (int k = 0; k < NV4; ++k) {
          const float s4 = (__expf(row.v[k].x - M) + __expf(row.v[k].y - M)) + (__expf(row.v[k].z - M) + __expf(row.v[k].w - M));
          sum += t + k * BLOCK < ng ? s4 : 0.0f;
        }
        sum = row16_sum(sum);
        const double ws = ((double)lane_f(sum, 0) + (double)lane_f(sum, 16)) +
                          ((double)lane_f(sum, 32) + (double)lane_f(sum, 48));
        if ((tid & 63) == 0) ((double*)(s_red + BLOCK / 64))[w] = ws;
      }
      // (behind the barrier, in the place of the granules, which all waves are done with: before it, with a place of their own for the
      // granules, 1500 frames took 25.5 KB and six work-groups a compute unit, now 22.4 KB and seven; us a decode: 256 utterances, beam 20
      // 13479 -> 13120, of 900 to 1300 frames, beam 10 8622 -> 8533, 128 of 2300 ids 1971 -> 1952, 37 with raw scores 1619 -> 1582, others
      // the same to half a per cent)
      lds_barrier();
      stage_state();
      TRACE_MARK(15);
      ShortList sl;
      sl.n0 = uni(s_cnt[0]); sl.n1 = uni(s_cnt[1]); sl.n2 = uni(s_cnt[2]); sl.n3 = uni(s_cnt[3]);
      sl.n = (sl.n0 + sl.n1) + (sl.n2 + sl.n3);
      // (NaNs in the row: fewer than K values may have been found)
      ok = sl.n >= K && max(max(sl.n0, sl.n1), max(sl.n2, sl.n3)) <= ShortList::WCAP;
      if (logits && (BIGK || w == 2)) {                    // (by one wave, beside the columns' loads)
        const double* sd = (const double*)(s_red + BLOCK / 64);
        row_lse = (float)((double)M + log((sd[0] + sd[1]) + (sd[2] + sd[3])));
        if (tid == 128) s_lse = row_lse;
      }
      if (!BIGK && ok && sl.n <= 64) {
        direct = take_k(w, s_ent, sl, K, (uint32_t*)s_mx, s_wid + 64 * w, s_av);
        wave_lds_fence();
      }
      if (!BIGK && ok && sl.n > 64 && sl.n <= 128) {
        direct = take_k_of_128(w, s_ent, sl, K, (uint32_t*)s_mx, s_wid + 64 * w, s_av);
        wave_lds_fence();
      }
      if (ok && !direct) {
        // exact rank, four lanes per entry; the rank is the candidate's place
        for (int e0 = 0; e0 < sl.n; e0 += BLOCK / 4) {
          const int en = e0 + (tid >> 2);
          const unsigned long long me = en < sl.n ? s_ent[sl.at(en)] : ~0ull;
          const int rank = list_rank_quad(s_ent, sl, me, tid & 3);
          if ((tid & 3) == 0 && en < sl.n && rank < K) {
            const int mid = (int)~(uint32_t)me;
            // (small K: the ids stay in LDS; the global copy is written with the scores at the end, so that
            // no store is pending when the candidates' columns are fetched)
            if (smallk) { s_cid[rank] = mid; s_av[rank] = key_to_att((uint32_t)(me >> 32)); }
            else g_cid[rank] = mid;
          }
        }
      }
    }
    if (!in_regs) stage_state();
    if (!ok) select_radix<BLOCK>(arow, V, K, p.blank_id, p.eos_id, s_work, s_scan, s_sel, smallk, s_cid, s_av, g_cid);
  } else {
    stage_state();
    const int lo_ex = min(p.blank_id, p.eos_id), hi_ex = max(p.blank_id, p.eos_id);
    for (int i = tid; i < K; i += BLOCK) {
      const int id = full_v_id(i, lo_ex, hi_ex);
      if (smallk) { s_cid[i] = id; s_av[i] = arow[id]; }
      else g_cid[i] = id;
    }
  }
  // candidates and f terms visible to the whole block (large K: the ids are read back from global memory)
  if (!direct) { if (smallk) lds_barrier(); else __syncthreads(); }
  auto cand_id = [&](int c) -> int {
    if (direct) return s_wid[64 * w + c];
    return smallk ? s_cid[c] : checked(p, g_cid[c], 0, V - 1, ERR_CAND_ID);
  };
  TRACE_MARK(3);

  // ---------------- 3. prefix scores ----------------------------------------------------
  constexpr int NSG = BLOCK / LPC;
  const int sg = tid / LPC, q = tid % LPC;
  const float* xu = p.xT + (size_t)u * V * p.Tp;
  // float4 i of a candidate's column from frame t0 on.  At most 65536 ids of 6176 frames: 32 bits hold the offset
  auto column = [&](int id, int i) {
    if (BIGK) return ((const float4*)(xu + (size_t)id * p.Tp + t0))[i];
    const uint32_t row = (uint32_t)__umul24((unsigned)id, (unsigned)(4 * p.Tp));
    return *(const float4*)((const char*)xu + (row + 4u * (uint32_t)t0 + 16u * (uint32_t)i));
  };
  float *g_inc = nullptr, *g_catt = nullptr, *g_pre = nullptr;
  double *g_ctc = nullptr, *g_joint = nullptr;
  if (BIGK) {
    const ScoreLatePtr a = score_late(late_args);
    const size_t g = (size_t)grp * K;
    g_inc = a->cand_inc + g; g_catt = a->cand_att + g; g_ctc = a->cand_ctc + g; g_joint = a->cand_joint + g; g_pre = a->cand_pre + g;
  }
  // more frames than one round of loads: where that is usual, the candidates' next rounds together
  constexpr bool TOGETHER = BIGK ? IT == 4 : NEAR && IT == 2;
  bool low = false;                                       // a sum that the frames left out may count for
  for (int cb = 0; cb < K; cb += NSG * CB) {              // (uniform: every chain takes part in every round)
    const int c0 = cb + sg;
    float4 x[CB][IT];
    int ids[CB];
    ChainSum sum[CB];
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int c = c0 + b * NSG;
      ids[b] = (c < K) ? cand_id(c) : -1;
#pragma unroll
      for (int it = 0; it < IT; ++it)                        // unconditional (clamped) loads: all in flight together
        x[b][it] = column(max(ids[b], 0), min(j0 + q + it * LPC, max(n4 - 1, 0)));
    }
    // the next frames of all candidates of the round
    auto next_round = [&](int j) {
#pragma unroll
      for (int b = 0; b < CB; ++b) {
#pragma unroll
        for (int it = 0; it < IT; ++it) x[b][it] = column(max(ids[b], 0), min(j + q + it * LPC, n4 - 1));
      }
    };
    if (TOGETHER && !e2g) {
      auto f_terms = [&](int b, int j, float4 (&f)[IT]) {
        const float4* f4 = (const float4*)(s_F + ((ids[b] == last) ? p.wp_max : 0)) + j;
#pragma unroll
        for (int it = 0; it < IT; ++it) f[it] = f4[q + it * LPC];
      };
#pragma unroll
      for (int b = 0; b < CB; ++b) {
        float4 f[IT];
        f_terms(b, j0, f);
        sum[b] = chain_first<LPC, IT>(x[b], f);
      }
      for (int j = j0 + LPC * IT; j < j1; j += LPC * IT) {
        next_round(j);
#pragma unroll
        for (int b = 0; b < CB; ++b) {
          float4 f[IT];
          f_terms(b, j, f);
          chain_more<LPC, IT>(sum[b], x[b], f);
        }
      }
    }
    Lse upto[CB], last_r[CB];
    if (e2g) {
      // the sums in two parts: frames up to T - R (needed on their own below) and the last R frames
      const int tc = T - R;
#pragma unroll
      for (int b = 0; b < CB; ++b) { upto[b].m = last_r[b].m = LOG0F; upto[b].s = last_r[b].s = 0.0f; }
      for (int j = 0; j < n4; j += LPC * IT) {
        if (j > 0) next_round(j);
#pragma unroll
        for (int b = 0; b < CB; ++b) {
          const float4* f4 = (const float4*)(s_F + ((ids[b] == last) ? p.wp_max : 0));
#pragma unroll
          for (int it = 0; it < IT; ++it) {
            const int i = j + q + it * LPC, tb = t0 + 4 * i;
            const float4 f = f4[i];
            float4 fv;
            fv.x = tb <= tc ? f.x : LOG0F; fv.y = tb + 1 <= tc ? f.y : LOG0F;
            fv.z = tb + 2 <= tc ? f.z : LOG0F; fv.w = tb + 3 <= tc ? f.w : LOG0F;
            upto[b] = lse_join(upto[b], lse_block(x[b][it], fv));
            fv.x = tb > tc ? f.x : LOG0F; fv.y = tb + 1 > tc ? f.y : LOG0F;
            fv.z = tb + 2 > tc ? f.z : LOG0F; fv.w = tb + 3 > tc ? f.w : LOG0F;
            last_r[b] = lse_join(last_r[b], lse_block(x[b][it], fv));
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int c = c0 + b * NSG;
      if (ids[b] < 0) continue;                            // uniform over the LPC lanes of a chain
      const int id = ids[b];
      const float4* f4 = (const float4*)(s_F + ((id == last) ? p.wp_max : 0));   // Fb follows F
      float inc = LOG0F, pre = LOG0F;
      if (!e2g) {
        if (!TOGETHER) {
          float4 f[IT];
#pragma unroll
          for (int it = 0; it < IT; ++it) f[it] = f4[j0 + q + it * LPC];
          sum[b] = chain_first<LPC, IT>(x[b], f);
          for (int i0 = j0 + LPC * IT; i0 < j1; i0 += LPC * IT) { // (windows beyond one round of loads)
            float4 y[IT];
#pragma unroll
            for (int it = 0; it < IT; ++it) { y[it] = column(id, min(i0 + q + it * LPC, n4 - 1)); f[it] = f4[i0 + q + it * LPC]; }
            chain_more<LPC, IT>(sum[b], y, f);
          }
        }
        inc = chain_finish<LPC>(sum[b]);
        if (NEAR) low |= inc <= sum_low;
      } else {
        pre = lse_finish<LPC>(upto[b]);
        inc = lse_finish<LPC>(lse_join(upto[b], last_r[b]));
      }
      if (q == 0 && wave_rank) {
        // (joint scores and sort keys: one lane per candidate at the end, not one pass per chain here)
        s_inc[c] = inc;                                    // (eos-run rule armed: the sum up to frame T - R so far)
      } else if (q == 0) {
        const float av = (smallk ? s_av[c] : arow[id]) - row_lse;
        const bool valid = inc > LOG0_CLASS;
        const double ctc = valid ? offr + (double)inc : LOG0D;
        const double J = valid ? lam * ctc + (1.0 - lam) * (double)av + jbase : LOG0D;
        // small K: scores stay in LDS for the ranking below; per-candidate arrays in global memory
        // (read back by ctcbs_peek only) are written from there at the very end, so that no store
        // is pending while columns are still being fetched
        if (smallk) {
          s_J[c] = J; s_inc[c] = inc; s_av[c] = av;
          s_key[c] = joint_key(J, 0ull, 0, valid && J == J);
          if (e2) s_pre[c] = pre;
        } else {
          g_inc[c] = inc; g_catt[c] = av; g_ctc[c] = ctc; g_joint[c] = J;
          if (e2) g_pre[c] = pre;
        }
      }
    }
  }
  if (NEAR && __ballot(low) != 0ull) {
    // Such sums again, over the frames whose f term lies within the margin of the least of them, unless those are among the frames summed.
    // Sharp posteriors have many such sums (a candidate 30 nats down at the near frames), and f falls as sharply, so that it takes few
    // frames more (posteriors twice and three times as sharp, against the whole window for each such sum: 16 whole utterances 2155 -> 1518 us
    // a decode, of 1500 frames 3730 -> 1790, 128 3850 -> 2700, margins of 70 3785 -> 3205; all frames at once 1705, 2230, 3255, 3425).
    wave_lds_fence();
    float least = 0.0f;                                    // (sum_low lies below -16)
    for (int c = sg; c < K; c += NSG) { const float v = s_inc[c]; if (v <= sum_low) least = fminf(least, v); }
    least = fminf(fminf(lane_f(least, 0), lane_f(least, 16)), fminf(lane_f(least, 32), lane_f(least, 48)));
    const float f_low = fmaxf(least - NEAR_MARGIN - 9.0f, LOG0_CLASS);   // (at most e^9 frames)
    int ja = j0, jb = j1;
#pragma unroll 1
    for (int i0 = 0; i0 < n4; i0 += 64) {
      const float4 f = ((const float4*)s_F)[min(i0 + (tid & 63), n4 - 1)];
      const unsigned long long m = __ballot(fmaxf(fmaxf(f.x, f.y), fmaxf(f.z, f.w)) > f_low);
      if (m != 0ull) { ja = min(ja, i0 + __ffsll((long long)m) - 1); jb = max(jb, min(i0 + 64 - __clzll((long long)m), n4)); }
    }
    if (ja < j0 || jb > j0 + (j1 - j0 + LPC * IT - 1) / (LPC * IT) * (LPC * IT)) {
#pragma unroll 1
      for (int c = sg; c < K; c += NSG) {
        if (!(s_inc[c] <= sum_low)) continue;              // uniform over the LPC lanes of a chain
        const int id = cand_id(c);
        const float4* f4 = (const float4*)(s_F + ((id == last) ? p.wp_max : 0));
        ChainSum a;
        a.M = LOG0F; a.s = 0.0f;
#pragma unroll 1
        for (int j = ja; j < jb; j += LPC * IT) {
          float4 y[IT], f[IT];
#pragma unroll
          for (int it = 0; it < IT; ++it) {
            const int i = min(j + q + it * LPC, n4 - 1);
            y[it] = column(id, i);
            f[it] = j + q + it * LPC < n4 ? f4[i] : make_float4(LOG0F, LOG0F, LOG0F, LOG0F);
          }
          chain_more<LPC, IT>(a, y, f);
        }
        const float inc = chain_finish<LPC>(a);
        if (q == 0) s_inc[c] = inc;
      }
    }
  }

  TRACE_MARK(4);
  // ---------------- 4. eos-run rule, group list, outputs -----------------------------------
  // (few candidates: the first wave runs this test alone, further down, without a barrier)
  int fire = 0;
  if (e2g) {
    // Frame T is one of the R frames and there X_T is simply the best full prefix score of the
    // extensions, which is already known: most eligible hypotheses fail this test and skip the rest.
    if (smallk) lds_barrier(); else __syncthreads();       // s_inc / g_inc of all candidates written
    float xt = -3.0e38f;
    for (int c = tid; c < K; c += BLOCK) xt = fmaxf(xt, canon0(smallk ? s_inc[c] : g_inc[c]));
    xt = row16_max(xt);
    xt = fmaxf(fmaxf(lane_f(xt, 0), lane_f(xt, 16)), fmaxf(lane_f(xt, 32), lane_f(xt, 48)));
    if ((tid & 63) == 0) s_e2w[tid >> 6] = xt;
    if (tid == 0) s_e2w[BLOCK / 64] = (rs <= T && re >= T) ? canon0(eos_p + (float)BT) : LOG0F;
    lds_barrier();
    float XT = s_e2w[0];
#pragma unroll
    for (int w2 = 1; w2 < BLOCK / 64; ++w2) XT = fmaxf(XT, s_e2w[w2]);
    const float ET = s_e2w[BLOCK / 64];
    const bool maybe = (ET > LOG0_CLASS) && (XT < LOG0_CLASS || ET > XT);
    lds_barrier();                                         // s_e2w is reused below
    if (maybe) {
    // the last R frames, sixteen at a time: every lane carries the
    // running prefix score of its candidates from chunk to chunk through the pre array (each entry
    // is only ever touched by one lane from here on) and keeps, per frame, the best score it has seen
    constexpr int E2C = 16;
    for (int k0 = 0; k0 < R; k0 += E2C) {
      float xmax[E2C];
#pragma unroll
      for (int k = 0; k < E2C; ++k) xmax[k] = -3.0e38f;
      for (int c = tid; c < K; c += BLOCK) {
        const int id = smallk ? s_cid[c] : g_cid[c];
        const float* colf = xu + (size_t)id * p.Tp;
        const float* ff = s_F + ((id == last) ? p.wp_max : 0);
        float xv[E2C];
#pragma unroll
        for (int k = 0; k < E2C; ++k) xv[k] = colf[min(T - R + 1 + k0 + k, T)];   // all loads in flight
        float acc = smallk ? s_pre[c] : g_pre[c];
#pragma unroll
        for (int k = 0; k < E2C; ++k) {
          if (k0 + k < R) {
            acc = lae(acc, ff[T - R + 1 + k0 + k - t0] + xv[k]);
            xmax[k] = fmaxf(xmax[k], canon0(acc));
          }
        }
        if (smallk) s_pre[c] = acc; else g_pre[c] = acc;
      }
#pragma unroll
      for (int k = 0; k < E2C; ++k) {                      // max over the wave, one slot per wave and frame
        if (k0 + k < R) {
          float v = row16_max(xmax[k]);
          v = fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
          if ((tid & 63) == 0) s_e2w[(tid >> 6) * MAX_EOS_RUN + k0 + k] = v;
        }
      }
    }
    if (tid == 0) s_nvalid = 1;                            // reused as the "all frames passed" flag
    lds_barrier();
    if (tid < R) {
      const float Et = e2_Et;
      float X = s_e2w[tid];
#pragma unroll
      for (int w2 = 1; w2 < BLOCK / 64; ++w2) X = fmaxf(X, s_e2w[w2 * MAX_EOS_RUN + tid]);
      // E_t > X_t with log0 on the left never true, log0 on the right always true
      const bool gt = (Et > LOG0_CLASS) && (X < LOG0_CLASS || Et > X);
      if (!gt) s_nvalid = 0;                               // every writer stores the same value
    }
    lds_barrier();
    fire = s_nvalid;
    }                                                      // maybe
    lds_barrier();                                         // s_nvalid is reset below
  }
  auto group_outputs = [&](int n) {
    const double je = s_eos[1];
    score_late(late_args)->grp[grp] = GroupOut{n, fire, s, e, s_eos[0],
                          logits && je > (double)LOG0_CLASS ? je - s_eos[4] * (double)row_lse : je,
                          (long long)K * (long long)W, {0, 0, 0, 0, 0, 0}};
  };
  if (!smallk && tid == 0) group_outputs(0);               // (the list builder counts)

  if (smallk) {
    if (wave_rank) {
      // one lane of the first wave per entry from here on
      constexpr int E2W = 16;                              // eos-run rule: frames per round of loads
      float xv0[E2W];
      if (e2 && tid < 64) {                    // the candidate's posteriors of the last R frames: on
        const float* colf = xu + (size_t)cand_id(tid < K ? tid : 0) * p.Tp;   // their way while the other waves finish
#pragma unroll
        for (int k = 0; k < E2W; ++k) xv0[k] = colf[min(T - R + 1 + k, T)];
      }
      lds_barrier();                                       // prefix scores complete; the other waves are done
      // (small batches) or they broadcast a quarter of the entries each, turned as in take_k
      const bool share = early && !e2;
      if (!share && tid >= 64) return;
      const int te = ((tid & 63) + 16 * w) & 63;           // (the first wave: tid)
      const bool has = te < K;
      const int id = cand_id(has ? te : 0);
      if (logits) row_lse = s_lse;
      if (e2) {
        // eos-run rule by one wave.  The sums so far stop at frame T - R; walking through the last R frames
        // completes them and gives, on the way, X_t = best running prefix score of the extensions at frame
        // t, to be held against E_t (in lane t - (T-R+1) since the start of the kernel).
        auto wave_max = [](float v) {
          v = row16_max(v);
          return fmaxf(fmaxf(lane_f(v, 0), lane_f(v, 16)), fmaxf(lane_f(v, 32), lane_f(v, 48)));
        };
        const float* colf = xu + (size_t)id * p.Tp;
        const float* ff = s_e2f + ((id == last) ? MAX_EOS_RUN : 0);
        float acc = has ? s_inc[tid] : LOG0F;
        fire = 1;
        for (int k0 = 0; k0 < R; k0 += E2W) {
          float xv[E2W];
          if (k0 == 0) {
#pragma unroll
            for (int k = 0; k < E2W; ++k) xv[k] = xv0[k];
          } else {
#pragma unroll
            for (int k = 0; k < E2W; ++k) xv[k] = colf[min(T - R + 1 + k0 + k, T)];   // all loads in flight
          }
#pragma unroll
          for (int k = 0; k < E2W; ++k) {
            if (k0 + k < R) {                              // (uniform)
              acc = lae(acc, ff[k0 + k] + xv[k]);
              const float X = wave_max(has ? canon0(acc) : -3.0e38f);
              const float Et = k0 == 0 ? lane_f(e2_Et, k) : lane_f(e2_Et, k + E2W);
              // E_t > X_t with log0 on the left never true, log0 on the right always true
              if (!((Et > LOG0_CLASS) && (X < LOG0_CLASS || Et > X))) fire = 0;
            }
          }
        }
        if (has) s_inc[tid] = canon0(acc);                 // the whole window's sum
        wave_lds_fence();
      }
      // rank by (joint desc, token asc) on 64-bit keys; joint score (Eq. (1)) and sort key of entry `te`
      const float inc = has ? s_inc[te] : LOG0F;
      const float av = s_av[has ? te : 0] - row_lse;
      const bool valid = inc > LOG0_CLASS;
      const double ctc = valid ? s_eos[3] + (double)inc : LOG0D;
      const double J = valid ? lam * ctc + s_eos[4] * (double)av + s_eos[2] : LOG0D;
      // equal scores go by token id: the id in 16 bits (below 65536 here; scores equal to within 2^-36 relative count as
      // equal then), or, every id a candidate, the lane, which ascends with the id (2^-46)
      const bool by_lane = (p.mode & SC_RESTRICTED) == 0;
      const unsigned long long me = joint_key(J, by_lane ? 63ull : 0xFFFFull, by_lane ? 63 - te : 0xFFFF - (id & 0xFFFF),
                                              has && valid && J == J);
      int rank;                                            // (lanes past the last entry hold zeros)
      if (share) {
        ((uint8_t*)s_mx)[4 * te + w] = (uint8_t)lanes_above<16>(me, 16);
        lds_barrier();
        if (w != 0) return;
        rank = (int)((((const uint32_t*)s_mx)[tid] * 0x01010101u) >> 24);
      } else rank = lanes_above<16>(me, K);
      const int nv = __popcll(__ballot(me != 0ull));
      if (!fire && me != 0ull && rank < Wb) score_late(late_args)->grp_list[(size_t)grp * Wb + rank] = ListEntry{J, id, inc, av, 0};
      if (tid == 0) group_outputs(fire ? 0 : min(nv, Wb));
      if ((p.mode & SC_PAIRS) && has) ((double2*)score_late(late_args)->cand_joint)[(size_t)grp * K + tid] = double2{J, ctc};
      if ((p.mode & SC_KEEP) && has) {
        const ScoreLatePtr a = score_late(late_args);
        const size_t g = (size_t)grp * K + tid;
        a->cand_id[g] = id; a->cand_inc[g] = inc; a->cand_att[g] = av; a->cand_ctc[g] = ctc; a->cand_joint[g] = J;
      }
    } else {
      // rank by (joint desc, token asc), exact comparison: four lanes per candidate
      if (tid == 0) s_nvalid = 0;
      lds_barrier();                                       // scores complete
      if (!fire) {
        const int part = tid & 3;
        for (int e0 = 0; e0 < K; e0 += BLOCK / 4) {
          const int ee = e0 + (tid >> 2);
          const bool mv = ee < K && s_key[ee] != 0ull;
          const double me = mv ? s_J[ee] : LOG0D;
          const int mtok = ee < K ? s_cid[ee] : 0x7fffffff;
          int rank = 0;
          for (int c = part; c < K; c += 4) {
            const double o = s_key[c] != 0ull ? s_J[c] : LOG0D;
            rank += (o > me) || (o == me && s_cid[c] < mtok);
          }
          rank += dpp_i<0xB1, 0xf>(0, rank);               // quad_perm [1,0,3,2]
          rank += dpp_i<0x4E, 0xf>(0, rank);               // quad_perm [2,3,0,1]
          if (part == 0 && mv) {
            if (rank < Wb) score_late(late_args)->grp_list[(size_t)grp * Wb + rank] = ListEntry{me, s_cid[ee], s_inc[ee], s_av[ee], 0};
            atomicAdd(&s_nvalid, 1);
          }
        }
      }
      lds_barrier();
      if (tid == 0) group_outputs(fire ? 0 : min(s_nvalid, Wb));
      if (p.mode & SC_KEEP) {
        for (int c = tid; c < K; c += BLOCK) {
          const float inc = s_inc[c];
          g_cid[c] = s_cid[c]; g_inc[c] = inc; g_catt[c] = s_av[c];
          g_ctc[c] = inc > LOG0_CLASS ? offr + (double)inc : LOG0D;
          g_joint[c] = s_J[c];
        }
      }
    }
  }
  TRACE_MARK(5);
#ifdef CTCBS_TRACE
  const struct { unsigned long long* trace; } tr_to = {score_late(late_args)->trace};
  TRACE_FLUSH(tr_to, grp);
#endif
}

// Group list for candidate sets whose joint scores lie in global memory (K > block size; not the matrix form, see dense_top): one
// work-group per (utterance, beam slot).  Order: joint score descending (compared as the fp64 it is), then the candidate's
// place = token id ascending.  Every lane goes over its share of the scores as order-preserving 64-bit images; the largest
// upper halves of the lanes give a pivot that at least Wb of the scores reach (as for the candidates, see find_pivot), the
// few that do are packed into LDS with their places and ranked.  More than CAP of them (scores equal in the upper half, that
// is to 2^-20 relative): Wb rounds of a block-wide maximum.  (68 us at 4998 candidates, beam 20, with the rounds alone: a
// round costs 2 us.)
// Per launch at 300 candidates, beam 10, 64 utterances 6.3 us.
// EPT: scores per lane, held in registers; 0: as many as there are, read again (from L2) for each pass.
template <int N> struct Int { static constexpr int n = N; };
template <int EPT>
__global__ __launch_bounds__(256) void k_list_top(Params p, int cur) {
  constexpr int BLOCK = 256, NW = BLOCK / 64, CAP = 512;
  __shared__ unsigned long long s_k[2][NW];
  __shared__ int s_c[2][NW];
  __shared__ __align__(16) unsigned long long s_ent[CAP + 4];
  __shared__ __align__(16) int s_at[CAP + 4];
  __shared__ uint32_t s_thr[NW];
  __shared__ int s_n;
  const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6);
  const int grp = (int)(blockIdx.y * gridDim.x + blockIdx.x), u = blockIdx.y, K = p.K, Wb = p.Wb;
  // (what decides whether there is anything to do, and the slot, are asked for together)
  const uint8_t finished = FETCH(p.finished + u);
  const int live = FETCH(&p.rec[cur][grp].live), stopped = FETCH(&p.grp[grp].stopped);
  const double* J = p.cand_joint + (size_t)grp * K;
  const float* ginc = p.cand_inc + (size_t)grp * K;
  if (finished || !live) return;                            // the score kernel already wrote a count of 0
  if (stopped) { if (tid == 0) p.grp[grp].n = 0; return; }
  // f(k, key) over the lane's scores, N loads in flight: candidate me + k * BLOCK (me = tid), key its score's image (0: not
  // a competitor)
  auto read_scores = [&](auto n_loads, int me, auto&& f) {
    constexpr int N = decltype(n_loads)::n;
    auto some = [&](int k0) {
      double jv[N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        jv[k] = J[min(me + (k0 + k) * BLOCK, K - 1)];
      }
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const int c = me + (k0 + k) * BLOCK;
        f(k0 + k, c < K ? joint_image(jv[k]) : 0ull);
      }
    };
    if (EPT > 0 && N >= (EPT < 16 ? EPT : 16)) {
#pragma unroll
      for (int k0 = 0; k0 < EPT; k0 += N) some(k0);
    } else {
#pragma unroll 1
      for (int k0 = 0; k0 * BLOCK < K; k0 += N) some(k0);
    }
  };
  using Loads = Int<(EPT == 0 || EPT > 20) ? 16 : EPT>;
  unsigned long long key[EPT > 0 ? EPT : 1];
  uint32_t kmax = 0u;
  read_scores(Loads(), tid, [&](int k, unsigned long long kk) {
    if (EPT > 0) key[EPT > 0 ? k : 0] = kk;
    kmax = max(kmax, (uint32_t)(kk >> 32));
  });
  auto each = [&](auto&& f) {
    if (EPT > 0) {
#pragma unroll
      for (int k = 0; k < (EPT > 0 ? EPT : 1); ++k) f(k, key[k]);
    } else read_scores(Loads(), tid, f);
  };
  auto emit = [&](int c, int r) {
    c = min(c, K - 1);
    const size_t g = (size_t)grp * K + c;
    const int id = checked(p, p.cand_id[g], 0, p.V - 1, ERR_CAND_ID);
    p.grp_list[(size_t)grp * Wb + r] = ListEntry{J[c], id, ginc[c], p.cand_att[g], 0};
  };
  // pivot on the upper halves: every wave's share of Wb
  const int have = min(max(K - 64 * w, 0), 64), all = K < BLOCK ? K : BLOCK;
  const int r = (Wb * have + all - 1) / all;
  uint32_t thr = 0u;
#pragma unroll
  for (int bit = 31; bit >= 10; --bit) {
    const uint32_t t = thr | (1u << bit);
    if (__popcll(__ballot(kmax >= t)) >= r) thr = t;
  }
  if (lane == 0) s_thr[w] = r > 0 ? thr : 0xffffffffu;
  if (tid == 0) s_n = 0;
  lds_barrier();
  const uint32_t L = max(min(min(s_thr[0], s_thr[1]), min(s_thr[2], s_thr[3])), 1u);
  int me0 = tid;
  LOADED(me0);                                              // (or the places of all scores stay in registers from the loads on)
  each([&](int k, unsigned long long kk) {
    if ((uint32_t)(kk >> 32) >= L) {
      const int pos = atomicAdd(&s_n, 1);
      if (pos < CAP) { s_ent[pos] = kk; s_at[pos] = me0 + k * BLOCK; }
    }
  });
  lds_barrier();
  const int n = uni(s_n);
  if (n <= CAP) {
    if (tid < 4) { s_ent[n + tid] = 0ull; s_at[n + tid] = 0; }
    lds_barrier();
    const ulonglong2* e2 = (const ulonglong2*)s_ent;
    const int q = (n + 3) >> 2;
    for (int e0 = 0; e0 < n; e0 += BLOCK / 4) {
      const int e = e0 + (tid >> 2);
      const unsigned long long me = e < n ? s_ent[e] : ~0ull;
      const int at = e < n ? s_at[e] : 0;
      int rank = 0, equal = 0;                              // (its own entry among the equal ones)
      for (int i = tid & 3; i < q; i += 4) {
        const ulonglong2 a = e2[2 * i], b = e2[2 * i + 1];
        rank += ((int)(a.x > me) + (int)(a.y > me)) + ((int)(b.x > me) + (int)(b.y > me));
        equal += ((int)(a.x == me) + (int)(a.y == me)) + ((int)(b.x == me) + (int)(b.y == me));
      }
      rank += dpp_i<0xB1, 0xf>(0, rank);                   // quad_perm [1,0,3,2]
      rank += dpp_i<0x4E, 0xf>(0, rank);                   // quad_perm [2,3,0,1]
      equal += dpp_i<0xB1, 0xf>(0, equal);
      equal += dpp_i<0x4E, 0xf>(0, equal);
      if (__ballot(equal > 1) != 0ull)                      // (uniform, rare: equal scores go by place)
        for (int i = 0; i < n; ++i) rank += (int)(s_ent[i] == me) & (int)(s_at[i] < at);
      if ((tid & 3) == 0 && e < n && rank < Wb) emit(at, rank);
    }
    if (tid == 0) p.grp[grp].n = min(n, Wb);
    return;
  }
  // rounds: the best behind the one taken last
  LOADED(me0);
  unsigned long long last = ~0ull;
  int last_c = 0, found = 0;
  for (int rd = 0; rd < Wb; ++rd) {
    // (a lane's places ascend: the first of equals stays.  Those before the last one taken are taken too, of its equals
    // those up to its place.  The scores are read again in every form: struck out in registers they cost the usual way
    // 30 registers more)
    unsigned long long best = 0ull;
    int bk = 0;
    const int k_taken = (last_c - me0) >> 8;                // (rounded down: BLOCK places apart)
    read_scores(Int<8>(), me0, [&](int k, unsigned long long kk) {
      const bool left = kk < last || (kk == last && k > k_taken);
      if (left && kk > best) { best = kk; bk = k; }
    });
    int bc = best != 0ull ? me0 + bk * BLOCK : 0x7fffffff;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const unsigned long long ob = __shfl_xor(best, o);
      const int oc = __shfl_xor(bc, o);
      if (ob > best || (ob == best && oc < bc)) { best = ob; bc = oc; }
    }
    if (lane == 0) { s_k[rd & 1][w] = best; s_c[rd & 1][w] = bc; }
    lds_barrier();                                          // (two buffers: one barrier per round is enough)
    best = s_k[rd & 1][0]; bc = s_c[rd & 1][0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
      const unsigned long long ob = s_k[rd & 1][i];
      const int oc = s_c[rd & 1][i];
      if (ob > best || (ob == best && oc < bc)) { best = ob; bc = oc; }
    }
    if (best == 0ull) break;                                // uniform: no finite candidate left
    if (tid == 0) emit(bc, rd);
    last = best; last_c = bc;
    ++found;
  }
  if (tid == 0) p.grp[grp].n = found;
}
