// Host side of the ctcbs C ABI (see include/ctcbs.h): argument checks, device memory,
// kernel launches.  Every step of the decoding path runs in the kernels of k_*.h.
#include "../../include/ctcbs.h"

#include <hip/hip_runtime.h>
#include <math.h>
#include <chrono>
#include <map>
#include <mutex>
#include <new>
#include <stdlib.h>
#include <string.h>
#include <thread>
#include <vector>

#include "common.h"
#include "k_finalize.h"
#include "k_ingest.h"
#include "k_score.h"
#include "k_dense.h"
#include "k_select.h"

static thread_local int g_last_hip = 0;

#ifndef CTCBS_EARLY_GROUPS         // (the CPU build of a test sets 0)
#define CTCBS_EARLY_GROUPS 256    // groups up to which the score kernel fetches rows before it knows of any utterance (k_score: flags)
#endif

#define STATIC_LDS 2560            // bytes: no form of the score kernel declares more LDS of its own

#ifndef CTCBS_SPLIT_GROUPS         // (the CPU build of the tests sets 0: small batches through the other kernel)
#define CTCBS_SPLIT_GROUPS 2048   // (utterance, beam slot) groups up to which the split select kernel runs, see step_impl
#endif

#define HIPCHK(expr)                                   \
  do {                                                 \
    hipError_t _e = (expr);                            \
    if (_e != hipSuccess) { g_last_hip = (int)_e; return CTCBS_EHIP; } \
  } while (0)

struct ctcbs {
  ctcbs_config_t cfg;
  Params p;
  Params p_step;       // the parameter block of the last step enqueued
  int32_t off_f, off_small, wp_max;   // the score kernel's LDS layout
  hipStream_t stream;
  int device;          // the device the handle lives on (current at creation)
  std::vector<void*> allocs;
  std::vector<int32_t> lens, lmax;
  int32_t step;        // steps enqueued
  int32_t cur;         // buffer holding the current beam
  int32_t l_cap;       // largest step cap over the batch
  int32_t l_cap_alloc; // step cap of an utterance of t_max frames: what the buffers are sized for
  int32_t known_finished;
  size_t score_smem_bytes;
  int score_block, select_block;
  int select_lps;              // select kernel: lanes per new hypothesis
  bool select_wide;            // windows beyond 128 frames are common
  int score_form;              // score kernel: windows up to 128 frames; 192 frames a round; wider ones, 33 to 48 candidates (see create_impl)
  bool score_bigk;
  bool want_near;              // the score kernel sums near frames first: the select kernels look for them
  int score_nv4;               // granules of an attention row per lane
  bool dense;                  // every id a candidate: the kernels of k_dense.h
  // Pinned, device-mapped host memory, one allocation: the progress word that the score kernel refreshes every
  // step (upper half: the step that has begun, lower half: utterances finished before it), the batch set-up that
  // the ingest kernels read (lengths, step caps, first batch-wide window), and the results that k_finalize writes.
  // Kernels access it directly: a transfer between pageable memory and the device costs 20-30 us here, and a
  // decode needed three on the way in and six on the way out.
  void* h_pin;
  unsigned long long* h_flag;
  int32_t* h_setup;
  const int32_t* d_setup;
  Results h_res, d_res;        // host and device addresses of the result arrays
  int32_t res_cap;
  // optional per-kernel timing
  bool profiling;
  std::vector<hipEvent_t> events;   // 3 per recorded step: before score, after score, after select
  size_t ev_used;
};

template <typename T>
static int dev_alloc(ctcbs* h, T** out, size_t n) {
  void* ptr = nullptr;
  size_t bytes = n * sizeof(T);
  if (bytes == 0) bytes = sizeof(T);
  hipError_t e = hipMalloc(&ptr, bytes);
  if (e != hipSuccess) { g_last_hip = (int)e; (void)hipGetLastError(); return CTCBS_ENOMEM; }
  h->allocs.push_back(ptr);
  *out = (T*)ptr;
  return CTCBS_OK;
}

static void free_all(ctcbs* h) {
  for (void* q : h->allocs) (void)hipFree(q);
  h->allocs.clear();
  if (h->h_pin) { (void)hipHostFree(h->h_pin); h->h_pin = nullptr; }
}

static int step_cap(const ctcbs_config_t* c, int T) {
  int l = T;
  if (c->max_len_ratio > 0.0f) { int r = (int)floor((double)c->max_len_ratio * (double)T); if (r < l) l = r; }
  if (c->max_len_abs > 0 && c->max_len_abs < l) l = c->max_len_abs;
  if (l < 1) l = 1;
  return l;
}

extern "C" const char* ctcbs_strerror(int code) {
  switch (code) {
    case CTCBS_OK: return "ok";
    case CTCBS_DONE: return "all utterances finished";
    case CTCBS_EINVAL: return "invalid argument or unsupported size";
    case CTCBS_ENOMEM: return "out of memory";
    case CTCBS_EHIP: return "HIP runtime error";
    case CTCBS_ESTATE: return "call not valid in this state";
    case CTCBS_ECAP: return "output capacity too small";
    default: return "unknown ctcbs error code";
  }
}

extern "C" int ctcbs_last_hip_error(void) { return g_last_hip; }

static int validate(const ctcbs_config_t* c) {
  if (c->n_utt < 1 || c->t_max < 1 || c->t_max > 6140 || c->vocab < 3) return CTCBS_EINVAL;
  if (c->beam < 1 || c->beam > MAX_BEAM) return CTCBS_EINVAL;
  if (c->blank_id < 0 || c->blank_id >= c->vocab || c->eos_id < 0 || c->eos_id >= c->vocab ||
      c->blank_id == c->eos_id) return CTCBS_EINVAL;
  if (c->cand_k < 0) return CTCBS_EINVAL;
  bool restricted = c->cand_k > 0 && c->cand_k < c->vocab - 2;
  if (!(c->ctc_weight >= 0.0f && c->ctc_weight <= 1.0f)) return CTCBS_EINVAL;
  if (c->length_bonus != c->length_bonus || c->max_len_ratio != c->max_len_ratio || c->max_len_ratio < 0.0f)
    return CTCBS_EINVAL;
  if (c->max_len_abs < 0) return CTCBS_EINVAL;
  if (c->end_flags & ~7) return CTCBS_EINVAL;
  if ((c->end_flags & CTCBS_END_BASELINE) && (c->end_m < 1 || c->end_m > MAX_END_M)) return CTCBS_EINVAL;
  if ((c->end_flags & CTCBS_END_TAU_COUNT) && c->end_c < 0) return CTCBS_EINVAL;
  if ((c->end_flags & CTCBS_END_EOS_RUN) && (c->eos_run < 1 || c->eos_run > MAX_EOS_RUN)) return CTCBS_EINVAL;
  if (c->poll_every < 0) return CTCBS_EINVAL;
  if (c->att_is_logits != 0 && c->att_is_logits != 1) return CTCBS_EINVAL;
  if (c->win_union != 0 && c->win_union != 1) return CTCBS_EINVAL;
  if (c->keep_candidates != 0 && c->keep_candidates != 1) return CTCBS_EINVAL;
  if ((long long)c->n_utt * c->beam > (1ll << 24)) return CTCBS_EINVAL;
  return CTCBS_OK;
}

// Per-batch part of the initialisation: lengths, step caps, transposed posteriors, empty beams.
static int ingest(ctcbs* h, const float* d_ctc_logp, const int32_t* h_lens) {
  const ctcbs_config_t& c = h->cfg;
  Params& p = h->p;
  const int U = c.n_utt;
  std::vector<int32_t> lens(h_lens, h_lens + U), lmax(U);
  int l_cap = 1, n_empty = 0;
  for (int u = 0; u < U; ++u) {
    if (lens[u] < 0 || lens[u] > c.t_max) return CTCBS_EINVAL;
    if (lens[u] == 0) { lmax[u] = 1; ++n_empty; continue; }   // an unused slot of the batch
    lmax[u] = step_cap(&c, lens[u]);
    if (lmax[u] > l_cap) l_cap = lmax[u];
  }
  hipStream_t st = h->stream;
  // (nothing still reads the set-up words: the previous ingest ended with a synchronisation)
  h->lens.swap(lens); h->lmax.swap(lmax); h->l_cap = l_cap;
  int e_max = 0;                                 // step 1: every hypothesis is empty, tau = tau~ = 0
  for (int u = 0; u < U; ++u) {
    const int e = c.win_m2 < h->lens[u] ? c.win_m2 : h->lens[u];
    if (e > e_max) e_max = e;
    h->h_setup[4 + u] = h->lens[u];
    h->h_setup[4 + U + u] = h->lmax[u];
  }
  h->h_setup[0] = 0x7fffffff; h->h_setup[1] = -1; h->h_setup[2] = 0; h->h_setup[3] = e_max;
  hipLaunchKernelGGL(k_setup, dim3((U + 255) / 256), dim3(256), 0, st, p, h->d_setup, n_empty);
  HIPCHK(hipGetLastError());
  {
    const int nvt = (p.V + INGEST_TOK - 1) / INGEST_TOK, ntt = (c.t_max + 5 + 31) / 32;   // stored indices 0 .. t_max + 4
    const int n_tiles = nvt * ntt, per_xcd = (n_tiles + 7) / 8;
    const dim3 tg(8 + 8 * per_xcd, U);           // (the first eight columns: the empty-prefix state, see k_ingest)
    if (p.V % 4 == 0 && ((uintptr_t)d_ctc_logp & 15) == 0)
      hipLaunchKernelGGL(k_ingest<true>, tg, dim3(256), 0, st, p, d_ctc_logp, nvt, n_tiles, per_xcd);
    else
      hipLaunchKernelGGL(k_ingest<false>, tg, dim3(256), 0, st, p, d_ctc_logp, nvt, n_tiles, per_xcd);
  }
  HIPCHK(hipGetLastError());
  h->step = 0; h->cur = 0; h->known_finished = n_empty;
  h->profiling = false; h->ev_used = 0;
  HIPCHK(hipStreamSynchronize(st));
  *h->h_flag = (unsigned)n_empty;                // (after the wait: steps of the batch before may have been under way)
  return CTCBS_OK;
}

static int create_impl(ctcbs* h, const float* d_ctc_logp, const int32_t* h_lens) {
  const ctcbs_config_t& c = h->cfg;
  Params& p = h->p;
  memset(&p, 0, sizeof p);
  const int U = c.n_utt, V = c.vocab, Wb = c.beam;
  const bool restricted = c.cand_k > 0 && c.cand_k < V - 2;
  const int K = restricted ? c.cand_k : V - 2;
  p.U = U; p.V = V; p.Wb = Wb; p.K = K;
  p.Tp = ((c.t_max + 5 + 31) / 32) * 32;        // frames 0..t_max plus slack for aligned float4 reads; rows of whole 128-byte lines
  p.t_max = c.t_max; p.blank_id = c.blank_id; p.eos_id = c.eos_id; p.restricted = restricted ? 1 : 0;
  p.win_m1 = c.win_m1; p.win_m2 = c.win_m2; p.end_flags = c.end_flags;
  p.end_m = (c.end_m >= 1 && c.end_m <= MAX_END_M) ? c.end_m : 1;
  p.end_c = c.end_c; p.eos_run = c.eos_run; p.end_d = c.end_d;
  p.lambda = (double)c.ctc_weight; p.beta = (double)c.length_bonus;
  p.att_logits = c.att_is_logits ? 1 : 0;
  p.win_union = c.win_union ? 1 : 0;
  p.union_utt = c.win_union && U * Wb <= CTCBS_SPLIT_GROUPS ? 1 : 0;
  // large candidate sets go through the per-candidate arrays in global memory whatever the caller asked for
  p.keep_cand = (c.keep_candidates || K > 256 || (!restricted && K > 64)) ? KEEP_ARRAYS : (!restricted ? KEEP_PAIRS : KEEP_NONE);
  // every id a candidate (not: few ids, the eos-run rule, raw decoder scores, the batch-wide window): the kernels of
  // k_dense.h; up to 64 ids k_score ranks the list itself.  They leave
  // increments and attention values in memory; the rest follows from those and is written only if asked to (ctcbs_peek)
  h->dense = !restricted && K > 64 && !(c.end_flags & CTCBS_END_EOS_RUN) && !c.att_is_logits && !c.win_union;
  if (h->dense) p.keep_cand = c.keep_candidates ? KEEP_ARRAYS : KEEP_NONE;

  // capacity for any batch of lengths <= t_max (the step cap grows with the length)
  h->l_cap_alloc = step_cap(&c, c.t_max);
  h->l_cap = h->l_cap_alloc;
  p.l_cap = h->l_cap_alloc;

  // (the score kernel's grid is whole eights of utterances: what it reads first has entries for the last of them)
  const size_t U8 = ((size_t)U + 7) & ~(size_t)7;
  const size_t UW = (size_t)U * Wb, UW8 = U8 * Wb;
  int rc;
#define A(ptr, n) if ((rc = dev_alloc(h, &(ptr), (n))) != CTCBS_OK) return rc
  A(p.xT, (size_t)U * V * p.Tp);
  A(p.Bcum, (size_t)U * p.Tp);
  A(p.lens, (size_t)U); A(p.lmax, (size_t)U);
  for (int b = 0; b < 2; ++b) {
    A(p.gphi[b], UW * p.Tp); A(p.gb[b], UW * p.Tp);
    A(p.rec[b], UW8);
  }
  A(p.uinfo, U8);
  {
    const size_t nc = p.keep_cand == KEEP_ARRAYS ? UW * K : 1;   // (not kept: never touched)
    const size_t nd = h->dense ? UW * dense_row(K) : nc;
    A(p.cand_id, nc); A(p.cand_inc, nd); A(p.cand_att, nd);
    A(p.cand_pre, !h->dense && (c.end_flags & CTCBS_END_EOS_RUN) ? nc : 1);
    A(p.cand_ctc, nc); A(p.cand_joint, p.keep_cand == KEEP_PAIRS ? 2 * UW * K : nc);
    A(p.dense_F, h->dense ? UW * p.Tp : 1); A(p.dense_slot, h->dense ? 2 * UW : 1); A(p.dense_eos, h->dense ? 2 * UW : 1);
    A(p.dense_left, h->dense ? UW : 1);
    const size_t n_best = h->dense ? (size_t)U * ((K + 15) / 16) * dense_pitch(Wb) : 1;
    A(p.dense_best, n_best);
    HIPCHK(hipMemsetAsync(p.dense_best, 0xff, n_best * sizeof(double), h->stream));   // (NaN: no score)
  }
  A(p.grp, UW); A(p.grp_list, UW * Wb);
  A(p.utt, (size_t)U); A(p.finished, U8);   /* read as whole words by the score kernel */ A(p.cells, (size_t)U); A(p.groups, (size_t)U);
  A(p.n_finished, (size_t)1); A(p.union_win, p.union_utt ? (size_t)4 * U : (size_t)4); A(p.err, (size_t)1);
  const size_t trie_n = (size_t)(h->l_cap_alloc + 1) * UW;
  A(p.trie_parent, trie_n * 3); p.trie_token = p.trie_parent + trie_n; p.trie_tau = p.trie_token + trie_n;
  A(p.out_parent, UW * 5); p.out_token = p.out_parent + UW; p.out_score = (float*)(p.out_token + UW);
  p.out_tau = p.out_parent + 3 * UW; p.out_tau_end = p.out_tau + UW;
  A(p.out_live, UW * 3); p.out_eos_added = p.out_live + UW; p.out_stopped = p.out_eos_added + UW;
  if (UW8 > UW)                                  // utterances that do not exist: their records stay dead
    for (int b = 0; b < 2; ++b) HIPCHK(hipMemsetAsync(p.rec[b] + UW, 0, (UW8 - UW) * sizeof(HypRec), h->stream));
#ifdef CTCBS_TRACE
  A(p.trace, UW * 16);
#endif
  h->res_cap = h->l_cap_alloc;
#undef A

  {
    const size_t n_setup = 4 + (size_t)2 * U, n_res = (size_t)U * h->res_cap;
    const size_t o_setup = 64, o_res = o_setup + ((n_setup * 4 + 63) & ~(size_t)63);
    const size_t bytes = o_res + ((size_t)U * 4 + n_res * 2) * 4;
    void* hp = nullptr;
    hipError_t e = hipHostMalloc(&hp, bytes, hipHostMallocMapped);
    if (e != hipSuccess) { g_last_hip = (int)e; (void)hipGetLastError(); return CTCBS_ENOMEM; }
    h->h_pin = hp;
    void* dp = nullptr;
    HIPCHK(hipHostGetDevicePointer(&dp, hp, 0));
    h->h_flag = (unsigned long long*)hp;
    *h->h_flag = 0;
    p.host_progress = (unsigned long long*)dp;
    h->h_setup = (int32_t*)((char*)hp + o_setup);
    h->d_setup = (const int32_t*)((char*)dp + o_setup);
    auto results = [&](void* base) {
      Results r;
      r.ntok = (int32_t*)((char*)base + o_res); r.flags = r.ntok + U; r.err = r.flags + U;
      r.score = (float*)(r.err + U);
      r.tokens = (int32_t*)(r.score + U); r.frames = r.tokens + n_res;
      return r;
    };
    h->h_res = results(hp); h->d_res = results(dp);
  }
  // launch shapes of the per-step kernels
  h->score_block = 256;
  // (a batch-wide window is about as wide as its margins where labels come at about the same rate in all utterances: 21 utterances,
  // margins of 5 and 60, 1525 us a decode against 1549 with the form for wide windows)
  // (no window is wider than the longest utterance, and three frames more where it does not start on a multiple of four)
  const int longest = c.t_max + 3;
  const int margins = c.win_m1 >= 0 && c.win_m2 >= 0 && c.win_m1 + c.win_m2 < longest ? c.win_m1 + c.win_m2 + 1 + 3 : longest;
  h->score_form = margins <= 128 ? 0 : (c.win_m1 >= 0 && c.win_m2 >= 0 && margins <= 192 ? 1 : 2);
  // Wider windows: three candidates per chain and 128 frames a round where the last round has few empty places (33 to 48 candidates),
  // else two and 192: an empty place costs what a candidate does.  74 utterances of 359 to 983 frames, whole, beam 2, us a
  // decode, three / two: 16 candidates 2848 / 2601, 24 2886 / 2786, 32 2885 / 2794, 40 2840 / 2946, 50 3373 / 3167, 64 3516 / 3293; 16
  // utterances, beam 10: 16 candidates 2391 / 2216, 64 2961 / 2747; 16 of 200 to 500 frames, 40 candidates 1405 / 1430.
  if (h->score_form == 2 && K <= 64 && (K <= 32 || K > 48)) h->score_form = 1;
  // LDS of the score kernel: the short list (or the radix histogram), the f terms, the per-candidate arrays
  size_t off = restricted ? (size_t)PIVOT_CAP * 8 : 0;
  h->off_f = (int32_t)off;
  // the f terms, padded to whole rounds of the column loads, which NEAR starts anywhere in the window
  h->score_bigk = K > 64 || V > 65536;
  const int round_frames = 4 * 16 * (h->score_form == 1 ? 3 : (h->score_form == 2 && h->score_bigk ? 4 : 2));
  h->wp_max = (p.Tp + round_frames - 1) / round_frames * round_frames + (h->score_form != 0 && !h->score_bigk ? round_frames : 0);
  h->want_near = h->score_form != 0 && !h->score_bigk && !h->dense;
  const size_t terms = (size_t)2 * h->wp_max * 4, gran = restricted ? (size_t)4 * ShortList::GCAP * 20 : 0;   // (the short list's granules lie there before)
  off += terms > gran ? terms : gran;
  h->off_small = (int32_t)off;
  off += (size_t)(h->score_bigk ? (K <= h->score_block ? K : 0) : 64) * 32 + 8;
  h->score_nv4 = V <= 3072 ? 3 : (V <= 5120 ? 5 : (V <= 10240 ? 10 : 16));
  h->score_smem_bytes = off;
  if (off + STATIC_LDS > 160 * 1024) return CTCBS_EINVAL;
  // Survivors of the select kernels: per-hypothesis windows whose margins keep them within 128 (256) frames, but for a
  // hypothesis whose two time indices lie far apart, go 16 lanes x 8 frames (32 x 8) each, others 64 x 8.
  const int span = c.win_union ? longest : margins;
  h->select_lps = span <= 128 ? 16 : (span <= 256 ? 32 : 64);
  h->select_wide = span > 128;
  // one wave for the ended set and one round of the others for the new hypotheses, as far as a work-group goes
  const int nw = 1 + (Wb * h->select_lps + 63) / 64;
  h->select_block = 64 * (nw <= 4 ? 4 : (nw <= 8 ? 8 : 16));

  return ingest(h, d_ctc_logp, h_lens);
}

extern "C" int ctcbs_create(const ctcbs_config_t* cfg, const float* d_ctc_logp, const int32_t* h_lens,
                            ctcbs_t** out) {
  if (out) *out = nullptr;
  if (!cfg || !d_ctc_logp || !h_lens || !out) return CTCBS_EINVAL;
  int rc = validate(cfg);
  if (rc != CTCBS_OK) return rc;
  ctcbs* h = new (std::nothrow) ctcbs();
  if (!h) return CTCBS_ENOMEM;
  h->h_pin = nullptr;
  h->cfg = *cfg;
  h->stream = (hipStream_t)cfg->stream;
  if (hipGetDevice(&h->device) != hipSuccess) { g_last_hip = (int)hipGetLastError(); delete h; return CTCBS_EHIP; }
  rc = create_impl(h, d_ctc_logp, h_lens);
  if (rc != CTCBS_OK) { free_all(h); delete h; return rc; }
  *out = h;
  return CTCBS_OK;
}

// Kernels that want more than 64 KB of LDS (`bytes` dynamic ones beside their own) need the attribute raised first.  It belongs to
// the kernel, not to a handle: it is only ever raised (handles of different sizes, on different
// threads, share it), and only when a launch needs more than what is already allowed.
static hipError_t allow_lds(const void* kernel, size_t bytes) {
  if (bytes + STATIC_LDS <= 64 * 1024) return hipSuccess;
  static std::mutex mu;
  static std::map<const void*, size_t> allowed;
  std::lock_guard<std::mutex> lock(mu);
  try {
    size_t& have = allowed[kernel];
    if (bytes <= have) return hipSuccess;
    hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) have = bytes;
    return e;
  } catch (...) {                                          // (the map could not grow)
    return hipErrorOutOfMemory;
  }
}

template <int BLOCK, int CB, int IT, int NV4, bool NEAR, bool BIGK>
static hipError_t launch_score_as(ctcbs* h, const Params& p, const float* att, int l) {
  static_assert(LastArg<decltype(&k_score<BLOCK, CB, IT, NV4, NEAR, BIGK>)>::offset() == offsetof(ScoreKernarg, late), "score_late reads them there");
  hipError_t ea = allow_lds((const void*)k_score<BLOCK, CB, IT, NV4, NEAR, BIGK>, h->score_smem_bytes);
  if (ea != hipSuccess) return ea;
  const int in_regs = p.restricted && p.V >= 8 && p.V <= 4 * NV4 * BLOCK ? 1 : 0;
  const int sh = 3;                              // (also below eight utterances: one of 437 frames 1090 -> 1035 us a decode)
  const int flags = in_regs | (p.U * p.Wb <= CTCBS_EARLY_GROUPS ? 2 : 0) | sh << 4 | (p.K == 1 ? 0 : p.Wb - 1) << 8;
  const dim3 grid(1u << sh, (unsigned)p.Wb, (unsigned)(p.U + (1 << sh) - 1) >> sh);
  ScoreArgs a;
  a.xT = p.xT; a.Bcum = p.Bcum; a.gphi = p.gphi[h->cur]; a.gb = p.gb[h->cur];
  a.lambda = p.lambda; a.beta = p.beta;
  a.Tp = p.Tp; a.K = p.K; a.blank_id = p.blank_id; a.eos_id = p.eos_id; a.win_m1 = p.win_m1; a.win_m2 = p.win_m2;
  a.end_flags = p.end_flags; a.eos_run = p.eos_run; a.wp_max = h->wp_max; a.off_f = h->off_f; a.off_small = h->off_small;
  a.mode = (p.restricted ? SC_RESTRICTED : 0) | (p.att_logits ? SC_LOGITS : 0) | (p.win_union ? SC_UNION : 0) |
           (p.keep_cand == KEEP_ARRAYS ? SC_KEEP : 0) | (p.keep_cand == KEEP_PAIRS ? SC_PAIRS : 0) | (p.union_utt ? SC_UNION_UTT : 0);
  a.err = p.err;
  ScoreLate b;
  b.grp_list = p.grp_list; b.grp = p.grp; b.union_win = p.union_win; b.n_finished = p.n_finished; b.host_progress = p.host_progress;
  b.cand_id = p.cand_id; b.cand_inc = p.cand_inc; b.cand_att = p.cand_att; b.cand_pre = p.cand_pre; b.cand_ctc = p.cand_ctc;
  b.cand_joint = p.cand_joint; b.trace = p.trace;
  hipLaunchKernelGGL((k_score<BLOCK, CB, IT, NV4, NEAR, BIGK>), grid, dim3(BLOCK), h->score_smem_bytes,
                     h->stream, (const HypRec*)p.rec[h->cur], (const UttInfo*)p.uinfo, (const uint32_t*)p.finished,
                     att, (int)p.Wb, (int)p.V, flags, l, (int)p.U, a, b);
  return hipGetLastError();
}

// the kernel's form: registers for the row as the vocabulary needs them (up to 3072, 5120, 10240, 16384 ids; larger
// ones never hold it), and the paths for many candidates only where they can be taken (see k_score)
template <int BLOCK, int CB, int IT, bool NEAR>
static hipError_t launch_score(ctcbs* h, const Params& p, const float* att, int l) {
  if (h->score_bigk) {                             // (wide windows: 2 x 4)
    constexpr int CBK = NEAR && IT == 2 ? 2 : CB, ITK = NEAR && IT == 2 ? 4 : IT;
    if (h->score_nv4 <= 5) return launch_score_as<BLOCK, CBK, ITK, 5, false, true>(h, p, att, l);
    return launch_score_as<BLOCK, CBK, ITK, 16, false, true>(h, p, att, l);
  }
  switch (h->score_nv4) {
    case 3: return launch_score_as<BLOCK, CB, IT, 3, NEAR, false>(h, p, att, l);
    case 5: return launch_score_as<BLOCK, CB, IT, 5, NEAR, false>(h, p, att, l);
    case 10: return launch_score_as<BLOCK, CB, IT, 10, NEAR, false>(h, p, att, l);
    default: return launch_score_as<BLOCK, CB, IT, 16, NEAR, false>(h, p, att, l);
  }
}

// Every id a candidate.  32 candidates per work-group where that gives every compute unit its four work-groups (each reads
// the slots' F once), and where chunks of 16 leave the select kernel more of them than its lanes hold (4096; us a decode with 16 / 32
// candidates, beam 20, 1500 frames, 5000 ids: one utterance 5105 / 4702, three 5708 / 5164, six 6945 / 5949; 9000 ids, beam 10, one 4621 / 4437);
// 16 otherwise (20 utterances of 400 to 900 frames, 1000 ids, 640 work-groups of 32: 2968 / 3196).
template <int NT>
static hipError_t launch_dense_scores(ctcbs* h, const Params& p, int l) {
  const dim3 grid((unsigned)(p.K + 16 * NT - 1) / (16 * NT), (unsigned)p.U);
#define CTCBS_DENSE(MT)                                                                                            \
  hipLaunchKernelGGL((k_dense_scores<NT, MT>), grid, dim3(256), 0, h->stream, (const float*)p.xT, (const float*)p.dense_F, \
                     (const DenseSlot*)p.dense_slot, (int)p.Wb, (int)p.Tp, (int)p.V, (int)p.K, p, l, h->cur)
  if (p.Wb <= 16) CTCBS_DENSE(1); else CTCBS_DENSE(2);
#undef CTCBS_DENSE
  return hipGetLastError();
}
#ifndef CTCBS_WIDE_CHUNKS          // (a CPU build of the tests sets 1)
#define CTCBS_WIDE_CHUNKS 1024     // work-groups of 32 candidates from which on there are no smaller ones
#endif
static int dense_chunk_bits(const Params& p) {
  return (long long)p.U * ((p.K + 31) / 32) >= CTCBS_WIDE_CHUNKS || (long long)dense_pitch(p.Wb) * ((p.K + 15) / 16) > 256 * DENSE_KEYS ? 5 : 4;
}
static bool split_select(const Params& p) { return p.U * p.Wb <= CTCBS_SPLIT_GROUPS; }
static hipError_t launch_dense(ctcbs* h, const Params& p, const float* att, int l) {
  if (l == 1 || !split_select(p)) {                        // (else the select kernel of the step before has done it)
    hipLaunchKernelGGL((k_dense_prep<256>), dim3(p.Wb, p.U), dim3(256), (size_t)p.Tp * 4, h->stream, p, l, h->cur);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  Params q = p;
  q.dense_att = att;
  return dense_chunk_bits(p) == 5 ? launch_dense_scores<2>(h, q, l) : launch_dense_scores<1>(h, q, l);
}

// The groups' lists from joint scores in global memory.  Up to 8192 scores stay in registers between the passes.
static hipError_t launch_lists(ctcbs* h, const Params& p) {
  const dim3 grid(p.Wb, p.U);
#define CTCBS_LIST(E) hipLaunchKernelGGL((k_list_top<E>), grid, dim3(256), 0, h->stream, p, h->cur)
  if (p.K <= 1024) CTCBS_LIST(4); else if (p.K <= 5120) CTCBS_LIST(20); else if (p.K <= 8192) CTCBS_LIST(32); else CTCBS_LIST(0);
#undef CTCBS_LIST
  return hipGetLastError();
}

// Looks at the progress word after step l has been enqueued, without draining the stream, and keeps the host
// from running more than a few steps ahead of the device: far enough that the device always has work queued
// (a step's launches take the host less time than the device needs to run them), and no further, because every
// step that is already queued when the last utterance finishes still runs, for nothing (a dead step takes about
// 6 us; with a look every eight steps and two intervals of lead, up to sixteen of them ended every decode).  A caller who
// asks for a look at more than CTCBS_POLL_CLOSE steps' distance wants to be let go on: it gets its two intervals.
#define CTCBS_STEPS_AHEAD 5
#define CTCBS_POLL_CLOSE 16
static int steps_ahead(int poll_every) {
  const int two = 2 * (poll_every < (1 << 20) ? poll_every : 1 << 20);   // (no decode has more steps)
  return poll_every > CTCBS_POLL_CLOSE || two < CTCBS_STEPS_AHEAD ? two : CTCBS_STEPS_AHEAD;
}
static int follow_progress(ctcbs* h, int l) {
  const int ahead = steps_ahead(h->cfg.poll_every);
  unsigned long long v = *(volatile unsigned long long*)h->h_flag;
  if ((int)(v >> 32) + ahead < l) {
    // (the wait ends: the stream's work ends, or hipStreamQuery reports why it does not)
    std::chrono::steady_clock::time_point asked = std::chrono::steady_clock::now();
    for (long spins = 1;; ++spins) {
      v = *(volatile unsigned long long*)h->h_flag;
      if ((int)(v >> 32) + ahead >= l) break;
      if ((spins & 63) != 0) continue;
      const auto now = std::chrono::steady_clock::now();
      if (now - asked < std::chrono::milliseconds(1)) {
        if (spins > (1 << 14)) std::this_thread::yield();
        continue;
      }
      asked = now;
      const hipError_t e = hipStreamQuery(h->stream);
      if (e == hipSuccess) { v = *(volatile unsigned long long*)h->h_flag; break; }   // everything enqueued has run
      if (e != hipErrorNotReady) { g_last_hip = (int)e; return CTCBS_EHIP; }
    }
  }
  h->known_finished = (int32_t)(uint32_t)v;
  return CTCBS_OK;
}

// One step with the kernels working on `p`: the handle's own parameter block, or a copy of it whose
// per-step scratch arrays lie elsewhere (ctcbs_step_static).
static int step_impl(ctcbs_t* h, const Params& with, const float* d_att_logp, ctcbs_step_out_t* out) {
  if (!h || !d_att_logp) return CTCBS_EINVAL;
  if (h->known_finished >= with.U || h->step >= h->l_cap) return CTCBS_DONE;
  const int l = h->step + 1;
  Params p = with;
  if (h->dense) { p.dense_slot += (size_t)h->cur * p.U * p.Wb; p.dense_eos += (size_t)h->cur * p.U * p.Wb; }
  hipEvent_t* ev = nullptr;
  if (h->profiling && h->ev_used + 3 <= h->events.size()) {
    ev = &h->events[h->ev_used];
    h->ev_used += 3;
    HIPCHK(hipEventRecord(ev[0], h->stream));
  }
  hipError_t e;
  if (h->dense) e = launch_dense(h, p, d_att_logp, l);
  else
    e = h->score_form == 0 ? launch_score<256, 3, 2, false>(h, p, d_att_logp, l)
        : h->score_form == 1 ? launch_score<256, 2, 3, true>(h, p, d_att_logp, l)
                             : launch_score<256, 3, 2, true>(h, p, d_att_logp, l);
  HIPCHK(e);
  if (ev) HIPCHK(hipEventRecord(ev[1], h->stream));       // (a list builder below counts as selection)
  if (!h->dense && p.K > h->score_block) HIPCHK(launch_lists(h, p));
  // Small batches leave most compute units idle in the one-work-group-per-utterance form: there the
  // split form (one work-group per new beam slot, each ranking the utterance's lists itself) is
  // faster.  Large batches fill the chip either way and the Wb-fold repeated ranking only costs.  Split / per
  // utterance, us per launch, windows of 101 frames:
  //   beam 4:  512 groups 7.3 / 8.7, 1024 8.0 / 8.9, 2048 9.5 / 9.7, 4096 11.8 / 10.7
  //   beam 10: 640 7.6 / 9.0, 1280 8.7 / 9.3, 2560 10.3 / 10.0, 5120 14.1 / 11.7
  //   beam 20: 1280 10.2 / 10.9, 2560 14.4 / 11.6, 5120 21.3 / 12.1
  // (windows of 161 frames, beam 20: 1280 14.0 / 12.5, 2560 20.8 / 13.2: there the line would lie lower)
  const bool split = split_select(p);
  size_t sel_lds = (size_t)36 * ((p.Wb * p.Wb + 63) & ~63) + 32;
  if (h->dense) {                                          // (no keys; split: then dense_terms)
    sel_lds = (size_t)20 * ((p.Wb * p.Wb + 63) & ~63) + (size_t)DenseTopList::BYTES * p.Wb;
    if (split && sel_lds < (size_t)p.Tp * 4) sel_lds = (size_t)p.Tp * 4;
  }
  SelectArgs a;
  const int nxt = h->cur ^ 1;
  a.xT = p.xT; a.Bcum = p.Bcum; a.gphi = p.gphi[h->cur]; a.gb = p.gb[h->cur]; a.gphi_new = p.gphi[nxt]; a.gb_new = p.gb[nxt];
  a.rec_new = p.rec[nxt]; a.trie = p.trie_parent + (size_t)l * p.U * p.Wb; a.out = p.out_parent; a.out8 = p.out_live;
  a.trie_stride = (uint32_t)(p.trie_token - p.trie_parent);
  a.U = p.U; a.V = p.V; a.Tp = p.Tp; a.blank_id = p.blank_id; a.end_flags = p.end_flags; a.end_m = p.end_m; a.end_c = p.end_c;
  a.end_d = p.end_d; a.win_union = p.win_union; a.win_m2 = p.win_m2; a.want_near = h->want_near; a.err = p.err; a.finished = p.finished;
  a.n_finished = p.n_finished; a.cells = p.cells; a.groups = p.groups; a.union_win = p.union_win; a.trace = p.trace;
  a.lambda = p.lambda; a.slots = p.dense_slot; a.beta = p.beta; a.win_m1 = p.win_m1; a.dense_F = p.dense_F;
  a.slots_next = h->p.dense_slot + (size_t)nxt * p.U * p.Wb; a.eos_next = h->p.dense_eos + (size_t)nxt * p.U * p.Wb;
  a.best = p.dense_best; a.inc = p.cand_inc; a.att = p.cand_att; a.K = p.K; a.eos_id = p.eos_id;
  a.chunk_bits = dense_chunk_bits(p); a.n_chunks = (p.K + (1 << a.chunk_bits) - 1) >> a.chunk_bits; a.pitch = dense_pitch(p.Wb);
  const int wb_m = (65536 / p.Wb + 1) << 8 | p.Wb;         // (see k_select)
#define CTCBS_SELECT(K, G, BS, LDS, L)                                                                       \
  hipLaunchKernelGGL(K, G, dim3(BS), LDS, h->stream, (const HypRec*)p.rec[h->cur], p.utt, (const GroupOut*)p.grp, \
                     (const ListEntry*)p.grp_list, (const UttInfo*)p.uinfo, wb_m, L, (int)p.U, a)
  if (split) {
    const int sh = 3;
    const dim3 grid(1u << sh, (unsigned)p.Wb + 1, (unsigned)(p.U + (1 << sh) - 1) >> sh);
    if (h->dense) CTCBS_SELECT((k_select_split<256, false, true>), grid, 256, sel_lds, l | sh << 28);
    else if (h->want_near) CTCBS_SELECT((k_select_split<256, true, false>), grid, 256, sel_lds, l | sh << 28);
    else if (h->select_wide || p.Wb > 12) CTCBS_SELECT((k_select_split<256, false, false>), grid, 256, sel_lds, l | sh << 28);
    else CTCBS_SELECT((k_select_split<64, false, false>), grid, 64, sel_lds, l | sh << 28);
  } else {
    const dim3 grid(p.U);
#define CTCBS_SELECT_LPS(BS, D)                                                              \
  do {                                                                                       \
    if (h->select_lps == 16) CTCBS_SELECT((k_select<BS, 16, 8, D>), grid, BS, sel_lds, l);   \
    else if (h->select_lps == 32) CTCBS_SELECT((k_select<BS, 32, 8, D>), grid, BS, sel_lds, l); \
    else CTCBS_SELECT((k_select<BS, 64, 8, D>), grid, BS, sel_lds, l);                       \
  } while (0)
    switch (h->select_block) {
      case 256: if (h->dense) CTCBS_SELECT_LPS(256, true); else CTCBS_SELECT_LPS(256, false); break;
      case 512: if (h->dense) CTCBS_SELECT_LPS(512, true); else CTCBS_SELECT_LPS(512, false); break;
      default: if (h->dense) CTCBS_SELECT_LPS(1024, true); else CTCBS_SELECT_LPS(1024, false); break;
    }
#undef CTCBS_SELECT_LPS
  }
#undef CTCBS_SELECT
  HIPCHK(hipGetLastError());
  if (ev) HIPCHK(hipEventRecord(ev[2], h->stream));
  h->step = l;
  h->cur ^= 1;
  h->p_step = p;                           // where this step's intermediate arrays lie (ctcbs_peek)
  int polled = -1;
  if (h->cfg.poll_every > 0) {
    const int rc = follow_progress(h, l);
    if (rc != CTCBS_OK) return rc;
    if (l % h->cfg.poll_every == 0) polled = h->known_finished;
  }
  if (out) {
    out->step = l; out->n_finished = polled;
    out->d_parent = p.out_parent; out->d_token = p.out_token; out->d_score = p.out_score;
    out->d_live = p.out_live; out->d_finished = p.finished; out->d_tau = p.out_tau;
    out->d_tau_end = p.out_tau_end; out->d_eos_added = p.out_eos_added; out->d_stopped = p.out_stopped;
  }
  return CTCBS_OK;
}

extern "C" int ctcbs_step(ctcbs_t* h, const float* d_att_logp, ctcbs_step_out_t* out) {
  if (!h || !d_att_logp) return CTCBS_EINVAL;
  return step_impl(h, h->p, d_att_logp, out);
}

// ---- the step for callers that cannot allocate --------------------------------------------------
// Same kernels, same results; the arrays that carry a step's intermediate values from the score kernel
// to the select kernel (windows, eos scores, the groups' best-first lists, stop flags, work counts) lie
// in a fixed array in the library's own image instead of memory the handle allocated.  Every GPU holds
// its own copy of that array at its own address, so its address is asked for once per device.
#define CTCBS_STATIC_SCRATCH_BYTES ((11u << 19) + 512u)   // (what static_step_takes lets in at most, see there)
#define CTCBS_MAX_DEVICES 64
static __device__ __align__(256) unsigned char scratch[CTCBS_STATIC_SCRATCH_BYTES];
static std::mutex g_scratch_mu;
static unsigned char* g_scratch_ptr[CTCBS_MAX_DEVICES];     // device address of `scratch` on each device (0: not asked yet)

// What the call takes: a limit of its interface (include/ctcbs.h), not of the arrays as they are laid out now.
static bool static_step_takes(const ctcbs* h) {
  const Params& p = h->p;
  if (p.K > h->score_block) return false;
  // every id a candidate: only long inputs
  if (!p.restricted && !(p.end_flags & CTCBS_END_EOS_RUN) && !p.att_logits && !p.win_union &&
      p.Tp <= 2048 && (size_t)4 * p.Wb * p.Tp <= 150 * 1024) return false;
  // 40 bytes per group and 24 per list entry within 4 MiB, in arrays of 4 and 8 bytes an entry, each rounded up to 256.  (A
  // group's line holds 64 now: at most 24 more for each of at most 65536 groups, a beam of 1.)
  const size_t UW = (size_t)p.U * p.Wb, L = UW * p.Wb;
  auto r = [](size_t n) { return (n + 255) & ~(size_t)255; };
  return 4 * r(UW * 4) + 3 * r(UW * 8) + r(L * 8) + 4 * r(L * 4) <= (4u << 20);
}

extern "C" int ctcbs_step_static(ctcbs_t* h, const float* d_att_logp, ctcbs_step_out_t* out) {
  if (!h || !d_att_logp) return CTCBS_EINVAL;
  if (!static_step_takes(h)) return CTCBS_EINVAL;
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev != h->device || dev < 0 || dev >= CTCBS_MAX_DEVICES) return CTCBS_ESTATE;   // the handle's device must be current
  unsigned char* base = nullptr;
  {
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
      void* ptr = nullptr;
      HIPCHK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
      g_scratch_ptr[dev] = (unsigned char*)ptr;
    }
    base = g_scratch_ptr[dev];
  }
  if (!base) return CTCBS_EHIP;
  if (h->known_finished >= h->p.U || h->step >= h->l_cap) return CTCBS_DONE;
  Params p = h->p;
  const size_t UW = (size_t)p.U * p.Wb, L = UW * p.Wb;
  size_t off = 0;
  auto take = [&](size_t bytes) { unsigned char* q = base + off; off += (bytes + 255) & ~(size_t)255; return q; };
  // (the array keeps what the last call on this GPU, of any handle, left: the score kernel writes every group's
  // line, and the select kernel reads no list entry past a line's count)
  p.grp = (GroupOut*)take(UW * sizeof(GroupOut));
  p.grp_list = (ListEntry*)take(L * sizeof(ListEntry));
  if (off > CTCBS_STATIC_SCRATCH_BYTES) return CTCBS_EINVAL;   // (cannot be, see static_step_takes)
  return step_impl(h, p, d_att_logp, out);
}

extern "C" int ctcbs_reset(ctcbs_t* h, const float* d_ctc_logp, const int32_t* h_lens) {
  if (!h || !d_ctc_logp || !h_lens) return CTCBS_EINVAL;
  return ingest(h, d_ctc_logp, h_lens);
}

extern "C" int ctcbs_poll(ctcbs_t* h, int32_t* n_finished) {
  if (!h) return CTCBS_EINVAL;
  int32_t v = 0;
  HIPCHK(hipMemcpyAsync(&v, h->p.n_finished, sizeof v, hipMemcpyDeviceToHost, h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  h->known_finished = v;
  if (n_finished) *n_finished = v;
  return CTCBS_OK;
}

extern "C" int ctcbs_finalize(ctcbs_t* h, int32_t* h_tokens, int32_t cap, int32_t* h_ntok, float* h_score,
                              int32_t* h_frames, int32_t* h_flags) {
  if (!h || !h_tokens || !h_ntok || !h_score || cap < 0) return CTCBS_EINVAL;
  const int U = h->p.U, rc_cap = h->res_cap;
  const size_t fin_lds = (size_t)(h->l_cap_alloc + 1) * h->p.Wb + (size_t)h->l_cap_alloc + 1;
  const int use_lds = fin_lds <= 60 * 1024;
  hipLaunchKernelGGL((k_finalize<256>), dim3(U), dim3(256), use_lds ? fin_lds : 0, h->stream, h->p, h->cur,
                     h->step, rc_cap, use_lds, h_frames != nullptr ? 1 : 0, h->d_res);
  HIPCHK(hipGetLastError());
  HIPCHK(hipStreamSynchronize(h->stream));
  const Results& r = h->h_res;
  int32_t err = 0;
  for (int u = 0; u < U; ++u) err |= r.err[u];
  if (err != 0) return CTCBS_ESTATE;     // a kernel's consistency check failed during this decode: no result
  for (int u = 0; u < U; ++u) {
    const int n = r.ntok[u];
    h_score[u] = r.score[u];
    if (n < 0 || n > cap) return CTCBS_ECAP;
    h_ntok[u] = n;
    memcpy(h_tokens + (size_t)u * cap, r.tokens + (size_t)u * rc_cap, (size_t)n * 4);
    if (h_frames) memcpy(h_frames + (size_t)u * cap, r.frames + (size_t)u * rc_cap, (size_t)n * 4);
    if (h_flags) h_flags[u] = r.flags[u];
  }
  return CTCBS_OK;
}

extern "C" int ctcbs_stats(ctcbs_t* h, uint64_t* cells, uint64_t* groups, int32_t* steps) {
  if (!h) return CTCBS_EINVAL;
  std::vector<unsigned long long> c(h->p.U), g(h->p.U);
  HIPCHK(hipMemcpyAsync(c.data(), h->p.cells, c.size() * 8, hipMemcpyDeviceToHost, h->stream));
  HIPCHK(hipMemcpyAsync(g.data(), h->p.groups, g.size() * 8, hipMemcpyDeviceToHost, h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  unsigned long long tot = 0, gt = 0;
  for (auto v : c) tot += v;
  for (auto v : g) gt += v;
  if (cells) *cells = tot;
  if (groups) *groups = gt;
  if (steps) *steps = h->step;
  return CTCBS_OK;
}

extern "C" int ctcbs_profile(ctcbs_t* h, int32_t enable) {
  if (!h) return CTCBS_EINVAL;
  if (enable && h->events.empty()) {
    h->events.resize((size_t)3 * (h->l_cap_alloc + 1));
    for (size_t i = 0; i < h->events.size(); ++i) {
      hipError_t e = hipEventCreate(&h->events[i]);
      if (e != hipSuccess) {
        for (size_t k = 0; k < i; ++k) (void)hipEventDestroy(h->events[k]);
        h->events.clear();
        g_last_hip = (int)e;
        return CTCBS_EHIP;
      }
    }
  }
  h->profiling = enable != 0;
  h->ev_used = 0;
  return CTCBS_OK;
}

extern "C" int ctcbs_profile_read(ctcbs_t* h, double* score_ms, double* select_ms, int32_t* n_steps) {
  if (!h) return CTCBS_EINVAL;
  HIPCHK(hipStreamSynchronize(h->stream));
  double a = 0.0, b = 0.0;
  for (size_t i = 0; i + 3 <= h->ev_used; i += 3) {
    float ms = 0.0f;
    HIPCHK(hipEventElapsedTime(&ms, h->events[i], h->events[i + 1])); a += ms;
    HIPCHK(hipEventElapsedTime(&ms, h->events[i + 1], h->events[i + 2])); b += ms;
  }
  if (score_ms) *score_ms = a;
  if (select_ms) *select_ms = b;
  if (n_steps) *n_steps = (int32_t)(h->ev_used / 3);
  return CTCBS_OK;
}

extern "C" int ctcbs_peek(ctcbs_t* h, int32_t what, void* h_dst, size_t bytes, size_t* need) {
  if (!h) return CTCBS_EINVAL;
  const Params& p = h->step > 0 ? h->p_step : h->p;
  const size_t UW = (size_t)p.U * p.Wb;
  const void* src = nullptr; size_t sz = 0;
  int32_t k = p.K;
  const bool cand = what == CTCBS_PEEK_CAND_ID || what == CTCBS_PEEK_CAND_CTC || what == CTCBS_PEEK_CAND_JOINT;
  if (cand && p.keep_cand == KEEP_NONE && !h->dense) return CTCBS_ESTATE;   // created without keep_candidates
  switch (what) {
    case CTCBS_PEEK_CAND_ID: src = p.cand_id; sz = UW * p.K * 4; break;
    case CTCBS_PEEK_CAND_CTC: src = p.cand_ctc; sz = UW * p.K * 8; break;
    case CTCBS_PEEK_CAND_JOINT: src = p.cand_joint; sz = UW * p.K * 8; break;
    case CTCBS_PEEK_WIN_S: case CTCBS_PEEK_WIN_E: sz = UW * 4; break;
    case CTCBS_PEEK_CTC_EOS: case CTCBS_PEEK_JOINT_EOS: sz = UW * 8; break;
    case CTCBS_PEEK_N_CAND:
      if (need) *need = 4;
      if (h_dst && bytes >= 4) memcpy(h_dst, &k, 4);
      return CTCBS_OK;
    default: return CTCBS_EINVAL;
  }
  if (need) *need = sz;
  if (h_dst && bytes && cand && p.keep_cand != KEEP_ARRAYS) {
    // every id a candidate: ids ascend; scores lie there in pairs, or follow from increments and attention values
    const int lo_ex = p.blank_id < p.eos_id ? p.blank_id : p.eos_id, hi_ex = p.blank_id < p.eos_id ? p.eos_id : p.blank_id;
    const size_t w = what == CTCBS_PEEK_CAND_ID ? 4 : 8, K = (size_t)p.K;
    const bool pairs = p.keep_cand == KEEP_PAIRS;
    try {
      std::vector<DenseLeft> slots(pairs ? 0 : UW);
      std::vector<float> inc(pairs ? 0 : K), att(pairs ? 0 : K);
      std::vector<double> both(pairs ? 2 * K : 0);
      if (!pairs) HIPCHK(hipMemcpyAsync(slots.data(), p.dense_left, UW * sizeof(DenseLeft), hipMemcpyDeviceToHost, h->stream));
      HIPCHK(hipStreamSynchronize(h->stream));
      for (size_t g = 0; g < UW && g * K * w < bytes; ++g) {
        if (pairs) HIPCHK(hipMemcpyAsync(both.data(), p.cand_joint + 2 * g * K, 16 * K, hipMemcpyDeviceToHost, h->stream));
        else {
          HIPCHK(hipMemcpyAsync(inc.data(), p.cand_inc + g * dense_row(p.K), 4 * K, hipMemcpyDeviceToHost, h->stream));
          HIPCHK(hipMemcpyAsync(att.data(), p.cand_att + g * dense_row(p.K), 4 * K, hipMemcpyDeviceToHost, h->stream));
        }
        HIPCHK(hipStreamSynchronize(h->stream));
        for (size_t c = 0; c < K && (g * K + c + 1) * w <= bytes; ++c) {
          char* d = (char*)h_dst + (g * K + c) * w;
          int32_t id = (int32_t)c;
          if (id >= lo_ex) ++id;
          if (id >= hi_ex) ++id;
          double ctc = LOG0D, joint = LOG0D;
          if (pairs) { joint = both[2 * c]; ctc = both[2 * c + 1]; }
          else if (inc[c] > LOG0_CLASS) {
            ctc = slots[g].offr + (double)inc[c];
            joint = dense_joint(p.lambda, dense_base(p.lambda, slots[g]), inc[c], att[c]);
          }
          if (what == CTCBS_PEEK_CAND_ID) memcpy(d, &id, w);
          else memcpy(d, what == CTCBS_PEEK_CAND_CTC ? &ctc : &joint, w);
        }
      }
    } catch (const std::bad_alloc&) { return CTCBS_ENOMEM; }
  } else if (h_dst && bytes && !src) {                            // a field of the groups' lines
    std::vector<GroupOut> g(UW);
    HIPCHK(hipMemcpyAsync(g.data(), p.grp, UW * sizeof(GroupOut), hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
    for (size_t i = 0; i < UW; ++i) {
      const size_t w = sz / UW;
      if ((i + 1) * w > bytes) break;
      char* d = (char*)h_dst + i * w;
      if (what == CTCBS_PEEK_WIN_S) memcpy(d, &g[i].win_s, w);
      else if (what == CTCBS_PEEK_WIN_E) memcpy(d, &g[i].win_e, w);
      else if (what == CTCBS_PEEK_CTC_EOS) memcpy(d, &g[i].ctc_eos, w);
      else memcpy(d, &g[i].joint_eos, w);
    }
  } else if (h_dst && bytes) {
    HIPCHK(hipMemcpyAsync(h_dst, src, bytes < sz ? bytes : sz, hipMemcpyDeviceToHost, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
  }
  return CTCBS_OK;
}

#ifdef CTCBS_TRACE
extern "C" int ctcbs_trace_read(ctcbs_t* h, unsigned long long* dst) {
  HIPCHK(hipMemcpyAsync(dst, h->p.trace, (size_t)h->p.U * h->p.Wb * 16 * 8, hipMemcpyDeviceToHost, h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  return CTCBS_OK;
}
#endif

#include "sched.h"

extern "C" void ctcbs_destroy(ctcbs_t* h) {
  if (!h) return;
  (void)hipStreamSynchronize(h->stream);
  for (hipEvent_t e : h->events) (void)hipEventDestroy(e);
  free_all(h);
  delete h;
}
