// Shared device-side definitions of the ctcbs kernels (gfx950, wave64).
//
// Numeric form.  Every hypothesis g keeps two CTC forward variables per frame (all its paths, the
// paper's phi_t(g) of Eq. (3), and those of them that end in blank) as fp32 values in a STORED form: gamma_t(g) = stored_t + B_t + off'(g), with B_t the
// utterance's cumulative blank log-posterior (fp64, Params::Bcum) and off'(g) an fp64 offset
// per hypothesis (HypRec::off).  Staying in blank leaves the stored value unchanged, so stored
// values are O(1) near the frames that matter however long the utterance is and however
// negative the cumulative score has become; the parts that grow (B_t, off') and the cumulative
// CTC, attention and joint scores are fp64, one add per hypothesis and step.
// log0 is the finite sentinel -1e30 (anything below -1e29 is treated as log0).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#define CTCBS_WAVE 64
#define LOG0F (-1.0e30f)
#define LOG0_CLASS (-1.0e29f)
#define LOG0D (-1.0e30)
// Blank log-posteriors enter the per-frame reference B_t (see Params::Bcum) floored at this value, so
// that B_t stays finite even if a frame gives blank probability zero.
#define BLANK_FLOOR (-1.0e4f)
#define MAX_BEAM 32
// A prefix score is a sum over frames of exp(f + x), x <= 0, and most of it comes from the frames round the hypothesis's last
// label: away from them f falls by nats with every label that is missed.  A record says which frames have f above
// -NEAR_DEPTH; the score kernel sums those, and others only for candidates whose sum does not exceed by 2^26 (NEAR_MARGIN)
// all that they could add, their number times exp(-NEAR_DEPTH) (those among them that can count).  (Increments of 40 candidates lie 9
// to 16 nats below the largest f on posteriors of 5000 ids, whose bound is -20 for 300 frames left out.)  Where a "log-posterior" above NEAR_X_MAX was given,
// that bound does not hold and all frames are summed.
#define NEAR_DEPTH 44.0f
#define NEAR_MARGIN 18.1f
#define NEAR_X_MAX 0.0625f
#define NEAR_ENOUGH 8
#define MAX_END_M 8
#define MAX_EOS_RUN 32

// Phase time stamps for kernel tuning; compiled in only with -DCTCBS_TRACE (never in the
// shipped library).  TRACE_POINT stores at once (cheap to place, but the store is then waited
// for by the next wait on the memory counter); TRACE_MARK keeps the stamp in registers and
// TRACE_FLUSH stores them all at the end of the kernel, which leaves the timing undisturbed.
#ifdef CTCBS_TRACE
#define TRACE_POINT(p, blk, i) do { if ((p).trace && threadIdx.x == 0) (p).trace[(size_t)(blk) * 16 + (i)] = wall_clock64(); } while (0)
#define TRACE_DECL unsigned long long tr_[16] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}
#define TRACE_MARK(i) do { tr_[i] = wall_clock64(); } while (0)
#define TRACE_MARK_AT(ptr, i) do { (ptr)[i] = wall_clock64(); } while (0)
#define TRACE_ARG tr_
#define TRACE_FLUSH(p, blk) do { if ((p).trace && threadIdx.x == 0) { _Pragma("unroll") for (int i_ = 0; i_ < 16; ++i_) if (tr_[i_]) (p).trace[(size_t)(blk) * 16 + i_] = tr_[i_]; } } while (0)
#else
#define TRACE_POINT(p, blk, i) do { } while (0)
#define TRACE_DECL do { } while (0)
#define TRACE_MARK(i) do { } while (0)
#define TRACE_MARK_AT(ptr, i) do { } while (0)
#define TRACE_ARG nullptr
#define TRACE_FLUSH(p, blk) do { } while (0)
#endif

typedef float f32x4 __attribute__((__vector_size__(16)));

struct UttState {            // per utterance, touched by one thread of the select kernel
  double best_score;         // best joint score in the ended set
  double ring_score[MAX_END_M];  // best ended score per length, lengths l, l-1, ... (ring by l % M)
  double fb_score;
  int32_t ring_tag[MAX_END_M];
  int32_t n_ended, best_step, best_slot, cnt_tau_T;
  int32_t finished_step;     // 0 while running
  int32_t pad;
};

// One hypothesis of the current beam: a 64-byte line, so that a work-group fetches the whole
// record of its hypothesis with one uniform (scalar-path) load.
struct __align__(64) HypRec {
  int32_t live;              // slot holds a hypothesis
  int32_t last;              // its last label (-1: the empty hypothesis)
  int32_t rs, re;            // stored range of its forward variables (log0 outside)
  int32_t tau, tau_end;      // first argmax of the label / blank variable (the two argmax equations of Sec. 3.2.2)
  int32_t ref;               // reference frame r: prefix-score increments are relative to off' + B_r
  uint32_t near_frames;            // first and last frame (16 bits each) whose phi is within NEAR_DEPTH of off' + B_r (none: last < first)
  double off;                // off'(g): log psi(g) = off'(g) + B_r(g) up to the rounding of the re-basing
  double att;                // cumulative attention log-prob, Eq. (2)
  double joint;              // joint score of the hypothesis, Eq. (1)
  double bref;               // B_r (copied from Bcum so that no load depends on `ref`)
};

struct ListEntry {           // one entry of a group's best-first list
  double J;                  // joint score
  int32_t tok;
  float inc, att;            // prefix-score increment, this step's attention log-prob
  int32_t pad;
};

// What the score kernel hands to the select kernel about one group, in one 64-byte line.
struct __align__(64) GroupOut {
  int32_t n;                 // entries of the group's best-first list
  int32_t stopped;           // eos-run rule fired
  int32_t win_s, win_e;      // window (empty: win_e < win_s)
  double ctc_eos, joint_eos; // eos scores
  long long cells;           // prefix-score terms
  int32_t pad[6];
};

struct __align__(32) UttInfo {   // per utterance, constant over a decode
  int32_t T, lmax;           // frames, step cap
  double BT;                 // B_T
  int32_t above0;            // some log-posterior is above NEAR_X_MAX
  int32_t pad[3];
};

struct DenseSlot;            // (k_score.h)
struct DenseEos;
struct DenseLeft;

// nothing (every id a candidate: what k_dense.h leaves); all arrays; joint and prefix score side by side in cand_joint
enum { KEEP_NONE = 0, KEEP_ARRAYS = 1, KEEP_PAIRS = 2 };

struct Params {
  // sizes and configuration
  int32_t U, V, Wb, K, Tp, t_max, blank_id, eos_id;
  int32_t restricted;        // 1: top-K attention candidates; 0: every id but blank/eos
  int32_t att_logits;        // 1: the step input holds unnormalised logits (log_softmax folded in)
  int32_t win_union;         // 1: one window for the whole batch (min start / max end over all hypotheses)
  int32_t win_m1, win_m2, end_flags, end_m, end_c, eos_run, l_cap;
  float end_d;
  double lambda, beta;
  // posteriors, token-major: xT[(u*V + k)*Tp + t] = log p^c(z_t = k), t = 1..T_u; 0 elsewhere
  float* xT;
  int32_t* lens;             // [U]
  int32_t* lmax;             // [U] step cap per utterance
  // Cumulative blank log-posterior per utterance, fp64: Bcum[u*Tp + t] = sum_{v<=t} max(x_v(blank),
  // BLANK_FLOOR), Bcum[u*Tp] = 0.  Forward variables are stored with B_t taken out: for a hypothesis
  // g with offset off'(g), gamma_t(g) = stored_t + B_t + off'(g).  On the path that stays in blank the
  // stored value does not change from frame to frame, so stored values stay within tens of nats of
  // zero however long the utterance is, and the large part (B_t) is carried in fp64.
  double* Bcum;
  UttInfo* uinfo;            // [U]
  // hypothesis state, two buffers (index b): forward variables [b][U][Wb][Tp] (stored form) and
  // per-hypothesis records [b][U][Wb].  gphi: phi_t = n_t (+) b_t, gb: b_t; the label variable n_t alone is needed
  // while its hypothesis is made only (every later use is of the sum, or of b_t if the label repeats)
  float* gphi[2];
  float* gb[2];
  HypRec* rec[2];
  float* dense_F;            // [U][Wb][Tp] every id a candidate: exp of the f terms (k_dense.h)
  DenseSlot* dense_slot;     // [2][U][Wb], by the record's buffer (a step's: its own)
  DenseEos* dense_eos;       // [2][U][Wb] (likewise)
  DenseLeft* dense_left;     // [U][Wb] what ctcbs_peek needs of the last step in which a slot held a hypothesis
  double* dense_best;        // [U][chunks][dense_pitch] the best joint score that each slot has in each work-group's candidates (NaN: none)
  const float* dense_att;    // this step's attention rows
  int32_t keep_cand;         // KEEP_*: which of the per-candidate arrays below a step fills (ctcbs_peek; large K needs them)
  // per-step scratch between the score and the select kernel
  int32_t* cand_id;          // [U][Wb][K]
  float* cand_inc;           // [U][Wb][K] log psi(g.c) - off(g) (every id a candidate: rows of dense_row(K))
  float* cand_att;           // [U][Wb][K] this step's attention log-prob of c (likewise)
  float* cand_pre;           // [U][Wb][K] scratch of the eos-run rule
  double* cand_ctc;          // [U][Wb][K] log psi(g.c)
  double* cand_joint;        // [U][Wb][K]
  GroupOut* grp;             // [U][Wb]
  ListEntry* grp_list;       // [U][Wb][Wb] the group's best-first list
  // utterance state
  UttState* utt;             // [U]
  uint8_t* finished;         // [U]
  unsigned long long* cells; // [U] prefix-score terms so far
  unsigned long long* groups;// [U] live (utterance, beam) groups so far
  int32_t* n_finished;       // [1]
  int32_t* err;              // [1] bits set by the kernels' own consistency checks (0: none failed)
  // batch-wide window, per step parity: (min tau, max of min(tau~ + M2, T)) over live hypotheses; [2][2] for the whole
  // batch, or [2][U][2] per utterance (split select kernel: its work-groups do not know whether the utterance finishes)
  int32_t* union_win;
  int32_t union_utt;         // 1: per utterance
  unsigned long long* host_progress;   // [1] in pinned host memory, see publish_progress
  // back-pointer trie, level l holds the hypotheses of length l: [l_cap+1][U][Wb]
  int32_t* trie_parent;
  int32_t* trie_token;
  int32_t* trie_tau;
  // step outputs
  int32_t* out_parent;
  int32_t* out_token;
  float* out_score;
  uint8_t* out_live;
  int32_t* out_tau;
  int32_t* out_tau_end;
  uint8_t* out_eos_added;
  uint8_t* out_stopped;
  unsigned long long* trace; // [max(U*Wb, U)][16] per-block phase time stamps (tuning builds only)
};

// Kernel arguments that a work-group needs early, kept in one block of few 64-byte lines: left to itself the compiler
// fetches arguments one by one where they are first used, and in a kernel of a few microseconds every first touch
// of a line is a trip to memory in a chain of them.  PIN makes a value be in scalar registers from here on, so that
// loads written above it are issued together and waited for once.  LOADED does the same for vector registers: without it
// the compiler moves a load into the branch that alone uses it, behind the arrival of the loads before, and a
// round of loads becomes a chain of them; FETCH is a load that stays where it is written, without a wait.  SCHED_FENCE: no instruction is moved across (a prefetch stays ahead of the work).
// OPAQUE: what follows from a scalar is worked out again, not kept.  STORE_ASIDE, LOAD_ASIDE: past the L2, which holds what the kernels read again.  STORE_FLAG: several
// may store it, all the same value, for later kernels.
#if defined(__AMDGCN__)
#define PIN4(a, b, c, d) __asm__ volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d))
#define LOADED(a) __asm__ volatile("" : "+v"(a))
#define OPAQUE(a) __asm__ volatile("" : "+s"(a))
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
#define FETCH(ptr) __hip_atomic_load(ptr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT)
#define FETCH_SCALAR(ptr) (*(const __attribute__((address_space(4))) int32_t*)(unsigned long long)(ptr))   // (uniform address, written by earlier kernels only)
#define STORE_ASIDE(v, ptr) __builtin_nontemporal_store(v, ptr)
#define STORE_FLAG(v, ptr) __hip_atomic_store(ptr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT)
#define LOAD_ASIDE(ptr) __builtin_nontemporal_load(ptr)
#else
#define PIN4(a, b, c, d) do { } while (0)
#define LOADED(a) do { } while (0)
#define OPAQUE(a) do { } while (0)
#define SCHED_FENCE() do { } while (0)
#define FETCH(ptr) (*(ptr))
#define FETCH_SCALAR(ptr) (*(const int32_t*)(ptr))
#define STORE_ASIDE(v, ptr) (*(ptr) = (v))
#define STORE_FLAG(v, ptr) __atomic_store_n(ptr, v, __ATOMIC_RELAXED)
#define LOAD_ASIDE(ptr) (*(ptr))
#endif

// arguments of the score kernel behind the preloaded ones
struct ScoreArgs {
  const float* xT;
  const double* Bcum;
  const float *gphi, *gb;    // of the current buffer
  double lambda, beta;
  int32_t Tp, K, blank_id, eos_id, win_m1, win_m2, end_flags, eos_run;
  int32_t wp_max, off_f, off_small;   // LDS layout: floats per f array, byte offsets
  int32_t mode;              // SC_* bits
  int32_t* err;
};
// those that it needs late, or not every time: read where they are used (score_late), not held from the start.  Loaded early with
// the others they ran the kernel out of scalar registers: 16 to 20 went into lanes of a vector register at once, so that the first
// thing every wave did was to wait for its arguments, and the record was asked for a trip to memory later (one utterance
// 1011 -> 1005 us a decode, 512 8380 -> 8338).
struct ScoreLate {
  ListEntry* grp_list;
  GroupOut* grp;
  int32_t* union_win;
  const int32_t* n_finished;
  unsigned long long* host_progress;
  int32_t* cand_id;
  float *cand_inc, *cand_att, *cand_pre;
  double *cand_ctc, *cand_joint;
  unsigned long long* trace;
};
struct ScoreKernarg {        // all of them, as they lie in the kernel's argument segment
  const HypRec* rec_now;
  const UttInfo* uinfo;
  const uint32_t* fin_words;
  const float* att;
  int32_t Wb, V, flags, l, U;
  ScoreArgs p;
  ScoreLate late;
};
// where a kernel's last argument lies in that segment: each argument at the next multiple of its alignment
template <class F>
struct LastArg;
template <class... A>
struct LastArg<void (*)(A...)> {
  static constexpr size_t offset() {
    size_t at = 0, last = 0;
    ((last = (at + alignof(A) - 1) / alignof(A) * alignof(A), at = last + sizeof(A)), ...);
    return last;
  }
};
#if defined(__AMDGCN__)
typedef const __attribute__((address_space(4))) ScoreLate* ScoreLatePtr;
__device__ __forceinline__ ScoreLatePtr score_late(const ScoreLate&) {
  const __attribute__((address_space(4))) char* k = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t at;
  __asm__ volatile("s_movk_i32 %0, %1" : "=s"(at) : "i"(offsetof(ScoreKernarg, late)));   // (a constant it could see, the compiler
  return (ScoreLatePtr)(k + at);                           // would load from early and hold with the others)
}
#else
typedef const ScoreLate* ScoreLatePtr;
__device__ __forceinline__ ScoreLatePtr score_late(const ScoreLate& q) { return &q; }
#endif
enum { SC_RESTRICTED = 1, SC_LOGITS = 2, SC_UNION = 4, SC_KEEP = 8, SC_UNION_UTT = 16, SC_PAIRS = 32 };

// arguments of the select kernels behind the preloaded ones
struct SelectArgs {
  const float* xT;
  const double* Bcum;
  const float *gphi, *gb;    // of the current buffer
  float *gphi_new, *gb_new;  // of the other one
  HypRec* rec_new;
  int32_t* trie;             // back-pointers of this level: parent, token, tau, each trie_stride apart
  int32_t* out;              // step outputs, each UW apart: parent, token, score (float), tau, tau_end
  uint8_t* out8;             // live, eos_added, stopped, each UW apart
  uint32_t trie_stride;
  int32_t U, V, Tp, blank_id, end_flags, end_m, end_c;
  float end_d;
  int32_t win_union, win_m2;
  int32_t want_near;         // the score kernel looks at HypRec::near_frames
  int32_t* err;
  uint8_t* finished;
  int32_t* n_finished;
  unsigned long long *cells, *groups;
  int32_t* union_win;
  unsigned long long* trace;
  // every id a candidate (dense_top)
  double lambda;
  const DenseSlot* slots;
  DenseSlot* slots_next;     // for the next step (dense_terms)
  DenseEos* eos_next;
  float* dense_F;
  double beta;
  int32_t win_m1;
  const double* best;        // (Params::dense_best)
  const float *inc, *att;    // [U][Wb][dense_row(K)]
  int32_t K, n_chunks, chunk_bits, eos_id;
  int32_t pitch;             // (dense_pitch)
};

// entries per chunk of Params::dense_best: odd, so that a chunk's slots and the slots' same chunks lie in places that differ modulo 64
// (dense_top); the spare entry is never written after ctcbs_create
__host__ __device__ __forceinline__ int dense_pitch(int Wb) { return Wb | 1; }

// floats in a row of increments, or attention values, where every id is a candidate: whole 128-byte lines, so that a work-group's share of a
// row is lines of its own (the work-groups of an utterance are on different XCDs, and each writes its part of a shared line to memory by itself)
__host__ __device__ __forceinline__ int dense_row(int K) { return (K + 31) & ~31; }

// Order-preserving 64-bit image of a joint score; 0: not a competitor (log0, NaN).  And back.
__device__ __forceinline__ unsigned long long joint_image(double J) {
  const long long b = __double_as_longlong(J);
  return (unsigned long long)(b ^ ((b >> 63) | (long long)0x8000000000000000ull)) & (J > (double)LOG0_CLASS ? ~0ull : 0ull);
}
__device__ __forceinline__ double image_joint(unsigned long long k) {
  return __longlong_as_double((long long)((k >> 63) ? (k & 0x7fffffffffffffffull) : ~k));
}

// natural logarithm of a normal positive number: the hardware's log2 times ln 2 (about 1.5 ulp; the
// library's logf spends a dozen instructions more on denormal arguments and the last half ulp)
__device__ __forceinline__ float fast_logf(float x) { return __builtin_amdgcn_logf(x) * 0.69314718055994531f; }

__device__ __forceinline__ float lae(float a, float b) {
  // log(e^a + e^b); with both operands at the log0 sentinel the result stays in the log0 class
  float m = fmaxf(a, b);
  float d = -fabsf(a - b);
  return m + fast_logf(1.0f + __expf(d));
}

// Work-group barrier for data exchanged through LDS only.  __syncthreads() also waits for the
// wave's outstanding global loads and stores (they share one counter with nothing to tell them
// apart); here they stay in flight: prefetched rows and columns keep arriving, and stores of
// results nobody in this work-group reads back are not waited for.  Never use it to publish
// global memory to other waves of the block.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Between LDS stores of some lanes of a wave and LDS loads of the same addresses by other lanes of that
// wave.  The hardware needs nothing here (a wave's LDS instructions execute in order, all lanes of an
// instruction together); the call keeps the compiler from moving LDS accesses across this point and gives
// a CPU build of the kernels, where lanes are threads, its synchronisation point.
__device__ __forceinline__ void wave_lds_fence() { __builtin_amdgcn_wave_barrier(); }

// Consistency checks on indices that come from device data (candidate ids, list entries, time
// indices): a value outside its range is clamped into it, so that no access leaves its array, and
// the step's error bit is set; ctcbs_finalize then reports CTCBS_ESTATE instead of a result.
enum { ERR_CAND_ID = 1, ERR_WINDOW = 2, ERR_LIST_ENTRY = 4, ERR_TOKEN = 8, ERR_TIME_INDEX = 16, ERR_BACKTRACK = 32 };
template <class P>
__device__ __forceinline__ int checked(const P& p, int v, int lo, int hi, int bit) {
  if (v < lo || v > hi) { atomicOr(p.err, bit); v = v < lo ? lo : hi; }
  return v;
}

// The same for several values in a row: no branch for each (a branch costs a lone wave 40 cycles, taken or not), their
// bits are collected and reported together.
__device__ __forceinline__ int clamped(int v, int lo, int hi, int bit, int& bad) {
  const int c = min(max(v, lo), hi);
  bad |= c != v ? bit : 0;
  return c;
}
template <class P>
__device__ __forceinline__ void report(const P& p, int bad) {
  if (bad != 0) atomicOr(p.err, bad);
}

// For the host's non-blocking look: the step that has begun and the count of utterances finished before it, in one
// 64-bit store to pinned host memory (uncached: it needs no fence to arrive, and nothing here waits for it: as a volatile
// store, with the count through the vector path, the wave waited for its row, for the count and for the bus).  By one wave.
__device__ __forceinline__ void publish_progress(unsigned long long* host_progress, const int32_t* n_finished, int l) {
#if defined(__AMDGCN__)
  const int n = FETCH_SCALAR(n_finished);
  if ((threadIdx.x & 63) == 0)
    __hip_atomic_store(host_progress, (unsigned long long)(unsigned)l << 32 | (unsigned)n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
#else
  if ((threadIdx.x & 63) == 0) *(volatile unsigned long long*)host_progress = (unsigned long long)(unsigned)l << 32 | (unsigned)*n_finished;
#endif
}

__device__ __forceinline__ uint32_t near_pack(int lo, int hi) { return lo <= hi ? (uint32_t)lo | (uint32_t)hi << 16 : 0xffffu; }

__device__ __forceinline__ float canon0(float v) { return v < LOG0_CLASS ? LOG0F : v; }

// ---- wave64 data movement through DPP (no LDS round trip) -----------------------------------
// row_shr:n = 0x110+n and row_ror:n = 0x120+n act inside each row of 16 lanes; row_bcast:15
// (0x142) / row_bcast:31 (0x143) copy the last lane of a row / of the lower half-wave into
// the following row(s); wave_shr:1 = 0x138.  Lanes without a source keep `old`.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i(int old, int src) {
  return __builtin_amdgcn_update_dpp(old, src, CTRL, ROW_MASK, 0xf, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float old, float src) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src), CTRL, ROW_MASK,
                                                    0xf, false));
}

// all-reduce inside each row of 16 lanes (commutative op through rotations)
// (a rotation gives every lane a source, so there is no old value to keep: the move can then be folded
// into the instruction that consumes it)
template <int CTRL>
__device__ __forceinline__ float rot_f(float src) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(src), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, rot_f<0x128>(v));
  v = fmaxf(v, rot_f<0x124>(v));
  v = fmaxf(v, rot_f<0x122>(v));
  v = fmaxf(v, rot_f<0x121>(v));
  return v;
}
__device__ __forceinline__ float row16_sum(float v) {
  v += rot_f<0x128>(v);
  v += rot_f<0x124>(v);
  v += rot_f<0x122>(v);
  v += rot_f<0x121>(v);
  return v;
}
__device__ __forceinline__ int row16_min_i(int v) {
  v = min(v, dpp_i<0x128, 0xf>(v, v));
  v = min(v, dpp_i<0x124, 0xf>(v, v));
  v = min(v, dpp_i<0x122, 0xf>(v, v));
  v = min(v, dpp_i<0x121, 0xf>(v, v));
  return v;
}
__device__ __forceinline__ float lane_f(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
// a value that all lanes of the wave hold alike, into a scalar register: the compiler cannot know it of what comes
// from LDS or from a wave's number, and without it loops and choices on such values run on vector registers with lane masks
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
// n += how many of the values v of lanes I .. I + 7 exceed the lane's own.  A value that one instruction puts into a scalar
// register can be read by the second next at the earliest; left to itself the compiler waits out that distance after
// every readlane and every comparison when scalar registers are scarce, 20 cycles a value instead of 13.  A readlane must
// not follow the instruction that wrote its vector register at once: the compiler does not look into the block, and what it
// puts in front of it may be just that, a copy of v or of one of its halves; hence the s_nop in every block (one for every
// four values: 12.65 -> 13.0 us a launch of the split select kernel at beam 20).
// (& in the constraints: the counts are written while the values are still read)
#if defined(__AMDGCN__)
#define ABOVE_ADD                                                                                                  \
  "v_addc_co_u32_e64 %0, vcc, 0, %0, vcc\n\tv_addc_co_u32_e64 %0, s[40:41], 0, %0, s[40:41]\n\t"                   \
  "v_addc_co_u32_e64 %0, s[42:43], 0, %0, s[42:43]\n\tv_addc_co_u32_e64 %0, s[44:45], 0, %0, s[44:45]\n\t"
#define ABOVE_32(A, B, C, D)                                                                                       \
  "v_readlane_b32 vcc_lo, %1, " A "\n\tv_readlane_b32 s40, %1, " B "\n\t"                                          \
  "v_readlane_b32 s42, %1, " C "\n\tv_readlane_b32 s44, %1, " D "\n\t"                                             \
  "v_cmp_gt_u32_e64 vcc, vcc_lo, %1\n\tv_cmp_gt_u32_e64 s[40:41], s40, %1\n\t"                                     \
  "v_cmp_gt_u32_e64 s[42:43], s42, %1\n\tv_cmp_gt_u32_e64 s[44:45], s44, %1\n\t" ABOVE_ADD
#define ABOVE_64(A, B, C, D)                                                                                       \
  "v_readlane_b32 vcc_lo, %2, " A "\n\tv_readlane_b32 vcc_hi, %3, " A "\n\t"                                       \
  "v_readlane_b32 s40, %2, " B "\n\tv_readlane_b32 s41, %3, " B "\n\t"                                             \
  "v_readlane_b32 s42, %2, " C "\n\tv_readlane_b32 s43, %3, " C "\n\t"                                             \
  "v_readlane_b32 s44, %2, " D "\n\tv_readlane_b32 s45, %3, " D "\n\t"                                             \
  "v_cmp_gt_u64_e64 vcc, vcc, %1\n\tv_cmp_gt_u64_e64 s[40:41], s[40:41], %1\n\t"                                   \
  "v_cmp_gt_u64_e64 s[42:43], s[42:43], %1\n\tv_cmp_gt_u64_e64 s[44:45], s[44:45], %1\n\t" ABOVE_ADD
#endif
template <int I>
__device__ __forceinline__ void above8(uint32_t v, int& n) {
#if defined(__AMDGCN__)
  __asm__("s_nop 0\n\t" ABOVE_32("%2", "%3", "%4", "%5") ABOVE_32("%6", "%7", "%8", "%9")
          : "+&v"(n)
          : "v"(v), "i"(I), "i"(I + 1), "i"(I + 2), "i"(I + 3), "i"(I + 4), "i"(I + 5), "i"(I + 6), "i"(I + 7)
          : "vcc", "s40", "s41", "s42", "s43", "s44", "s45");
#else
  for (int k = 0; k < 8; ++k) n += (uint32_t)__builtin_amdgcn_readlane((int)v, I + k) > v ? 1 : 0;
#endif
}
template <int I>
__device__ __forceinline__ void above8(unsigned long long v, int& n) {
#if defined(__AMDGCN__)
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  __asm__("s_nop 0\n\t" ABOVE_64("%4", "%5", "%6", "%7") ABOVE_64("%8", "%9", "%10", "%11")
          : "+&v"(n)
          : "v"(v), "v"(lo), "v"(hi), "i"(I), "i"(I + 1), "i"(I + 2), "i"(I + 3), "i"(I + 4), "i"(I + 5), "i"(I + 6), "i"(I + 7)
          : "vcc", "s40", "s41", "s42", "s43", "s44", "s45");
#else
  for (int k = 0; k < 8; ++k) {
    const unsigned long long o = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), I + k) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, I + k);
    n += o > v ? 1 : 0;
  }
#endif
}
// na, nb += how many of the values v of lanes I .. I + 7 exceed the lane's own a, b.
#if defined(__AMDGCN__)
#define ABOVE_2(A, B, C, D)                                                                                        \
  "v_readlane_b32 s46, %2, " A "\n\tv_readlane_b32 s47, %2, " B "\n\t"                                             \
  "v_readlane_b32 s48, %2, " C "\n\tv_readlane_b32 s49, %2, " D "\n\t"                                             \
  "v_cmp_gt_u32_e64 vcc, s46, %3\n\tv_cmp_gt_u32_e64 s[40:41], s47, %3\n\t"                                        \
  "v_cmp_gt_u32_e64 s[42:43], s48, %3\n\tv_cmp_gt_u32_e64 s[44:45], s49, %3\n\t" ABOVE_ADD                         \
  "v_cmp_gt_u32_e64 vcc, s46, %4\n\tv_cmp_gt_u32_e64 s[40:41], s47, %4\n\t"                                        \
  "v_cmp_gt_u32_e64 s[42:43], s48, %4\n\tv_cmp_gt_u32_e64 s[44:45], s49, %4\n\t"                                   \
  "v_addc_co_u32_e64 %1, vcc, 0, %1, vcc\n\tv_addc_co_u32_e64 %1, s[40:41], 0, %1, s[40:41]\n\t"                   \
  "v_addc_co_u32_e64 %1, s[42:43], 0, %1, s[42:43]\n\tv_addc_co_u32_e64 %1, s[44:45], 0, %1, s[44:45]\n\t"
#endif
template <int I>
__device__ __forceinline__ void above8(uint32_t v, uint32_t a, uint32_t b, int& na, int& nb) {
#if defined(__AMDGCN__)
  __asm__("s_nop 0\n\t" ABOVE_2("%5", "%6", "%7", "%8") ABOVE_2("%9", "%10", "%11", "%12")
          : "+&v"(na), "+&v"(nb)
          : "v"(v), "v"(a), "v"(b), "i"(I), "i"(I + 1), "i"(I + 2), "i"(I + 3), "i"(I + 4), "i"(I + 5), "i"(I + 6), "i"(I + 7)
          : "vcc", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49");
#else
  for (int k = 0; k < 8; ++k) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)v, I + k);
    na += o > a ? 1 : 0; nb += o > b ? 1 : 0;
  }
#endif
}
// the same over the first `count` lanes (uniform, up to STEP - 1 more are counted: they hold values below every other)
template <int STEP, class V>
__device__ __forceinline__ int lanes_above(V v, int count) {
  int n = 0;
#define ABOVE_STEP(I)                                            \
  if ((I) % STEP == 0 && (I) >= count) return n;                 \
  above8<(I)>(v, n);
  ABOVE_STEP(0) ABOVE_STEP(8) ABOVE_STEP(16) ABOVE_STEP(24) ABOVE_STEP(32) ABOVE_STEP(40) ABOVE_STEP(48) ABOVE_STEP(56)
#undef ABOVE_STEP
  return n;
}
// inclusive prefix sum over the 64 lanes
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t x, int /*lane*/) {
  int v = (int)x;
  v += dpp_i<0x111, 0xf>(0, v);
  v += dpp_i<0x112, 0xf>(0, v);
  v += dpp_i<0x114, 0xf>(0, v);
  v += dpp_i<0x118, 0xf>(0, v);
  v += dpp_i<0x142, 0xa>(0, v);
  v += dpp_i<0x143, 0xc>(0, v);
  return (uint32_t)v;
}

// Exclusive prefix sum of one uint32 per thread over the block; *total = block sum.
// scratch: one uint32 per wave (+1).  Contains two barriers.
template <int BLOCK>
__device__ __forceinline__ uint32_t block_excl_scan_u32(uint32_t v, uint32_t* scratch, uint32_t* total) {
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  constexpr int NW = BLOCK / 64;
  uint32_t inc = wave_incl_scan_u32(v, lane);
  __syncthreads();                    // scratch may still be read from a previous use
  if (lane == 63) scratch[w] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    uint32_t s = scratch[i];
    if (i < w) base += s;
    tot += s;
  }
  *total = tot;
  return base + inc - v;
}

// Order-preserving map of an attention log-prob to uint32 (larger value -> larger key).
// Excluded ids get key 0, NaN gets key 1: both sort below every number, -inf included.
__device__ __forceinline__ uint32_t att_key(float v, int id, int blank_id, int eos_id) {
  if (id == blank_id || id == eos_id) return 0u;
  if (v != v) return 1u;
  uint32_t u = __float_as_uint(v);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// k-th candidate id when every id except blank and eos is a candidate (ascending ids).
__device__ __forceinline__ int full_v_id(int i, int lo_ex, int hi_ex) {
  int id = i;
  if (id >= lo_ex) ++id;
  if (id >= hi_ex) ++id;
  return id;
}
