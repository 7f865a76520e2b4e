// Device functions of the kernels on their own, for tests/test_kernel_units.py: built like the rest of the CPU
// emulation, with the library's (copied) sources included.
#include "ctcbs.cpp"

// Sums of ncol candidates' terms over 4 * n4 frames (n4 a multiple of LPC * IT), as the score kernel forms them.
template <int LPC, int IT>
static void unit_chain_kernel(const float* x, const float* f, int ncol, int n4, float* out) {
  const int lane = threadIdx.x, q = lane % LPC;
  for (int c0 = 0; c0 < ncol; c0 += 64 / LPC) {
    const int c = min(c0 + lane / LPC, ncol - 1);
    const float4 *col = (const float4*)x + (size_t)c * n4, *ft = (const float4*)f + (size_t)c * n4;
    float4 y[IT], g[IT];
    for (int it = 0; it < IT; ++it) { y[it] = col[q + it * LPC]; g[it] = ft[q + it * LPC]; }
    ChainSum a = chain_first<LPC, IT>(y, g);
    for (int i0 = LPC * IT; i0 < n4; i0 += LPC * IT) {
      for (int it = 0; it < IT; ++it) { y[it] = col[i0 + q + it * LPC]; g[it] = ft[i0 + q + it * LPC]; }
      chain_more<LPC, IT>(a, y, g);
    }
    const float r = chain_finish<LPC>(a);
    if (q == 0) out[c] = r;
  }
}
extern "C" int unit_chain(int lpc, int it, const float* x, const float* f, int ncol, int n4, float* out) {
  if (n4 % (lpc * it) != 0) return -1;
#define UNIT_CHAIN(L, I) if (lpc == L && it == I) { hipLaunchKernelGGL((unit_chain_kernel<L, I>), dim3(1), dim3(64), 0, nullptr, x, f, ncol, n4, out); return 0; }
  UNIT_CHAIN(16, 2) UNIT_CHAIN(16, 3) UNIT_CHAIN(16, 4) UNIT_CHAIN(64, 4)
#undef UNIT_CHAIN
  return -1;
}

// One utterance's increments from the slots' F (mref: their M), every id a candidate: x [V][Tp], F [Wb][Tp], out [Wb][V - 2].
extern "C" int unit_dense(const float* x, const float* F, const float* mref, int T, int Tp, int V, int Wb, float* out) {
  Params p;
  memset(&p, 0, sizeof p);
  UttInfo ui{T, T, 0.0};
  alignas(4) uint8_t finished[4] = {0, 0, 0, 0};
  std::vector<DenseSlot> slots(Wb);
  for (int j = 0; j < Wb; ++j) { memset(&slots[j], 0, sizeof slots[j]); slots[j].last = -1; slots[j].s = 1; slots[j].e = T; slots[j].mref = mref[j]; }
  p.U = 1; p.V = V; p.Wb = Wb; p.K = V - 2; p.Tp = Tp; p.blank_id = 0; p.eos_id = V - 1; p.win_m1 = p.win_m2 = -1;
  p.finished = finished; p.uinfo = &ui;
  std::vector<float> att((size_t)Wb * V), kept((size_t)Wb * dense_row(p.K)), inc(kept.size());
  p.cand_inc = inc.data();
  std::vector<double> best((size_t)((p.K + 15) / 16) * dense_pitch(Wb));
  std::vector<DenseEos> eos(Wb);
  std::vector<DenseLeft> left(Wb);
  std::vector<GroupOut> grp(Wb);
  unsigned long long progress = 0;
  int32_t n_finished = 0;
  p.dense_att = att.data(); p.cand_att = kept.data(); p.dense_best = best.data(); p.dense_eos = eos.data(); p.dense_left = left.data();
  p.grp = grp.data(); p.host_progress = &progress; p.n_finished = &n_finished;
  const dim3 grid((unsigned)(p.K + 15) / 16, 1);
  if (Wb <= 16) hipLaunchKernelGGL((k_dense_scores<1, 1>), grid, dim3(256), 0, nullptr, x, F, slots.data(), Wb, Tp, V, p.K, p, 1, 0);
  else hipLaunchKernelGGL((k_dense_scores<1, 2>), grid, dim3(256), 0, nullptr, x, F, slots.data(), Wb, Tp, V, p.K, p, 1, 0);
  for (int j = 0; j < Wb; ++j) memcpy(out + (size_t)j * p.K, &inc[(size_t)j * dense_row(p.K)], (size_t)p.K * 4);
  return 0;
}
// The best Wb of all (slot, candidate) pairs: increments and attention values inc, att [Wb][K], the slots' base, in chunks of 1 << bits.  Out, per
// rank: score, slot, place; returns how many reached the pivot (or, after rounds, the last best chunk's score), n_chunks how many chunks.
template <int BLOCK>
static void unit_top_kernel(SelectArgs p, DenseTopLds<BLOCK>* t, unsigned char* lds, const double* base, int Wb, double* J, int* slot, int* place, int* counts) {
  double key[DENSE_KEYS];
  dense_fetch<BLOCK>(p, 0, key);
  if ((int)threadIdx.x < Wb) t->base[threadIdx.x] = base[threadIdx.x];
  lds_barrier();
  const int n = dense_top<BLOCK>(p, *t, DenseTopList(lds, Wb), 0, Wb, key, [&](int rank, double score, int s, int c, float, float) { J[rank] = score; slot[rank] = s; place[rank] = c; });
  if (threadIdx.x == 0) { counts[0] = n; counts[1] = t->n_chunks; }
}
extern "C" void unit_top(int block, double lambda, const float* inc, const float* att, const double* base, int Wb, int K, int bits, double* J, int* slot, int* place, int* counts) {
  SelectArgs p;
  memset(&p, 0, sizeof p);
  const int Kr = dense_row(K);
  std::vector<float> inc_rows((size_t)Wb * Kr), att_rows((size_t)Wb * Kr);
  for (int j = 0; j < Wb; ++j) {
    memcpy(&inc_rows[(size_t)j * Kr], inc + (size_t)j * K, (size_t)K * 4);
    memcpy(&att_rows[(size_t)j * Kr], att + (size_t)j * K, (size_t)K * 4);
  }
  p.lambda = lambda; p.inc = inc_rows.data(); p.att = att_rows.data(); p.K = K; p.chunk_bits = bits; p.n_chunks = (K + (1 << bits) - 1) >> bits; p.pitch = dense_pitch(Wb);
  std::vector<double> best((size_t)p.n_chunks * p.pitch, __builtin_nan(""));
  for (int c = 0; c < p.n_chunks; ++c)
    for (int j = 0; j < Wb; ++j) {
      double& b = best[(size_t)c * p.pitch + j];
      b = LOG0D;
      for (int k = c << bits; k < min(K, (c + 1) << bits); ++k) b = fmax(b, dense_joint(lambda, base[j], inc[(size_t)j * K + k], att[(size_t)j * K + k]));
    }
  p.best = best.data();
  unsigned char* lds = (unsigned char*)malloc((size_t)DenseTopList::BYTES * Wb);
  memset(lds, 0xa5, (size_t)DenseTopList::BYTES * Wb);
  auto run = [&](auto block_size) {
    constexpr int BLOCK = decltype(block_size)::value;
    DenseTopLds<BLOCK>* t = (DenseTopLds<BLOCK>*)malloc(sizeof(DenseTopLds<BLOCK>));
    memset((void*)t, 0xa5, sizeof *t);
    hipLaunchKernelGGL(unit_top_kernel<BLOCK>, dim3(1), dim3(BLOCK), 0, nullptr, p, t, lds, base, Wb, J, slot, place, counts);
    free(t);
  };
  if (block == 1024) run(Const<1024>()); else run(Const<256>());
  free(lds);
}
// The pivot for rows of log-probabilities: s_hist 256 words, mx the lanes' 256 maxima.
static void unit_pivot_kernel(uint32_t* s_hist, const float* mx, int K, float* out) {
  s_hist[threadIdx.x] = 0;
  lds_barrier();
  pivot_count(s_hist, mx[threadIdx.x]);
  lds_barrier();
  const float L = find_pivot_hist<256>(s_hist, mx, K);
  if ((threadIdx.x & 63) == 0) out[threadIdx.x >> 6] = L;
}
extern "C" void unit_pivot(const float* mx, int K, float* out) {
  alignas(16) uint32_t s_hist[256];
  alignas(16) float s_mx[256];
  memcpy(s_mx, mx, sizeof s_mx);
  hipLaunchKernelGGL(unit_pivot_kernel, dim3(1), dim3(256), 0, nullptr, (uint32_t*)s_hist, (const float*)s_mx, K, out);
}
extern "C" void unit_exp(const float* v, int n, float* out) { for (int i = 0; i < n; ++i) out[i] = exp_exact(v[i]); }
extern "C" int unit_steps_ahead(int poll_every) { return steps_ahead(poll_every); }
// column loads (one float4 of one lane each) of the score kernel so far, where the build counts them
extern "C" long long unit_columns() { return emu::n_columns; }
// atomicOr calls so far
extern "C" long long unit_atomic_ors() { return emu::n_atomic_or; }
// whether an utterance's posteriors were found to be no log-posteriors
extern "C" int unit_above0(const ctcbs* h, int u) { return h->p.uinfo[u].above0; }
// which forms of the kernels a handle runs: bits 0-1 score kernel's window form, 2 more than 64 candidates, 3 every id's own kernels, 4 near
// frames are looked for, 8-15 lanes per new hypothesis (select kernel of large batches)
extern "C" int unit_forms(const ctcbs* h) {
  return h->score_form | (h->score_bigk ? 4 : 0) | (h->dense ? 8 : 0) | (h->want_near ? 16 : 0) | h->select_lps << 8;
}
