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
