// Gate and up products of a prompt chunk with the SwiGLU as their epilogue
// (Sec. 3.3: the activation fused into the producing kernel): the plan and the
// launches of qgemm.h's kSwiglu mode.
#include "qgemm.h"

namespace qm {
namespace {

template <int BM, int WN, int WK, int FMT>
hipError_t launch_swiglu_tile(const QgemmArgs& a, hipStream_t st) {
  const int64_t panels = padded_rows(a.N) / kPanel;
  const int64_t blocks = WN == 1 ? 2 * panels : (2 * panels + WN - 1) / WN;
  const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>((a.M + BM - 1) / BM));
  hipLaunchKernelGGL((qgemm_kernel<BM, WN, WK, QgMode::kSwiglu, 2, false, FMT>), grid, dim3(WN * WK * 64), 0, st, a);
  return hipGetLastError();
}

}  // namespace

// The tile of the two matrices side by side (gemm_plan of 2n columns).  Those of
// several panels pair gate and up wavefronts; the single-panel ones pair column
// halves (32 gate and 32 up columns per workgroup), while 64 x 128 tiles would
// leave half the CUs or more without a workgroup, and give way to 64 x 128 with
// 2-way split-K above that.  Measured against the grouped GEMM and the
// elementwise kernel (us): Q4 2048 -> 2 x 8192 at m = 512 52.6 -> 42.4, at 128
// 22.2 -> 17.6; 1024 -> 2 x 3072 at m = 512 20.4 -> 15.6.  64 x 128 / single-panel
// tile: 3072 -> 2 x 8192 at m = 48 (128 workgroups of 64 x 128) Q8 22.1 / 17.5 (two
// calls 19.9), 4096 -> 2 x 3072 at 96 (96) 25.2 / 18.7, at 160 (144) 26.0 / 33.4,
// 2048 -> 2 x 5632 at 96 (176) Q4 15.6 / 18.2.
hipError_t launch_gemm_swiglu(int32_t fmt, const uint8_t* qg, const uint16_t* sg, const uint8_t* qu,
                              const uint16_t* su, const uint16_t* x, uint16_t* h, int64_t m, int64_t n, int64_t k,
                              int cu_count, hipStream_t st) {
  if (n == 0) return hipSuccess;
  QgemmArgs a{};
  a.a = x; a.M = m; a.K = k; a.N = n; a.h = h;
  a.q = qg; a.s = sg; a.q2 = qu; a.s2 = su;
  a.gq[0] = qg; a.gs[0] = sg; a.gq[1] = qu; a.gs[1] = su;
  const FewrowPlan f = fewrow_swiglu_plan(fmt, m, n, k, cu_count);
  if (f.rt != 0) return launch_fewrow_swiglu(a, fmt, f, st);
  const GemmPlan p = gemm_plan(m, 2 * padded_rows(n), k, cu_count);
  auto go = [&](auto ft) -> hipError_t {
    constexpr int F = decltype(ft)::value;
    if (p.bm == 128) return launch_swiglu_tile<128, 4, 1, F>(a, st);
    if (p.bm == 64 && p.wn == 4 && p.wk == 2) return launch_swiglu_tile<64, 4, 2, F>(a, st);
    if (p.bm == 64 && p.wn == 4) return launch_swiglu_tile<64, 4, 1, F>(a, st);
    // (Other single-panel plans have so few workgroups that they are on the
    // few-row kernel, but for activations it cannot address.)
    if (p.wn == 1 && 2 * (padded_rows(n) / kPanel) * ((m + 63) / 64) <= cu_count) {
      if (p.bm == 64 && p.wk == 8) return launch_swiglu_tile<64, 1, 8, F>(a, st);
      if (p.bm == 64 && p.wk == 4) return launch_swiglu_tile<64, 1, 4, F>(a, st);
      if (p.bm == 32 && p.wk == 4) return launch_swiglu_tile<32, 1, 4, F>(a, st);
      if (p.bm == 32 && p.wk == 2) return launch_swiglu_tile<32, 1, 2, F>(a, st);
      if (p.bm == 32 && p.wk == 1) return launch_swiglu_tile<32, 1, 1, F>(a, st);
    }
    return launch_swiglu_tile<64, 2, 2, F>(a, st);
  };
  switch (fmt) {
    case QM_Q4_G32: return go(std::integral_constant<int, QM_Q4_G32>{});
    case QM_Q8_G32: return go(std::integral_constant<int, QM_Q8_G32>{});
    case QM_Q2_G32: return go(std::integral_constant<int, QM_Q2_G32>{});
    case QM_Q3_G32: return go(std::integral_constant<int, QM_Q3_G32>{});
    case QM_Q5_G32: return go(std::integral_constant<int, QM_Q5_G32>{});
    case QM_Q6_G32: return go(std::integral_constant<int, QM_Q6_G32>{});
    case QM_F16: return go(std::integral_constant<int, QM_F16>{});
    case QM_BF16: return go(std::integral_constant<int, QM_BF16>{});
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qm
