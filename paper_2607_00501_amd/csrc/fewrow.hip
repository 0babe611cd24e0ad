// Dense launches of the few-row matmul kernel (fewrow.h): any format, one
// matrix or a group.
#include <cstdio>

#include "fewrow.h"

namespace qm {
namespace {

template <int FMT, int RT, int XR, int U>
hipError_t launch_tile(const QgemmArgs& a, hipStream_t st) {
  const int64_t subs = static_cast<int64_t>(a.gpanel[a.gcount]) * (4 / RT);
  const dim3 grid(static_cast<unsigned>(subs), static_cast<unsigned>((a.M + 4 * XR - 1) / (4 * XR)));
  hipLaunchKernelGGL((fewrow_kernel<FMT, RT, XR, U, QgMode::kDense>), grid, dim3(fr::kWaves * 64), 0, st, a);
  return hipGetLastError();
}

// The tiles fewrow_plan() can choose, in its order of preference.  RT <= 2
// tiles exist with one and two steps in flight.
#define QM_FEWROW_TILES(X) X(1, 2) X(1, 4) X(2, 2) X(2, 4) X(4, 2) X(4, 4) X(4, 8)

template <int FMT>
hipError_t launch_fmt(const QgemmArgs& a, const FewrowPlan& f, hipStream_t st) {
#define QM_FR(RT, XR) \
  if (f.rt == RT && f.xr == XR) \
    return RT <= 2 && f.u == 2 ? launch_tile<FMT, RT, XR, RT <= 2 ? 2 : 1>(a, st) : launch_tile<FMT, RT, XR, 1>(a, st);
  QM_FEWROW_TILES(QM_FR)
#undef QM_FR
  return hipErrorInvalidConfiguration;
}

}  // namespace

// The first tile of the list whose grid fits one workgroup per CU: more rows
// per workgroup mean fewer reads of the activations and of the weights, fewer
// workgroups idle CUs.  Measured on MI355X (256 CUs, weights from HBM, us per
// call, old: the tiles of gemm_plan):
//   Q4 3072 -> 2 x 8192: m = 8 14.4 -> 8.2, 16 14.9 -> 8.7, 32 15.3 -> 11.3
//   (256 panels: RT = 4; RT = 2 takes 8.9 / 10.4 / 13.7);
//   Q4 2048 -> 3072 wide: m = 8 7.3 -> 4.1, 32 7.7 -> 5.0, 77 7.9 -> 5.7
//   (RT = 1 / 2 / 4; two rounds of a smaller tile take 4.6 / 5.6 / 6.5);
//   Q4 8192 -> 3072: m = 8 17.4 -> 7.8, 64 18.8 -> 14.3.
// Where it loses, from a sweep over all formats: RT = 4 with fewer than 3/4
// workgroup per CU (dequantisation is the bound there and CUs idle; Q8 at
// m = 17, n = 4785: 12.5 vs 14.0), beyond 128 rows (Q4 1344 -> 1577 at m = 307:
// 7.9 vs 8.6), XR = 8 at long K (Q4 8192 -> 3072 at m = 128: 17.3 vs 18.1) and
// for Q8, F16 and BF16, whose weight registers are twice as many or more (F16
// 2048 -> 3072 at m = 64: 8.0 vs 8.8).  RT = 1 and 2 need no such line: few
// panels leave most of the chip idle whatever the tile, so they win as far as
// their grid fits, up to 2,048 rows of one panel (312 shapes of 256 and more rows
// in all formats: 1.14 to 2.4 x; Q4 2048 -> 64 at m = 1,024 3.8 vs 7.2, 8192 -> 64
// 12.8 vs 15.9, 2048 -> 256 at m = 512 4.6 vs 7.3).  Matrices with more panels
// than CUs take whole panels up to 16 rows, and up to 32 from K = 1024: with
// fewer K steps than wavefronts XR = 8 loses (K = 512, m = 24: 65,536 columns Q4
// 15.9 vs 15.5, Q8 18.3 vs 17.1, 151,936 34 vs 31 and 39 vs 33).  Two steps in
// flight help from K = 4096 (8192 -> 3072 at m = 8: 9.2 -> 7.8) and cost up to 6%
// at K = 1024.
FewrowPlan fewrow_plan(int32_t fmt, int64_t m, int64_t n, int64_t k, int cu_count) {
  // Tuning sweeps only: QM_FEWROW_PLAN="rt,xr,u" forces the plan (rt = 0: none).
  if (const char* e = tuning_override("QM_FEWROW_PLAN")) {
    FewrowPlan f{0, 0, 1};
    std::sscanf(e, "%d,%d,%d", &f.rt, &f.xr, &f.u);
    return f;
  }
  if (!fewrow_addressable(m, k)) return FewrowPlan{0, 0, 1};
  const int64_t panels = padded_rows(n) / kPanel;
  const bool wide = fmt_bits(fmt) >= 8;
  auto take = [&](int rt, int xr) {
    const int64_t groups = panels * (4 / rt) * ((m + 4 * xr - 1) / (4 * xr));
    if (groups > cu_count) return false;
    if (rt < 4 || m <= 16 || (m <= 32 && !wide)) return true;
    if (m > 128 || 4 * groups < 3 * cu_count) return false;
    return m <= 32 || (!fmt_float(fmt) && (xr < 8 || (!wide && k <= 4096)));
  };
#define QM_FR(RT, XR) \
  if (take(RT, XR)) return FewrowPlan{RT, XR, RT <= 2 && k >= 4096 ? 2 : 1};
  QM_FEWROW_TILES(QM_FR)
#undef QM_FR
  if (m <= (k >= 1024 ? 32 : 16) && panels > cu_count && fewrow_launchable(panels))
    return FewrowPlan{4, m <= 8 ? 2 : m <= 16 ? 4 : 8, 1};
  return FewrowPlan{0, 0, 1};
}

// kSwiglu on the few-row kernel (a.q / a.q2: gate / up).
#define QM_FEWROW_SWIGLU_TILES(X) X(1, 4) X(2, 4) X(2, 8)

// Every workgroup covers its rows of both matrices.  As in fewrow_plan, the
// first tile whose grid fits one workgroup per CU (Q4 2048 -> 2 x 8192: m = 16
// 9.3 -> 6.9 us against the grouped call and the elementwise kernel, 32 11.3 ->
// 8.5).  Wider matrices keep up to 16 rows on 16-row blocks (Q5 and Q6 with one
// weight tile, their registers leave no room for two: 3584 -> 2 x 18944 at m = 8
// Q6 25.6 vs 30.2) and up to 32 on 32-row blocks (there, Q4, us, few-row / two
// calls / GEMM tile: m = 8 19.5 / 20.9 / 35.6, 32 27.5 / 32.3 / 36.5; Q8 27.7 /
// 29.4 / 47.6, 38.9 / 42.3 / 48.6).  More rows: up to two 32-row blocks per CU
// where the single-panel GEMM tiles do not run (4096 -> 2 x 3072 at m = 160 Q4 20.5,
// 64 x 128 tile 23.4) or K is short (1024 -> 2 x 3072 at m = 96 Q4 8.0, tile 9.2; 2048
// -> 2 x 5632 at m = 48, 1.4 per CU, 12.6 / 13.0, Q6 16.8 / 16.4; 2 per CU at 2048 ->
// 2 x 8192 13.8 / 13.6 and 18.7 / 15.9), but not for Q8 and the float formats (2048 ->
// 2 x 8192 Q8 17.8, tile 14.1).
FewrowPlan fewrow_swiglu_plan(int32_t fmt, int64_t m, int64_t n, int64_t k, int cu_count) {
  if (!fewrow_addressable(m, k)) return FewrowPlan{0, 0, 1};
  const int64_t panels = padded_rows(n) / kPanel;
  auto groups = [&](int rt, int xr) { return panels * (4 / rt) * ((m + 4 * xr - 1) / (4 * xr)); };
#define QM_FR(RT, XR) \
  if (groups(RT, XR) <= cu_count) return FewrowPlan{RT, XR, 1};
  QM_FEWROW_SWIGLU_TILES(QM_FR)
#undef QM_FR
  const FewrowPlan wide = m > 16 ? FewrowPlan{2, 8, 1} : FewrowPlan{fmt == QM_Q5_G32 || fmt == QM_Q6_G32 ? 1 : 2, 4, 1};
  const int64_t g = groups(wide.rt, wide.xr);
  if (m <= 32 && fewrow_launchable(g)) return wide;
  const bool pair_tile = 2 * panels * ((m + 63) / 64) <= cu_count;       // as launch_gemm_swiglu
  if (m > 32 && fmt_bits(fmt) < 8 && g <= 2 * cu_count &&
      (!pair_tile || k <= 1024 || (k <= 2048 && 2 * g <= 3 * cu_count)))
    return wide;
  return FewrowPlan{0, 0, 1};
}

hipError_t launch_fewrow_swiglu(const QgemmArgs& a, int32_t fmt, const FewrowPlan& f, hipStream_t st) {
  auto go = [&](auto ft) -> hipError_t {
    constexpr int FMT = decltype(ft)::value;
    const unsigned panels = static_cast<unsigned>(padded_rows(a.N) / kPanel);
#define QM_FR(RT, XR)                                                                                             \
  if (f.rt == RT && f.xr == XR) {                                                                                 \
    hipLaunchKernelGGL((fewrow_kernel<FMT, RT, XR, 1, QgMode::kSwiglu>),                                          \
                       dim3(panels * (4 / RT), static_cast<unsigned>((a.M + 4 * XR - 1) / (4 * XR))),             \
                       dim3(fr::kWaves * 64), 0, st, a);                                                          \
    return hipGetLastError();                                                                                     \
  }
    QM_FEWROW_SWIGLU_TILES(QM_FR)
#undef QM_FR
    return hipErrorInvalidConfiguration;
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

hipError_t launch_fewrow(const QgemmArgs& a, int32_t fmt, const FewrowPlan& f, hipStream_t st) {
  switch (fmt) {
    case QM_Q4_G32: return launch_fmt<QM_Q4_G32>(a, f, st);
    case QM_Q8_G32: return launch_fmt<QM_Q8_G32>(a, f, st);
    case QM_Q2_G32: return launch_fmt<QM_Q2_G32>(a, f, st);
    case QM_Q3_G32: return launch_fmt<QM_Q3_G32>(a, f, st);
    case QM_Q5_G32: return launch_fmt<QM_Q5_G32>(a, f, st);
    case QM_Q6_G32: return launch_fmt<QM_Q6_G32>(a, f, st);
    case QM_F16: return launch_fmt<QM_F16>(a, f, st);
    case QM_BF16: return launch_fmt<QM_BF16>(a, f, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace qm
