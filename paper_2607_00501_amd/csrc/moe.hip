// Mixture-of-experts path: top-k routing, stable counting-sort bucketing,
// two grouped Q4 MFMA GEMMs (gate+up with a fused SwiGLU epilogue, then
// down with the gate weight folded in) and a deterministic combine.
//
// BaseRT runs MoE models (Sec. 4.1: Qwen3-30B-A3B, Gemma-4-26B-A4B) and
// reports its largest prefill margins there (Sec. 4.3); the kernels follow
// its fusion principle (Sec. 3.3: each fused step saves a launch and a
// global-memory round trip).  Everything is enqueued on one stream with no
// host round trip: per-expert row counts stay on the device, and each GEMM
// workgroup finds its (expert, row tile) from the counts itself.
#include <hip/hip_fp16.h>

#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <array>
#include <mutex>
#include <utility>

#include "fewrow.h"

namespace qm {
namespace {

// ------------------------------------------------------------------ route

constexpr int kRouteThreads = 256;   // one wavefront per token

// (value, index) order used by the router: larger value first, lower index
// on equal values.
__device__ inline void take_better(float& bv, int& be, float ov, int oe) {
  const bool better = ov > bv || (ov == bv && oe < be);
  bv = better ? ov : bv;
  be = better ? oe : be;
}

template <int CTRL>
__device__ inline void dpp_step(float& bv, int& be) {
  const float ov = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, bv), CTRL, 0xF, 0xF, false));
  const int oe = __builtin_amdgcn_mov_dpp(be, CTRL, 0xF, 0xF, false);
  take_better(bv, be, ov, oe);
}

// Every lane ends with the wavefront's best (value, index): DPP exchanges
// within each row of 16 lanes, then cross-row lane swaps between adjacent
// rows and between the two halves.
__device__ inline void wave_argmax(float& bv, int& be) {
  dpp_step<0xB1>(bv, be);    // quad_perm [1,0,3,2]
  dpp_step<0x4E>(bv, be);    // quad_perm [2,3,0,1]
  dpp_step<0x124>(bv, be);   // row_ror:4
  dpp_step<0x128>(bv, be);   // row_ror:8
  // Every lane now holds its 16-lane row's best.  v_permlane16_swap of a
  // value with itself gives each lane the pair {its row's, the adjacent
  // row's}; v_permlane32_swap the same across the two halves.  The order is
  // symmetric, so the better of each pair is the same in every lane.
  {
    const auto v = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, bv), __builtin_bit_cast(int, bv), false, false);
    const auto e = __builtin_amdgcn_permlane16_swap(be, be, false, false);
    bv = __builtin_bit_cast(float, static_cast<int>(v[0]));
    be = static_cast<int>(e[0]);
    take_better(bv, be, __builtin_bit_cast(float, static_cast<int>(v[1])), static_cast<int>(e[1]));
  }
  {
    const auto v = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(int, bv), __builtin_bit_cast(int, bv), false, false);
    const auto e = __builtin_amdgcn_permlane32_swap(be, be, false, false);
    bv = __builtin_bit_cast(float, static_cast<int>(v[0]));
    be = static_cast<int>(e[0]);
    take_better(bv, be, __builtin_bit_cast(float, static_cast<int>(v[1])), static_cast<int>(e[1]));
  }
}

// PER = logits per lane (n_experts <= 64 * PER), a power of two.
template <int PER>
__global__ __launch_bounds__(kRouteThreads) void route_kernel(const float* __restrict__ logits,
                                                              int64_t m, int E, int K,
                                                              int32_t* __restrict__ ids,
                                                              float* __restrict__ gates) {
  const int lane = threadIdx.x & 63;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * (kRouteThreads / 64) + (threadIdx.x >> 6);
  if (t >= m) return;
  const float* row = logits + t * E;
  float v[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = i * 64 + lane;
    v[i] = e < E ? row[e] : -INFINITY;
  }
  uint32_t taken = 0;         // bit i: item i of this lane already selected
  float my_v = -INFINITY;     // lane j < K ends up holding the j-th selected logit
  int my_e = 0;
  for (int j = 0; j < K; ++j) {
    // Lane-local best: highest value, lowest expert index on ties.
    float bv = -INFINITY;
    int be = 0x7FFFFFFF;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int e = i * 64 + lane;
      const bool ok = e < E && !((taken >> i) & 1u);
      const bool better = ok && (v[i] > bv || (v[i] == bv && e < be));
      bv = better ? v[i] : bv;
      be = better ? e : be;
    }
    // Wavefront argmax with the same order.
    wave_argmax(bv, be);
    if (lane == j) { my_v = bv; my_e = be; }
    if ((be & 63) == lane) taken |= 1u << (be >> 6);
  }
  // Softmax over the selected logits, relative to the largest (slot 0);
  // the denominator is a fixed-order butterfly sum over the lanes.
  const float vmax = __shfl(my_v, 0);
  const float ex = lane < K ? expf(my_v - vmax) : 0.0f;
  float denom = ex;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) denom += __shfl_xor(denom, off);
  if (lane < K) {
    ids[t * K + lane] = my_e;
    gates[t * K + lane] = ex / denom;
  }
}

// ----------------------------------------------------------------- bucket

constexpr int kBucketThreads = 1024;
constexpr int kBucketWaves = kBucketThreads / 64;
constexpr int kBucketUnroll = 8;
// Workgroups: each scatters a contiguous slice of about kBucketSlice
// assignments (two groups of 64 per wavefront), at most kBucketMaxGroups.
constexpr int64_t kBucketSlice = 2048;
constexpr int kBucketMaxGroups = 16;

// Lanes of the wavefront that hold the same expert id (one ballot per bit of
// the id, `bits` = bits needed for n_experts - 1), restricted to the valid
// lanes.
__device__ inline uint64_t match_expert(int e, bool valid, int bits) {
  uint64_t mask = __ballot(valid);
  for (int bit = 0; bit < bits; ++bit) {
    const bool set = (e >> bit) & 1;
    const uint64_t b = __ballot(valid && set);
    mask &= set ? b : ~b;
  }
  return mask;
}

// G workgroups of 16 wavefronts; workgroup g owns the contiguous slice
// [g*S, (g+1)*S) of the assignments and wavefront w of it the contiguous
// part [w*R, (w+1)*R) of that slice.  Pass 1: every workgroup counts all
// assignments per expert, its own per wavefront and the others split into
// those before and after its slice (LDS integer atomics: the counts do not
// depend on the order of the adds).  One pass over the experts then turns
// them into the expert offsets (written by workgroup 0 with the counts) and
// each wavefront's exclusive base: expert offset + assignments of the
// expert before the slice + those of earlier wavefronts in the slice.
// Pass 2 walks the wavefront's part again and places each assignment at
// base + rank among equal experts of its group of 64 lanes, the group's
// leader advancing the base.  The result is the stable counting sort by
// (expert, assignment id), the same for any G.  Groups past the end of a
// range are skipped (wavefront-uniform test).
__global__ __launch_bounds__(kBucketThreads) void bucket_kernel(const int32_t* __restrict__ ids,
                                                                int64_t A, int E,
                                                                int32_t* __restrict__ counts,
                                                                int32_t* __restrict__ offsets,
                                                                int32_t* __restrict__ sorted_assign) {
  __shared__ int base[kBucketWaves][1024];   // per-wavefront counts, then bases
  __shared__ int before[1024], after[1024];  // assignments outside the slice
  __shared__ int wsum[kBucketWaves];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  int bits = 0;
  while ((1 << bits) < E) ++bits;
  for (int w = 0; w < kBucketWaves; ++w) base[w][tid] = 0;
  before[tid] = 0;
  after[tid] = 0;
  __syncthreads();
  const int64_t S = (A + gridDim.x - 1) / gridDim.x;
  const int64_t slo = min<int64_t>(A, blockIdx.x * S), shi = min<int64_t>(A, slo + S);
  const int64_t R = ((shi - slo + kBucketWaves - 1) / kBucketWaves + 63) / 64 * 64;
  const int64_t lo = min<int64_t>(shi, slo + wave * R), hi = min<int64_t>(shi, lo + R);
  const uint64_t lower = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  // kBucketUnroll groups of 64 per round: all their id loads are issued first.
  for (int64_t b0 = lo; b0 < hi; b0 += 64 * kBucketUnroll) {
    int ev[kBucketUnroll];
#pragma unroll
    for (int u = 0; u < kBucketUnroll; ++u) {
      const int64_t a = b0 + u * 64 + lane;
      ev[u] = a < hi ? ids[a] : 0;
    }
#pragma unroll
    for (int u = 0; u < kBucketUnroll; ++u)
      if (b0 + u * 64 + lane < hi) atomicAdd(&base[wave][ev[u]], 1);
  }
  // The assignments outside the slice, strided over all threads.
  auto count_range = [&](int64_t rlo, int64_t rhi, int* dst) {
    for (int64_t b0 = rlo; b0 < rhi; b0 += static_cast<int64_t>(kBucketThreads) * kBucketUnroll) {
      int ev[kBucketUnroll];
#pragma unroll
      for (int u = 0; u < kBucketUnroll; ++u) {
        const int64_t a = b0 + u * kBucketThreads + tid;
        ev[u] = a < rhi ? ids[a] : 0;
      }
#pragma unroll
      for (int u = 0; u < kBucketUnroll; ++u)
        if (b0 + u * kBucketThreads + tid < rhi) atomicAdd(&dst[ev[u]], 1);
    }
  };
  count_range(0, slo, before);
  count_range(shi, A, after);
  __syncthreads();
  // Thread e: total count, per-wavefront exclusive prefix inside the slice;
  // then the exclusive scan of the totals over experts.
  const int e = tid;
  int total = before[e] + after[e];
  for (int w = 0; w < kBucketWaves; ++w) {
    const int c = base[w][e];
    base[w][e] = total - after[e];           // before[e] + earlier wavefronts
    total += c;
  }
  int incl = total;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d);
    if (lane >= d) incl += o;
  }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int off = incl - total;
  for (int w = 0; w < wave; ++w) off += wsum[w];
  for (int w = 0; w < kBucketWaves; ++w) base[w][e] += off;
  if (blockIdx.x == 0 && e < E) {
    counts[e] = total;
    offsets[e] = off;
  }
  if (blockIdx.x == 0 && e == 0) offsets[E] = static_cast<int32_t>(A);
  __syncthreads();
  for (int64_t b0 = lo; b0 < hi; b0 += 64 * kBucketUnroll) {
    int ev[kBucketUnroll];
#pragma unroll
    for (int u = 0; u < kBucketUnroll; ++u) {
      const int64_t a = b0 + u * 64 + lane;
      ev[u] = a < hi ? ids[a] : 0;
    }
#pragma unroll
    for (int u = 0; u < kBucketUnroll; ++u) {
      if (b0 + u * 64 >= hi) break;                      // wavefront-uniform
      const int64_t a = b0 + u * 64 + lane;
      const bool valid = a < hi;
      const uint64_t mask = match_expert(ev[u], valid, bits);
      const int rank = __popcll(mask & lower);
      if (valid) sorted_assign[base[wave][ev[u]] + rank] = static_cast<int32_t>(a);
      // every lane read its base before the leader advances it (same
      // wavefront, program order); the update is visible to the next group
      if (valid && rank == 0) base[wave][ev[u]] += __popcll(mask);
    }
  }
}

// ------------------------------------------- routing of a decode batch

// A few tokens (m rounded-up E <= 2048 logits, m top_k <= 128 assignments):
// routing and bucketing in one workgroup and one launch.  Both kernels above
// are chains of dependent steps (top_k wavefront argmaxes; counts, scan,
// ballots) on a few wavefronts; here every order statistic is a count, taken
// in parallel by the 1024 threads: the slot of an expert is the number of
// experts that go before it, the place of an assignment the number of
// assignments that go before it, an expert's offset the number of assignments
// to lower experts.  128 experts, top-8: 10.4 -> 4.2 us at one token, 11.0 ->
// 8.6 at 8; 64 experts, top-6: 9.7 -> 7.7 at 16.
constexpr int kSmallRouteLogits = 2048;
constexpr int kSmallRouteAssign = 128;
__host__ __device__ constexpr int small_route_log_stride(int E) { return E <= 64 ? 6 : E <= 128 ? 7 : 8; }
// The compares are m E^2; about 10 tokens of 128 experts is where the two
// launches above catch up.
inline bool small_route(int64_t m, int32_t e, int32_t k) {
  const int64_t s = 1 << small_route_log_stride(e);
  return m > 0 && e <= 256 && m * s <= kSmallRouteLogits && m * s * s <= 10 * 128 * 128 && m * k <= kSmallRouteAssign;
}

// Floats as integers of the same order, -0 as +0, NaN as 1 (below every
// number) and above the padding's 0.
__device__ __forceinline__ uint32_t order_key(float v) {
  if (v != v) return 1u;
  const uint32_t b = __builtin_bit_cast(uint32_t, v + 0.0f);
  return b & 0x80000000u ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float order_value(uint32_t k) {
  if (k == 1u) return __builtin_nanf("");
  return __builtin_bit_cast(float, k & 0x80000000u ? k & 0x7FFFFFFFu : ~k);
}

__global__ __launch_bounds__(1024) void route_small_kernel(const float* __restrict__ logits, int m, int E, int K,
                                                           int32_t* __restrict__ ids, float* __restrict__ gates,
                                                           int32_t* __restrict__ counts,
                                                           int32_t* __restrict__ offsets,
                                                           int32_t* __restrict__ sorted_assign) {
  __shared__ __attribute__((aligned(16))) uint32_t key[kSmallRouteLogits];      // rows of 2^ls, padded with 0
  __shared__ __attribute__((aligned(16))) int32_t sel_id[kSmallRouteAssign];    // padded with INT32_MAX
  __shared__ float sel_v[kSmallRouteAssign];
  const int tid = threadIdx.x;
  const int ls = small_route_log_stride(E), S = 1 << ls, A = m * K;
  for (int i = tid; i < m << ls; i += 1024) {
    const int t = i >> ls, e = i & (S - 1);
    key[i] = e < E ? order_key(logits[t * E + e]) : 0u;
  }
  if (tid < kSmallRouteAssign) sel_id[tid] = 0x7FFFFFFF;
  __syncthreads();
  // Slot of expert e among its token's: 2^lp threads a pair, each over a share
  // of the experts, four at a time.  An equal logit goes first if its index is
  // lower: below e's own four the test is key > ke - 1, from there on
  // key > ke, and equals inside the four are added at the end.
  int lp = 0;
  while (lp < 4 && m << (ls + lp + 1) <= 1024) ++lp;
  for (int it = tid; it < m << (ls + lp); it += 1024) {   // 64-lane groups stay whole
    const int pair = it >> lp, part = it & ((1 << lp) - 1);
    const int t = pair >> ls, e = pair & (S - 1);
    const uint4* row = reinterpret_cast<const uint4*>(key + (t << ls));
    const uint32_t ke = key[pair];
    const int e4 = e >> 2;
    int rank = 0;
#pragma unroll 4
    for (int o = part; o < S / 4; o += 1 << lp) {
      const uint4 ko = row[o];
      const uint32_t kk = o < e4 ? ke - 1u : ke;          // (padding: ke = 0, its rank is not used)
      rank += (ko.x > kk) + (ko.y > kk) + (ko.z > kk) + (ko.w > kk);
    }
    for (int off = 1; off < 1 << lp; off <<= 1) rank += __shfl_xor(rank, off);
    const uint4 own = row[e4];
    rank += ((e & 3) > 0 && own.x == ke) + ((e & 3) > 1 && own.y == ke) + ((e & 3) > 2 && own.z == ke);
    if (part == 0 && e < E && rank < K) {
      sel_id[t * K + rank] = e;
      sel_v[t * K + rank] = order_value(ke);
    }
  }
  __syncthreads();
  const int4* id4 = reinterpret_cast<const int4*>(sel_id);
  if (tid < E) {
    // Expert tid: its assignments and those of lower experts.
    int c = 0, lower = 0;
    for (int b = 0; b < A; b += 4) {
      const int4 v = id4[b / 4];
      c += (v.x == tid) + (v.y == tid) + (v.z == tid) + (v.w == tid);
      lower += (v.x < tid) + (v.y < tid) + (v.z < tid) + (v.w < tid);
    }
    counts[tid] = c;
    offsets[tid] = lower;
    if (tid == 0) offsets[E] = A;
  }
  const int a = tid - 512;                                // other wavefronts: assignment a
  if (a >= 0 && a < A) {
    const int id = sel_id[a];
    int pos = 0;
    for (int b = 0; b < A; b += 4) {
      const int4 v = id4[b / 4];
      pos += v.x < id || (v.x == id && b < a) ? 1 : 0;
      pos += v.y < id || (v.y == id && b + 1 < a) ? 1 : 0;
      pos += v.z < id || (v.z == id && b + 2 < a) ? 1 : 0;
      pos += v.w < id || (v.w == id && b + 3 < a) ? 1 : 0;
    }
    sorted_assign[pos] = a;
    // Softmax over the token's selected logits relative to the largest, the
    // denominator in the pairwise order of route_kernel's butterfly.
    const int s0 = a / K * K;
    const float vmax = sel_v[s0];
    float ex[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) ex[j] = j < K ? expf(sel_v[s0 + min(j, K - 1)] - vmax) : 0.0f;
#pragma unroll
    for (int w = 1; w < 16; w <<= 1)
#pragma unroll
      for (int j = 0; j < 16; j += 2 * w) ex[j] += ex[j + w];
    ids[a] = id;
    gates[a] = expf(sel_v[a] - vmax) / ex[0];
  }
}

// ---------------------------------------------------------------- combine

// y[t][n] = sum over slots j (in order) of the gate-weighted expert outputs
// (fp16 in the workspace, summed in fp32).  One thread per 8 outputs.
__global__ __launch_bounds__(256) void combine_kernel(const uint16_t* __restrict__ yp, float* __restrict__ y,
                                                      int64_t m, int64_t hidden, int K) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;   // 8-output index
  const int64_t h8 = hidden / 8;
  if (i >= m * h8) return;
  const int64_t t = i / h8, c = i % h8;
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // Slots in batches of 8: all loads of a batch are in flight before the
  // first add (Yp is read once: nontemporal); the adds keep slot order.
  for (int j0 = 0; j0 < K; j0 += 8) {
    half8v v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < K)
        v[u] = __builtin_nontemporal_load(reinterpret_cast<const half8v*>(yp + (t * K + j0 + u) * hidden) + c);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < K)
#pragma unroll
        for (int r = 0; r < 8; ++r) s[r] += static_cast<float>(v[u][r]);
  }
  float4* dst = reinterpret_cast<float4*>(y + t * hidden) + 2 * c;
  dst[0] = make_float4(s[0], s[1], s[2], s[3]);
  dst[1] = make_float4(s[4], s[5], s[6], s[7]);
}

hipError_t launch_combine(const MoeArgs& a, hipStream_t st) {
  const int64_t n8 = a.m * (a.hidden / 8);
  hipLaunchKernelGGL(combine_kernel, dim3(static_cast<unsigned>((n8 + 255) / 256)), dim3(256), 0, st, a.yp,
                     a.y, a.m, a.hidden, a.top_k);
  return hipGetLastError();
}

template <int BMG, int WKG, int BMD, int WKD, int WNG, int DG = 2, int DD = 2, bool NT = false, int FMT = QM_Q4_G32,
          int WND = WNG>
hipError_t launch_moe_tiles(const MoeArgs& a, hipStream_t st) {
  const int64_t A = a.m * a.top_k;
  // Upper bound on the number of (expert, row tile) pairs: sum of
  // ceil(count_e / BM) <= A / BM + E.  Workgroups past the last tile exit.
  auto tiles = [&](int bm) { return static_cast<unsigned>((A + bm - 1) / bm + a.n_experts); };
  QgemmArgs g{};
  g.counts = a.counts; g.offsets = a.offsets; g.sorted_assign = a.sorted_assign; g.topk_w = a.topk_w;
  g.topk_ids = a.topk_ids;
  g.n_experts = a.n_experts; g.top_k = a.top_k; g.M = A;
  // gate/up + SwiGLU: A = x rows gathered per assignment, N = inter, K = hidden
  g.q = a.gq; g.s = a.gs; g.q2 = a.uq; g.s2 = a.us; g.a = a.x; g.h = a.h; g.N = a.inter; g.K = a.hidden;
  // 1-D grids over (row tile, column block) units, rounded up to whole
  // rounds of XCD chunks (the XCD mapping is done in the kernel).
  auto grid = [&](int bm, int wn, int64_t n) {
    const int64_t ny = (padded_rows(n) + 64 * wn - 1) / (64 * wn);
    const int64_t round = static_cast<int64_t>(kXcds) * qg::kMoeChunkTiles * ny;
    const int64_t units = static_cast<int64_t>(tiles(bm)) * ny;
    return dim3(static_cast<unsigned>((units + round - 1) / round * round));
  };
  g.tiles = tiles(BMG);
  hipLaunchKernelGGL((qgemm_kernel<BMG, WNG, WKG, QgMode::kMoeGateUp, DG, NT, FMT>), grid(BMG, WNG, a.inter),
                     dim3(WNG * WKG * 64), 0, st, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // down, scaled by the gate weight and scattered to the assignment slot
  g.q = a.dq; g.s = a.ds; g.q2 = nullptr; g.s2 = nullptr; g.a = a.h; g.yp = a.yp; g.N = a.hidden; g.K = a.inter;
  g.tiles = tiles(BMD);
  hipLaunchKernelGGL((qgemm_kernel<BMD, WND, WKD, QgMode::kMoeDown, DD, NT, FMT>), grid(BMD, WND, a.hidden),
                     dim3(WND * WKD * 64), 0, st, g);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_combine(a, st);
}

// The two grouped products on the few-row kernel: RTG / RTD 16-row weight tiles
// and 4 XR bucket rows per workgroup.
template <int RTG, int RTD, int XR, int FMT>
hipError_t launch_moe_fewrow(const MoeArgs& a, hipStream_t st) {
  const int64_t A = a.m * a.top_k;
  QgemmArgs g{};
  g.counts = a.counts; g.offsets = a.offsets; g.sorted_assign = a.sorted_assign; g.topk_w = a.topk_w;
  g.topk_ids = a.topk_ids;
  g.n_experts = a.n_experts; g.top_k = a.top_k; g.M = A;
  // At most one (expert, row block) pair per assignment.
  g.tiles = std::min<int64_t>(A, (A + 4 * XR - 1) / (4 * XR) + a.n_experts);
  auto grid = [&](int rt, int64_t n) {
    const int64_t sp = 4 / rt, round = kXcds * sp;
    const int64_t units = g.tiles * (padded_rows(n) / kPanel) * sp;
    return dim3(static_cast<unsigned>((units + round - 1) / round * round));
  };
  g.q = a.gq; g.s = a.gs; g.q2 = a.uq; g.s2 = a.us; g.a = a.x; g.h = a.h; g.N = a.inter; g.K = a.hidden;
  hipLaunchKernelGGL((fewrow_kernel<FMT, RTG, XR, 1, QgMode::kMoeGateUp>), grid(RTG, a.inter), dim3(fr::kWaves * 64),
                     0, st, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  g.q = a.dq; g.s = a.ds; g.q2 = nullptr; g.s2 = nullptr; g.a = a.h; g.yp = a.yp; g.N = a.hidden; g.K = a.inter;
  hipLaunchKernelGGL((fewrow_kernel<FMT, RTD, XR, 1, QgMode::kMoeDown>), grid(RTD, a.hidden), dim3(fr::kWaves * 64),
                     0, st, g);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_combine(a, st);
}

}  // namespace

// Scratch of the allocation-free MoE entry point: h and the per-assignment
// outputs of one call, kMoeScratchBytes per device, held by every device the
// library runs on until the process ends.  In host code `scratch` names a
// host-side stand-in, never the device memory: its device address is looked
// up once per device (hipGetSymbolAddress, with that device current) and
// only that address is handed to kernels.  Every call on a device shares the
// same bytes, so calls that overlap on one device race.
static __device__ __align__(256) uint8_t scratch[kMoeScratchBytes];

namespace {
constexpr int kScratchDevices = 64;
void* g_scratch_ptr[kScratchDevices];
hipError_t g_scratch_status[kScratchDevices];
std::once_flag g_scratch_once[kScratchDevices];
}  // namespace

hipError_t moe_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kScratchDevices) return hipErrorInvalidDevice;
  std::call_once(g_scratch_once[dev], [dev]() {
    void* p = nullptr;
    g_scratch_status[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = g_scratch_status[dev] == hipSuccess ? p : nullptr;
  });
  if (g_scratch_status[dev] != hipSuccess) return g_scratch_status[dev];
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

size_t moe_workspace_bytes(int64_t m, int32_t top_k, int64_t hidden, int64_t inter) {
  const size_t A = static_cast<size_t>(m) * top_k;
  const size_t h_bytes = (A * inter * 2 + 255) / 256 * 256;
  const size_t yp_bytes = (A * hidden * 2 + 255) / 256 * 256;
  return h_bytes + yp_bytes;
}

hipError_t launch_route(const float* logits, int64_t m, int32_t e, int32_t k, int32_t* ids, float* w,
                        int32_t* counts, int32_t* offsets, int32_t* sorted_assign, hipStream_t st) {
  if (small_route(m, e, k)) {
    hipLaunchKernelGGL(route_small_kernel, dim3(1), dim3(1024), 0, st, logits, static_cast<int>(m), e, k, ids, w,
                       counts, offsets, sorted_assign);
    return hipGetLastError();
  }
  if (m > 0) {
    const unsigned blocks = static_cast<unsigned>((m + 3) / 4);
    const dim3 g(blocks), b(kRouteThreads);
    if (e <= 64) hipLaunchKernelGGL(route_kernel<1>, g, b, 0, st, logits, m, e, k, ids, w);
    else if (e <= 128) hipLaunchKernelGGL(route_kernel<2>, g, b, 0, st, logits, m, e, k, ids, w);
    else if (e <= 256) hipLaunchKernelGGL(route_kernel<4>, g, b, 0, st, logits, m, e, k, ids, w);
    else if (e <= 512) hipLaunchKernelGGL(route_kernel<8>, g, b, 0, st, logits, m, e, k, ids, w);
    else hipLaunchKernelGGL(route_kernel<16>, g, b, 0, st, logits, m, e, k, ids, w);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  const int64_t A = m * k;
  const unsigned groups = static_cast<unsigned>(
      std::min<int64_t>(kBucketMaxGroups, std::max<int64_t>(1, (A + kBucketSlice - 1) / kBucketSlice)));
  hipLaunchKernelGGL(bucket_kernel, dim3(groups), dim3(kBucketThreads), 0, st, ids, A, e, counts, offsets,
                     sorted_assign);
  return hipGetLastError();
}

// Where the expert products take the few-row kernel: at most 1.5 rows per
// expert in the mean (decode batches); grids that can be launched (at most a row
// block per assignment, two sub-panels of a gate/up panel, one of a down panel,
// rounded up over the XCDs; such activations, x rows for gate/up and h rows for
// down, are fewrow_addressable, as A times hidden or inter is below 2^29); and
// not too many workgroups for the work in them.  A workgroup costs some time
// whatever its K (8 wavefronts share K / 128 steps, then add their sums): about
// A (2 inter + hidden) / 64 of them lose against the tiles, unless K is long
// enough that their faster products make up for it (inter x hidden / 550); on
// the other side the tiles launch E (inter + hidden) / 256 workgroups, most of
// them empty.  Fitted to 1,140 layers of 32 to 1,024 experts, 512 x 256 to 4096 x
// 1536, 1/8 to 1.5 rows per expert (us for the three launches, few-row / tiles):
// 256 experts, top-8, 1024 -> 512, 48 tokens Q4 74 / 55, Q8 110 / 76; 24 tokens
// 49 / 48 and 74 / 67, 8 tokens 28 / 27 and 37 / 34; 1,024, top-16, 512 -> 256, 96
// tokens 228 / 83 and 324 / 117, 8 tokens 43 / 59 and 46 / 72; 128, top-8, 2048 ->
// 768, 24 tokens 73 / 83 and 105 / 110.  The rule is within 1% of the better one
// in the mean, 25% at most (Q6, 512 experts, 1024 -> 512, 16 tokens: 73 / 58).
bool moe_few_rows(int32_t fmt, int64_t m, int32_t top_k, int64_t n_experts, int64_t hidden, int64_t inter,
                  int cu_count) {
  const int64_t A = m * top_k;
  if (2 * A > 3 * n_experts || !fewrow_launchable(A * (padded_rows(inter) / kPanel) * 2 + 2 * kXcds) ||
      !fewrow_launchable(A * (padded_rows(hidden) / kPanel) + kXcds))
    return false;
  const int64_t per_2cu = fmt == QM_Q8_G32 ? 11 : fmt == QM_Q4_G32 || fmt == QM_Q6_G32 ? 17 : 14;   // workgroups
  return A * (2 * inter + hidden - inter * hidden / 550) <=
         32 * per_2cu * cu_count + n_experts * (inter + hidden) / 32;
}

namespace {

// few: the few-row kernel; else 32-row tiles up to 24 rows per expert (rpe), with
// 2-panel blocks for gate/up and down where narrow_g and narrow_d say so.
struct MoePlan { bool few, narrow_g, narrow_d; int64_t rpe; };

MoePlan moe_plan(int32_t fmt, int64_t m, int32_t top_k, int64_t n_experts, int64_t hidden, int64_t inter,
                 int cu_count) {
  const int64_t used = std::min<int64_t>(n_experts, m * top_k);
  auto blocks = [&](int64_t n) { return used * ((padded_rows(n) + 255) / 256); };
  return MoePlan{moe_few_rows(fmt, m, top_k, n_experts, hidden, inter, cu_count), 2 * blocks(inter) <= cu_count,
                 4 * blocks(hidden) <= 3 * cu_count, m * top_k / n_experts};
}

constexpr bool gate_up_32_rows(int32_t fmt) { return fmt == QM_Q5_G32 || fmt == QM_Q6_G32 || fmt == QM_Q8_G32; }

}  // namespace

const char* moe_tile_name(int32_t fmt, int64_t m, int32_t top_k, int64_t n_experts, int64_t hidden, int64_t inter,
                          int cu_count) {
  static thread_local char buf[64];
  const MoePlan p = moe_plan(fmt, m, top_k, n_experts, hidden, inter, cu_count);
  if (p.few)
    std::snprintf(buf, sizeof(buf), "few-row, 8 rows x 32 and 64");
  else if (p.rpe <= 24)
    std::snprintf(buf, sizeof(buf), "32-row bucket tiles x %d and %d panels", p.narrow_g ? 2 : 4, p.narrow_d ? 2 : 4);
  else
    std::snprintf(buf, sizeof(buf), "%d- and 64-row bucket tiles x 4 panels", gate_up_32_rows(fmt) ? 32 : 64);
  return buf;
}

hipError_t launch_moe(const MoeArgs& a, int cu_count, hipStream_t st) {
  // Tuning sweeps only: QM_MOE_PLAN="bm_gate_up,wk_gate_up,bm_down,wk_down,
  // depth_gate_up,depth_down,nontemporal".
  static const std::array<int, 7> forced = [] {
    std::array<int, 7> f{0, 0, 0, 0, 2, 2, 0};
    if (const char* e = tuning_override("QM_MOE_PLAN"))
      std::sscanf(e, "%d,%d,%d,%d,%d,%d,%d", &f[0], &f[1], &f[2], &f[3], &f[4], &f[5], &f[6]);
    return f;
  }();
  using P = std::array<int, 7>;
  if (a.format == QM_Q4_G32) {
    if (forced == P{32, 1, 32, 1, 2, 2, 0}) return launch_moe_tiles<32, 1, 32, 1, 4, 2, 2>(a, st);
    if (forced == P{64, 1, 64, 1, 2, 2, 0}) return launch_moe_tiles<64, 1, 64, 1, 4, 2, 2>(a, st);
    if (forced == P{32, 1, 32, 1, 2, 2, 1}) return launch_moe_tiles<32, 1, 32, 1, 4, 2, 2, true>(a, st);
    if (forced == P{64, 1, 64, 1, 2, 2, 1}) return launch_moe_tiles<64, 1, 64, 1, 4, 2, 2, true>(a, st);
  }
  // Per-chip tile choice by rows per expert: 32-row tiles when buckets are
  // small (decode-like prefill chunks), 64-row tiles otherwise.  While an
  // expert's rows fit one row tile, each weight panel is read by exactly one
  // workgroup: nontemporal weight loads (measured on MI355X with cold caches:
  // 132 -> 102 us at 8 rows per expert, 157 -> 143 us at 32; with several
  // row tiles per expert they lose the L2 reuse between tiles).  Q2 and
  // Q3 use the Q4 plan.  Q5, Q6 and Q8 keep their weights in registers
  // (their LDS stages do not fit beside two workgroups' A stages), and the
  // two-matrix gate/up tile then holds 64 rows only by spilling: their
  // gate/up tiles stay at 32 rows.
  // Where moe_few_rows() holds: the few-row kernel with 32-row sub-panels for
  // gate/up, whole panels for down and 8-row blocks; the 32 x 256 tiles leave 24
  // workgroups busy at one token.
  // Measured on MI355X (128 experts, top-8, 2048 -> 768 -> 2048, Q4, us for the
  // three launches): 45.9 -> 18.3 at 1 token, 46.8 -> 32.0 at 4, 77.1 -> 61.8 at
  // 16, 86.7 -> 80.0 at 32, 90.8 -> 93.0 at 64; Q3 and Q5 turn at 1.5 rows per
  // expert (Q3 95.8 -> 89.2 at 1, 103.8 -> 113.5 at 2).
  // 32-row tiles of a product whose 4-panel column blocks would leave CUs without
  // a workgroup: 2-panel blocks with 2-way split-K, twice the
  // workgroups with half the chain of K steps.  The lines (us, products and
  // combine, before / after, at 48 tokens): 32 experts of 1536 -> 1024, top-4 (128
  // and 192 blocks) Q4 42.1 / 33.6, Q8 48.6 / 42.6; 32 of 1024 -> 512 30.7 / 23.5;
  // 128 of 1024 -> 256, top-8 (128 blocks, down 4-panel) Q4 32.1 / 27.9.  Narrow
  // gate/up at 160 blocks (32 of 2048 -> 1280): Q4 51.4 / 48.0 but Q8 62.0 / 65.7;
  // at 192 (64 of 2048 -> 768) Q4 52.9 / 54.9, Q8 65.3 / 73.7.
  const auto [few, narrow_g, narrow_d, rpe] =
      moe_plan(a.format, a.m, a.top_k, a.n_experts, a.hidden, a.inter, cu_count);
  auto plan = [&, few = few, narrow_g = narrow_g, narrow_d = narrow_d, rpe = rpe](auto f) -> hipError_t {
    constexpr int F = decltype(f)::value;
    if (few) return launch_moe_fewrow<2, 4, 2, F>(a, st);
    if (rpe <= 24) {
      if (narrow_g && narrow_d) return launch_moe_tiles<32, 2, 32, 2, 2, 2, 2, true, F, 2>(a, st);
      if (narrow_g) return launch_moe_tiles<32, 2, 32, 1, 2, 2, 2, true, F, 4>(a, st);
      if (narrow_d) return launch_moe_tiles<32, 1, 32, 2, 4, 2, 2, true, F, 2>(a, st);
      return launch_moe_tiles<32, 1, 32, 1, 4, 2, 2, true, F, 4>(a, st);
    }
    if constexpr (gate_up_32_rows(F)) {
      return launch_moe_tiles<32, 1, 64, 1, 4, 2, 2, false, F>(a, st);
    } else {
      if (rpe <= 64) return launch_moe_tiles<64, 1, 64, 1, 4, 2, 2, true, F>(a, st);
      return launch_moe_tiles<64, 1, 64, 1, 4, 2, 2, false, F>(a, st);
    }
  };
  switch (a.format) {
    case QM_Q4_G32: return plan(std::integral_constant<int, QM_Q4_G32>{});
    case QM_Q8_G32: return plan(std::integral_constant<int, QM_Q8_G32>{});
    case QM_Q2_G32: return plan(std::integral_constant<int, QM_Q2_G32>{});
    case QM_Q3_G32: return plan(std::integral_constant<int, QM_Q3_G32>{});
    case QM_Q5_G32: return plan(std::integral_constant<int, QM_Q5_G32>{});
    case QM_Q6_G32: return plan(std::integral_constant<int, QM_Q6_G32>{});
    default: return hipErrorInvalidValue;   // F16 / BF16 experts are rejected by the API
  }
}

}  // namespace qm
