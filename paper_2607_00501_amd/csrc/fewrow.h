// Matrix product for few activation rows (a small decode batch, a short
// prompt, a small expert bucket): Y = A W'^T on v_mfma_f32_16x16x32_f16.
//
// What bounds it: the weights are read once, so it should run at the rate of
// the weight stream, like the GEMV; the 32- and 64-row MFMA tiles of qgemm.h
// spend a barrier, an LDS round trip and a mostly empty tile per 64-deep K
// step instead.  Mapping:
//  * a workgroup of 8 wavefronts owns 16 RT weight rows of one 64-row panel
//    (a sub-panel) and up to 4 XR activation rows; the wavefronts split K,
//    four groups (one per 16-lane quarter) at a time, and meet once, in LDS,
//    in a fixed order.  No barrier and no LDS access before that;
//  * the weights are the A operand.  Lane l loads the chunk of weight row
//    l%16, group 4t + l/16 (Q4: 16 bytes; a wavefront load covers four
//    contiguous 256-byte pieces) and dequantises it in registers to
//    fp16_RNE(s * q).  The 32-deep k block of MFMA j is relabelled (A and B
//    agree, so the sum is unchanged): quarter h covers k = 32 (4t + h) + 8j
//    .. + 7, so one chunk feeds four MFMAs with no cross-lane step;
//  * the activations are the B operand.  A wavefront loads its 128 k of the
//    rows coalesced (256 bytes of four rows per load) and turns them into
//    fragments through a 4 KiB LDS tile of its own, without a barrier (read
//    straight in fragment order, every load touches 32 cache lines instead of
//    8: Q4 3072 -> 2 x 8192 at m = 16 took 9.8 instead of 8.7 us, 32-row
//    workgroups 13.4 instead of 10.4).  A dequantised fragment is used for
//    all XR / 4 row tiles, an activation fragment for all RT weight tiles;
//  * the loads of U steps are issued before the first use.
// Up to 8 activation rows it runs at the rate of the weight stream plus the
// launch (28 MB in 8.2 us); with more, dequantisation binds: about 300 VALU
// instructions per 64 weight rows and 128 k, once per 4 XR activation rows.
#pragma once

#include <type_traits>

#include "chunk.h"
#include "qgemm.h"

namespace qm {
namespace fr {

constexpr int kWaves = 8;

// MFMA j's eight weights of a lane's chunk (k = 8j .. 8j + 7 of its group),
// as fp16: fp16_RNE(s * q), the stored F16, or BF16 converted to fp16.
template <int FMT, class DQ>
__device__ __forceinline__ half8v weight_frag(const uint32_t* d, int j, half2v s2, const DQ& c) {
  if constexpr (FMT == QM_F16) {
    return __builtin_bit_cast(half8v, u32x4{d[4 * j], d[4 * j + 1], d[4 * j + 2], d[4 * j + 3]});
  } else if constexpr (FMT == QM_BF16) {
    half8v o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = static_cast<_Float16>(__uint_as_float(d[4 * j + i] << 16));
      o[2 * i + 1] = static_cast<_Float16>(__uint_as_float(d[4 * j + i] & 0xFFFF0000u));
    }
    return o;
  } else if constexpr (FMT == QM_Q8_G32) {
    return qg::dequant_q8(d[2 * j], d[2 * j + 1], s2, c);
  } else if constexpr (FMT == QM_Q5_G32) {
    return qg::dequant_nib_hi<FMT>(d[j], d[4] >> (8 * (j >> 1)), j & 1, s2, c);
  } else if constexpr (FMT == QM_Q6_G32) {
    return qg::dequant_nib_hi<FMT>(d[j], d[4 + (j >> 1)], j & 1, s2, c);
  } else if constexpr (FMT == QM_Q2_G32) {
    return qg::dequant_crumb<FMT>(d[j >> 1], 0u, j & 1, s2, c);
  } else if constexpr (FMT == QM_Q3_G32) {
    return qg::dequant_crumb<FMT>(d[j >> 1], d[2] >> (8 * (j >> 1)), j & 1, s2, c);
  } else {
    return qg::dequant_dword(d[j], s2, c);
  }
}

// Two workgroups per CU (four wavefronts per SIMD, 128 VGPRs) where the
// registers allow: U steps of 4 XR activation and NM RT (W + 1) weight
// registers in flight, NM RT (16 fragment + 4 per row tile accumulator)
// ones, XR offsets.
constexpr bool two_matrices(QgMode mode) { return mode == QgMode::kMoeGateUp || mode == QgMode::kSwiglu; }
constexpr int waves_per_simd(int fmt, int rt, int xr, int u, int nm) {
  return u * (4 * xr + nm * rt * (fmt_bits(fmt) + 1)) + nm * rt * (16 + (xr + 3) / 4 * 4) + xr + 16 + 24 <= 128 ? 4 : 2;
}
template <int FMT, int RT, int XR, int U, QgMode MODE>
constexpr int kWavesPerSimd = waves_per_simd(FMT, RT, XR, U, two_matrices(MODE) ? 2 : 1);

template <int FMT, int RT, int XR, int U, QgMode MODE>
__device__ __forceinline__ void body(const QgemmArgs& p) {
  constexpr int NM = two_matrices(MODE) ? 2 : 1;
  constexpr int W = fmt_bits(FMT), CB = chunk_block_bytes(FMT);
  constexpr bool kFloat = fmt_float(FMT);
  constexpr int SP = 4 / RT;                              // sub-panels per panel
  constexpr int BR = 4 * XR;                              // activation rows per workgroup
  constexpr int MT = (XR + 3) / 4;                        // in 16-row tiles
  constexpr int TILES = RT * MT;
  // One 4 KiB activation tile per wavefront during the K loop, then the
  // partial sums.
  __shared__ float4v lds[kWaves * 64 * (NM * TILES > 4 ? NM * TILES : 4)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c = lane & 15, h = lane >> 4;
  const int64_t K = p.K;
  const int G = static_cast<int>(K / kGroup);

  // The workgroup's rows, matrix and sub-panel.
  int64_t row0, panel, mN = p.N;
  int rows, sub, expert = 0;
  const uint8_t* mq = p.q;
  const uint16_t* ms = p.s;
  float* my = p.y;
  if constexpr (MODE == QgMode::kDense) {
    row0 = static_cast<int64_t>(blockIdx.y) * BR;
    rows = static_cast<int>(min<int64_t>(BR, p.M - row0));
    // The sub-panels of a panel share the 128-byte lines of its scales: one XCD.
    xcd_group_member(blockIdx.x, p.gpanel[p.gcount], SP, &panel, &sub);
    const int gp = static_cast<int>(panel);
    mq = p.gq[0]; ms = p.gs[0]; my = p.gy[0]; mN = p.gn[0];
    int first = 0;
#pragma unroll
    for (int j = 1; j < kGemmGroupMax; ++j) {
      const bool in = j < p.gcount && gp >= p.gpanel[j];
      mq = in ? p.gq[j] : mq;
      ms = in ? p.gs[j] : ms;
      my = in ? p.gy[j] : my;
      mN = in ? p.gn[j] : mN;
      first = in ? p.gpanel[j] : first;
    }
    panel = gp - first;
  } else if constexpr (MODE == QgMode::kSwiglu) {
    row0 = static_cast<int64_t>(blockIdx.y) * BR;
    rows = static_cast<int>(min<int64_t>(BR, p.M - row0));
    xcd_group_member(blockIdx.x, padded_rows(mN) / kPanel, SP, &panel, &sub);
  } else {
    const int64_t ny = padded_rows(p.N) / kPanel * SP;
    const int64_t u = xcd_chunked(blockIdx.x, SP);
    if (u >= p.tiles * ny) return;                        // whole workgroup, before any barrier
    __shared__ int sh_e, sh_tile;
    qg::find_tile(p.counts, p.n_experts, BR, static_cast<int>(u / ny), &sh_e, &sh_tile);
    expert = __builtin_amdgcn_readfirstlane(sh_e);
    if (expert < 0) return;
    row0 = p.offsets[expert] + static_cast<int64_t>(__builtin_amdgcn_readfirstlane(sh_tile)) * BR;
    rows = static_cast<int>(min<int64_t>(BR, p.offsets[expert + 1] - row0));
    const int64_t sp = u % ny;
    panel = sp / SP;
    sub = static_cast<int>(sp % SP);
  }
  const uint8_t* wq[NM];
  const uint16_t* wsc[NM];
  const int64_t npanels = padded_rows(mN) / kPanel;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    wq[m] = (m == 0 ? mq : p.q2) + (expert * npanels + panel) * G * CB;
    wsc[m] = kFloat ? nullptr : (m == 0 ? ms : p.s2) + (expert * npanels + panel) * G * kPanel;
  }
  const int wrow = 16 * RT * sub + c;                     // weight row of tile 0 inside the panel
  // Activations: load i of a step takes rows 4i .. 4i + 3, 256 contiguous
  // bytes of each (16-byte piece lane % 16 of row 4i + lane / 16).  Offsets in
  // 16-byte units, 32 bits (the plans check fewrow_addressable).
  const u32x4* xbase = reinterpret_cast<const u32x4*>(p.a);
  uint32_t xoff[XR];
#pragma unroll
  for (int i = 0; i < XR; ++i) {
    int64_t r = row0 + min(4 * i + h, rows - 1);
    if constexpr (MODE == QgMode::kMoeGateUp) r = p.sorted_assign[r] / p.top_k;
    xoff[i] = static_cast<uint32_t>(r * (K / 8));
  }
  // The wavefront's tile in LDS: rows of 256 bytes, piece q of row r at
  // position q ^ r, so that the 16 rows of a fragment read cover all banks.
  u32x4* const xl = reinterpret_cast<u32x4*>(lds) + wave * 256;

  const std::conditional_t<FMT == QM_Q8_G32, qg::DequantRegsQ8, qg::DequantRegs> dq;
  float4v acc[NM][RT][MT];
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[m][rt][mt] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

  uint32_t wv[U][NM][RT][W];
  uint32_t sv[U][NM][RT];
  u32x4 xv[U][XR];
  // Loads of step t: the lane's group g and its 16-byte activation piece.
  auto load = [&](auto uu, int g, uint32_t piece) __attribute__((always_inline)) {
    constexpr int u = decltype(uu)::value;
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        load_chunk<FMT, true>(wq[m] + static_cast<int64_t>(g) * CB, wrow + 16 * rt, wv[u][m][rt]);
        if constexpr (!kFloat) sv[u][m][rt] = wsc[m][static_cast<int64_t>(g) * kPanel + wrow + 16 * rt];
        else sv[u][m][rt] = 0;
      }
#pragma unroll
    for (int i = 0; i < XR; ++i) xv[u][i] = xbase[xoff[i] + piece];
  };
  auto compute = [&](auto uu, int t) __attribute__((always_inline)) {
    constexpr int u = decltype(uu)::value;
    if (4 * t + 4 > G) {
      // The last step of a K that is no multiple of 128: both operands of
      // the groups past the end become zero (an infinity times zero would
      // not be).
      const bool ok = 4 * t + h < G, xok = 4 * t + (c >> 2) < G;
#pragma unroll
      for (int i = 0; i < XR; ++i) xv[u][i] = xok ? xv[u][i] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int m = 0; m < NM; ++m)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          sv[u][m][rt] = ok ? sv[u][m][rt] : 0u;
          if constexpr (kFloat)
#pragma unroll
            for (int i = 0; i < W; ++i) wv[u][m][rt][i] = ok ? wv[u][m][rt][i] : 0u;
        }
    }
    half8v a[NM][RT][4];
#pragma unroll
    for (int m = 0; m < NM; ++m)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const _Float16 f = __builtin_bit_cast(_Float16, static_cast<uint16_t>(sv[u][m][rt]));
#pragma unroll
        for (int j = 0; j < 4; ++j) a[m][rt][j] = weight_frag<FMT>(wv[u][m][rt], j, half2v{f, f}, dq);
      }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      // Through the wavefront's own LDS tile (no barrier: one wavefront's LDS
      // accesses are in order) from the load order to the fragment order.
      // Rows past 4 XR are never stored.
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (4 * mt + i < XR) xl[(4 * i + h) * 16 + (c ^ (4 * i + h))] = xv[u][4 * mt + i];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
      half8v b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = __builtin_bit_cast(half8v, xl[c * 16 + ((4 * h + j) ^ c)]);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int m = 0; m < NM; ++m)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            acc[m][rt][mt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[m][rt][j], b[j], acc[m][rt][mt], 0, 0, 0);
    }
  };
  const int Q = (G + 3) / 4;                              // steps of four groups
  for (int t0 = wave; t0 < Q; t0 += kWaves * U) {
    // Steps past the end re-read the last one and are not used; groups past
    // the end of the last step re-read the last group.
    [&]<int... I>(std::integer_sequence<int, I...>) __attribute__((always_inline)) {
      (load(std::integral_constant<int, I>{}, min(4 * min(t0 + kWaves * I, Q - 1) + h, G - 1),
            min(16 * min(t0 + kWaves * I, Q - 1) + c, 4 * G - 1)), ...);
      ((t0 + kWaves * I < Q ? compute(std::integral_constant<int, I>{}, t0 + kWaves * I) : void()), ...);
    }(std::make_integer_sequence<int, U>{});
  }

  __syncthreads();                                        // every activation tile is used up
  // The wavefronts' partial sums, added in order.  Tile element: lane l holds
  // weight rows 4 (l / 16) + 0..3 of activation row l % 16.
#pragma unroll
  for (int m = 0; m < NM; ++m)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) lds[(wave * NM * TILES + (m * RT + rt) * MT + mt) * 64 + lane] = acc[m][rt][mt];
  __syncthreads();
  const bool vec = MODE == QgMode::kDense    ? mN % 4 == 0 && (reinterpret_cast<uintptr_t>(my) & 15u) == 0
                   : MODE == QgMode::kSwiglu ? mN % 4 == 0 && (reinterpret_cast<uintptr_t>(p.h) & 7u) == 0
                                             : true;
  for (int e = tid; e < TILES * 64; e += kWaves * 64) {
    const int tile = e >> 6, l = e & 63;
    const int token = 16 * (tile % MT) + (l & 15);
    const int64_t n = panel * kPanel + 16 * (RT * sub + tile / MT) + 4 * (l >> 4);
    float4v v[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      v[m] = lds[(m * TILES + tile) * 64 + l];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) v[m] += lds[(w * NM * TILES + m * TILES + tile) * 64 + l];
    }
    if (token >= rows || n >= mN) continue;
    const int64_t r = row0 + token;
    auto h16 = [](float f) { return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f)); };
    if constexpr (MODE == QgMode::kDense) {
      float* dst = my + r * mN + n;
      if (vec) {
        *reinterpret_cast<float4v*>(dst) = v[0];
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < mN) dst[i] = v[0][i];
      }
    } else if constexpr (two_matrices(MODE)) {
      uint16_t o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = h16(qg::silu_mul(v[0][i], v[NM - 1][i]));
      uint16_t* dst = p.h + r * mN + n;
      if (vec) {
        *reinterpret_cast<uint2*>(dst) = make_uint2(o[0] | o[1] << 16, o[2] | o[3] << 16);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (n + i < mN) dst[i] = o[i];
      }
    } else {
      // An assignment whose bucket is not the expert topk_ids names gets a
      // NaN weight, so its token's output row is NaN.
      const int64_t asg = p.sorted_assign[r];
      const float w = p.topk_ids[asg] == expert ? p.topk_w[asg] : __builtin_nanf("");
      uint16_t o[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = h16(w * v[0][i]);
      *reinterpret_cast<uint2*>(p.yp + asg * mN + n) = make_uint2(o[0] | o[1] << 16, o[2] | o[3] << 16);
    }
  }
}

}  // namespace fr

template <int FMT, int RT, int XR, int U, QgMode MODE>
__global__ __launch_bounds__((fr::kWaves * 64), (fr::kWavesPerSimd<FMT, RT, XR, U, MODE>)) void
fewrow_kernel(QgemmArgs p) {
  fr::body<FMT, RT, XR, U, MODE>(p);
}

}  // namespace qm
