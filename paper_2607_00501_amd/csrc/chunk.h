// Loads of one weight row's share of a (panel, group) chunk block of the
// device layout, shared by the GEMV and the few-row matmul kernels.
#pragma once

#include "qm_internal.h"

namespace qm {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

// One lane's share of chunk block `blk` (panel row r): the planes, halves or
// quarters of the device layout, each a coalesced wavefront load.
template <int W, bool NT>
__device__ __forceinline__ void load_words(const uint8_t* p, uint32_t* d) {
  if constexpr (W == 4) {
    const u32x4 v = NT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)) : *reinterpret_cast<const u32x4*>(p);
    d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
  } else if constexpr (W == 2) {
    const u32x2 v = NT ? __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p)) : *reinterpret_cast<const u32x2*>(p);
    d[0] = v.x; d[1] = v.y;
  } else {
    d[0] = NT ? __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p)) : *reinterpret_cast<const uint32_t*>(p);
  }
}
template <int FMT, bool NT>
__device__ __forceinline__ void load_chunk(const uint8_t* blk, int r, uint32_t* d) {
  if constexpr (FMT == QM_Q4_G32) {
    load_words<4, NT>(blk + 16 * r, d);
  } else if constexpr (FMT == QM_Q8_G32) {
    load_words<4, NT>(blk + 16 * r, d);
    load_words<4, NT>(blk + 1024 + 16 * r, d + 4);
  } else if constexpr (FMT == QM_Q2_G32) {
    load_words<2, NT>(blk + 8 * r, d);
  } else if constexpr (FMT == QM_Q3_G32) {
    load_words<2, NT>(blk + 8 * r, d);
    load_words<1, NT>(blk + 512 + 4 * r, d + 2);
  } else if constexpr (FMT == QM_Q5_G32) {
    load_words<4, NT>(blk + 16 * r, d);
    load_words<1, NT>(blk + 1024 + 4 * r, d + 4);
  } else if constexpr (FMT == QM_Q6_G32) {
    load_words<4, NT>(blk + 16 * r, d);
    load_words<2, NT>(blk + 1024 + 8 * r, d + 4);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) load_words<4, NT>(blk + 1024 * j + 16 * r, d + 4 * j);
  }
}

}  // namespace qm
