// The gather of the pruned search (find_pruned.hip): the units' present positions in the
// spatial order, with the bounding boxes of every leaf, top and sixteen tops.  A device
// function, so that the last launch of an update, which leaves the positions final, can make
// the records for the next search in workgroups of their own beside its own work.
#pragma once

#include "gsn_internal.h"

namespace gsn {

template <int CTRL, typename Op>
__device__ __forceinline__ float row_step(float v, Op op) {
  return op(v, __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf,
                                                       true)));
}

// over the kPrunedLeaf lanes that hold a leaf, in every one of them
template <typename Op>
__device__ __forceinline__ float leaf_reduce(float v, Op op) {
  static_assert(kPrunedLeaf == 32, "two rows of 16 lanes");
  v = row_step<0xB1>(v, op);
  v = row_step<0x4E>(v, op);
  v = row_step<0x141>(v, op);
  v = row_step<0x140>(v, op);
  return op(v, __shfl_xor(v, 16));
}

// The records and boxes of top t, by a workgroup of kBlock threads (every thread calls it; it
// holds a barrier; red is LDS).  Slots of the last leaf past the order's end, and slots whose
// unit was removed (index -1), hold NaN records with index -1, whose keys are above every real
// one; leaves wholly past the end are not written (nobody reads them).
constexpr int kGatherRed = 6 * (kPrunedTop / kPrunedLeaf);

__device__ __forceinline__ void gather_top(const GatherArgs& g, int32_t t, float* red) {
  constexpr int kPer = kPrunedTop / kBlock, kFan = kPrunedTop / kPrunedLeaf;
  const float inf = __builtin_huge_valf();
  const int tid = threadIdx.x;
  int32_t unit[kPer];
  float4 w[kPer];
#pragma unroll
  for (int h = 0; h < kPer; ++h) {
    const int32_t pos = t * kPrunedTop + h * kBlock + tid;
    unit[h] = pos < g.slots ? g.pidx[pos] : -1;
  }
#pragma unroll
  for (int h = 0; h < kPer; ++h) {
    const bool live = unit[h] >= 0 && unit[h] < g.n;
    const int32_t i = live ? unit[h] : 0;
    const float nan = __builtin_nanf("");
    w[h] = make_float4(g.x[i], g.y[i], g.z[i], __int_as_float(i));
    if (!live) w[h] = make_float4(nan, nan, nan, __int_as_float(-1));
  }
#pragma unroll
  for (int h = 0; h < kPer; ++h) {
    const int32_t pos = t * kPrunedTop + h * kBlock + tid, lf = pos / kPrunedLeaf;
    const bool live = __float_as_int(w[h].w) >= 0, has = lf * kPrunedLeaf < g.slots;
    if (has) g.pq[pos] = w[h];
    float v[6] = {live ? w[h].x : inf, live ? w[h].y : inf, live ? w[h].z : inf,
                  live ? w[h].x : -inf, live ? w[h].y : -inf, live ? w[h].z : -inf};
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      v[a] = leaf_reduce(v[a], FMin());
      v[3 + a] = leaf_reduce(v[3 + a], FMax());
    }
    if (tid % kPrunedLeaf == 0) {
      if (has) {
        g.leaf[2 * lf] = make_float4(v[0], v[1], v[2], 0.0f);
        g.leaf[2 * lf + 1] = make_float4(v[3], v[4], v[5], 0.0f);
      }
      float* r = red + 6 * (lf % kFan);
#pragma unroll
      for (int a = 0; a < 6; ++a) r[a] = v[a];
    }
  }
  __syncthreads();
  if (tid < 6) {
    float v = red[tid];
    for (int k = 1; k < kFan; ++k) {
      const float r = red[6 * k + tid];
      v = tid < 3 ? fminf(v, r) : fmaxf(v, r);
    }
    reinterpret_cast<float*>(&g.top[2 * t + tid / 3])[tid % 3] = v;
    int32_t* u = &g.sup[kSupWords * (t / kFan) + tid];
    if (tid < 3) atomicMin(u, ord(v)); else atomicMax(u, ord(v));
  }
  // the other set of outer boxes, for the next gather
  if (t == 0)
    for (int32_t i = tid; i < g.sup_words; i += kBlock)
      g.sup_next[i] = i % kSupWords < 3 ? ord(inf) : ord(-inf);
}

}  // namespace gsn
