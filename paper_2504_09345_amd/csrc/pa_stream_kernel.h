// The stream-K decode kernel template and its picker by GQA group size s and
// waves per workgroup W (design in pa_stream.hip).  Each (element type, head
// dim, trace) combination is instantiated in one translation unit.
#pragma once

#include "pa_stream_body.h"

namespace pa {

template <typename T, int D, int S, int W, int SUB, int NBUF, bool MF, bool TR>
__global__ __launch_bounds__(64 * W * SUB) void stream_kernel(StreamArgs a) {
  __shared__ StreamSmem<W, SUB, D, MF> sm;
  stream_body<T, D, S, W, SUB, NBUF, MF, TR>(a, sm, blockIdx.x, gridDim.x);
}

template <typename T, int D, int S, bool TR>
const void* stream_pick_w(int W, int sub) {
  constexpr bool mf = kStreamMfma && sizeof(T) == 2;
  if (sub == 1) {
    switch (W) {
      case 1: return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 1, 1, kStreamRing, mf, TR>);
      case 2: return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 2, 1, kStreamRing, mf, TR>);
      case 4: return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 4, 1, kStreamRing, mf, TR>);
      case 8: return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 8, 1, kStreamRing, mf, TR>);
    }
  } else {
    constexpr int dtype = sizeof(T) == 2 ? 0 : 1;
    constexpr int n1 = stream_teams(dtype, D, 1), n2 = stream_teams(dtype, D, 2), n4 = stream_teams(dtype, D, 4);
    if (W == 1 && sub == n1) return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 1, n1, kStreamRing, mf, TR>);
    if (W == 2 && sub == n2) return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 2, n2, kStreamRing, mf, TR>);
    if (W == 4 && sub == n4) return reinterpret_cast<const void*>(&stream_kernel<T, D, S, 4, n4, kStreamRing, mf, TR>);
  }
  return nullptr;
}

template <typename T, int D, bool TR>
const void* stream_pick(int s, int W, int sub) {
  switch (s) {
    case 1: return stream_pick_w<T, D, 1, TR>(W, sub);
    case 2: return stream_pick_w<T, D, 2, TR>(W, sub);
    case 4: return stream_pick_w<T, D, 4, TR>(W, sub);
    case 6: return stream_pick_w<T, D, 6, TR>(W, sub);
    case 8: return stream_pick_w<T, D, 8, TR>(W, sub);
  }
  return nullptr;
}

}  // namespace pa
