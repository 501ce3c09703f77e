// The update of the weights of a backward-weights tile by the workgroup that holds their gradients (F_UPD_W).
//
// Included by pb_gemm.h.
#pragma once
#include "pb_device.h"

namespace pb {

// A tile of `rows` rows x 4 cv consecutive weights, its rows ldw floats apart in memory, the first weight at o0 (o0 and ldw
// multiples of 4); stage() puts its gradients into LDS as rows of `pitch` floats at T.  Bound by memory: 20 bytes per weight
// beside whatever else the launch streams.  The accumulators of a contraction give a lane 36-byte or 4-byte segments, and a
// wavefront that accesses them as they lie touches every cache line three to nine times: the tiles of the wide network took
// 29 us for it (2.5 TB/s over the launch).  Hence the way through LDS: a thread then owns whole 16-byte vectors that its
// neighbours continue, and U vectors per array are requested together, the first ones before the gradients are staged, the
// next ones before these are used.  512 ticks of the wide network 67.0 -> 61.9 ms, 384 of ResNet-50's stages at 64 pixels
// 93.0 -> 88.6, 256 at 224 pixels 154.9 -> 151.7, results bit for bit the same.  (U = 6 and 8 spill registers.)
// keep: the predicted weights stay in LDS in place of the gradients (the caller stores them in an order of its own).
template <int U, class F>
__device__ __forceinline__ void tile_update(const LDesc& d, lfloat* T, int pitch, int rows, int cv, unsigned o0, unsigned ldw, bool keep, F stage) {
  const float fa = UNIF(d.fa), fb = UNIF(d.fb), lrT = UNIF(d.flrT), lr = UNIF(d.flr), fm = UNIF(d.fm);
  const bool wform = UNI(d.flags) & F_LWP_W;
  gfloat* wp = GP((float*)d.w);
  gfloat* vp = GP(d.v);
  gfloat* hp = GP(d.what);
  const int tid = threadIdx.x, total = rows * cv;
  const float icv = frcp(cv);
  v4f w[2][U], v[2][U];
  auto issue = [&](auto B, int base) {
    constexpr int b = decltype(B)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int i = base + tid + u * BLK;
      i = i < total ? i : total - 1;
      const int r = fdiv(i, icv);
      const unsigned o = o0 + (unsigned)r * ldw + (unsigned)(4 * (i - r * cv));
      w[b][u] = *(const gv4*)(wp + o);
      v[b][u] = *(const gv4*)(vp + o);
    }
  };
  auto apply = [&](auto B, int base) {
    constexpr int b = decltype(B)::value;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + tid + u * BLK;
      if (i >= total) continue;
      const int r = fdiv(i, icv), c = i - r * cv;
      const unsigned o = o0 + (unsigned)r * ldw + (unsigned)(4 * c);
      lv4* g = (lv4*)(T + r * pitch + 4 * c);
      const v4f gv = *g;
      v4f v2, w2, h;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v2[e] = fmaf(fm, v[b][u][e], gv[e]);
        w2[e] = fmaf(-lr, fmaf(fa, v2[e], fb * gv[e]), w[b][u][e]);
        h[e] = wform ? fmaf(lrT, w2[e] - w[b][u][e], w2[e]) : fmaf(-lrT, v2[e], w2[e]);
      }
      *(gv4*)(vp + o) = v2;
      *(gv4*)(wp + o) = w2;
      if (keep) *g = h;
      else *(gv4*)(hp + o) = h;
    }
  };
  issue(IConst<0>(), 0);
  stage();
  __syncthreads();
  for (int base = 0; base < total; base += 2 * U * BLK) {
    if (base + U * BLK < total) issue(IConst<1>(), base + U * BLK);
    apply(IConst<0>(), base);
    if (base + U * BLK >= total) break;
    if (base + 2 * U * BLK < total) issue(IConst<0>(), base + 2 * U * BLK);
    apply(IConst<1>(), base + U * BLK);
  }
}

}  // namespace pb
