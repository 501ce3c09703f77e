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

// The same for a 3x3 layer whose weights and velocities lie in the order of the lanes of its backward-data tiles (F_W_PERM,
// see pb_device.h): runs of 64 lanes x 4 weights for 16 output channels, 16 input channels and one tap.  A wavefront takes
// every fourth run of the tile of 16 kgs rows x 16 2^lcg channels; the predicted weights stay in LDS.
template <int U, class F>
__device__ __forceinline__ void tile_update_lanes(const LDesc& d, lfloat* T, int pitch, int kgs, int lcg, int mt0, int c0, F stage) {
  const float fa = UNIF(d.fa), fb = UNIF(d.fb), lrT = UNIF(d.flrT), lr = UNIF(d.flr), fm = UNIF(d.fm);
  const bool wform = UNI(d.flags) & F_LWP_W;
  gfloat* wp = GP((float*)d.w);
  gfloat* vp = GP(d.v);
  const int lane = threadIdx.x & 63, wv = UNI((int)threadIdx.x >> 6), kb = UNI(d.K) >> 5;
  const int np = (9 * kgs) << lcg;
  lfloat* Tl = T + (lane >> 4) * pitch + (lane & 15) * 9;
  v4f w[2][U], v[2][U];
  auto run_of = [&](int p, int& lds) {
    const int g = UNI(fdiv(p, 1.f / 9.f)), tap = p - 9 * g, kg = g >> lcg, cg = g & ((1 << lcg) - 1), k = mt0 + 16 * kg;
    lds = 16 * kg * pitch + 144 * cg + tap;
    return (size_t)(((((c0 >> 4) + cg) * kb + (k >> 5)) * 9 + tap) * 2 + ((k >> 4) & 1)) * 256;
  };
  auto issue = [&](auto B, int i0) {
    constexpr int b = decltype(B)::value;
    const unsigned lb = here(16u * (unsigned)lane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = 4 * (i0 + u) + wv;
      int lds;
      const size_t o = run_of(p < np ? p : np - 1, lds);
      w[b][u] = *(const gv4*)((const gbyte*)(wp + o) + lb);
      v[b][u] = *(const gv4*)((const gbyte*)(vp + o) + lb);
    }
  };
  auto apply = [&](auto B, int i0) {
    constexpr int b = decltype(B)::value;
    const unsigned lb = here(16u * (unsigned)lane);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int p = 4 * (i0 + u) + wv;
      if (p >= np) continue;
      int lds;
      const size_t o = run_of(p, lds);
      v4f v2, w2;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lfloat* q = Tl + lds + 4 * e * pitch;
        const float g = *q;
        v2[e] = fmaf(fm, v[b][u][e], g);
        w2[e] = fmaf(-lr, fmaf(fa, v2[e], fb * g), w[b][u][e]);
        *q = wform ? fmaf(lrT, w2[e] - w[b][u][e], w2[e]) : fmaf(-lrT, v2[e], w2[e]);
      }
      *(gv4*)((gbyte*)(vp + o) + lb) = v2;
      *(gv4*)((gbyte*)(wp + o) + lb) = w2;
    }
  };
  const int n = (np + 3) >> 2;
  issue(IConst<0>(), 0);
  stage();
  __syncthreads();
  for (int i = 0; i < n; i += 2 * U) {
    if (i + U < n) issue(IConst<1>(), i + U);
    apply(IConst<0>(), i);
    if (i + U >= n) break;
    if (i + 2 * U < n) issue(IConst<0>(), i + 2 * U);
    apply(IConst<1>(), i + U);
  }
}

}  // namespace pb
