// 3x3 layers (padding 1, stride 1 or 2) of networks tiled for throughput: all three passes on
// v_mfma_f32_16x16x4_f32 without offset tables and without a staged weight operand.
//
// The patch-based tiles of pb_gemm.h spend 55-60 % of their time outside the MFMA loop (12 requests per thread
// and chunk, the stores of both operands into LDS, two barriers) and read LDS once per MFMA, offsets on top.
// Here the reduction is walked in blocks of 4 channels x 9 taps: lane group kq = lane / 16 supplies channel
// 4 b + kq in all nine MFMAs of block b, so
//   * a lane's nine weights of a block are the nine taps of one (output, input) channel pair, 36 contiguous bytes
//     in memory, forward and backward alike: they go straight into registers, one superblock ahead;
//   * its nine map values are a 3x3 window at a fixed lane offset into the zero-padded patch in LDS: three row
//     addresses, the columns are immediate offsets.
// A wave keeps MI x NI accumulators, so a window read from LDS feeds MI MFMAs and a weight NI.  The patch is double
// buffered, the next chunk's 16-byte requests (rows whose length is no multiple of 4 included: unaligned loads, the
// tail masked on its way into LDS) are in flight while this one is contracted; one barrier per chunk.
//
// Backward data of a stride-2 layer runs over the gradient's pixels: the nine taps of a gradient pixel's window
// fall into the four parity classes of the 2x2 input pixels it belongs to (4, 2, 2 and 1 taps), one accumulator
// set each -- a quarter of the work of a gradient spread out with zeros.
//
// Backward weights: MFMA rows are output channels, columns are 16 input channels for one tap, reduction = pixels
// (rows padded to a multiple of 4); nine accumulators per row subtile, so the output gradient is read once and
// the 6 (stride 2: 9) map values of a window row serve 12 MFMAs.
//
// 1x1 layers on maps of fewer than 64 pixels (step_d1_t): both operands go straight from memory into registers, no LDS
// and no barrier; such a layer streams its weights and is bound by their way from memory.
//
// Included by pb_gemm.h.
#pragma once
#include "pb_device.h"

namespace pb {

// acc += a[tap] * window, see above.  MODE 1 forward, 2 backward data.
template <int MODE, bool S2, int MI, int NI>
__device__ __forceinline__ void step_dc_t(const LDesc& d, int tile_, int t, lfloat* smem) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
  constexpr int UB = 4 / MI;               // blocks per superblock: 36 weight registers whatever MI
  constexpr int NC = S2 ? 4 : 1;           // accumulator sets
  constexpr int NR = S2 ? 2 : 3;           // window rows (columns) read
  const int tid = threadIdx.x, lane = tid & 63, wv = UNI(tid >> 6), li = lane & 15, kq = lane >> 4;
  const int wk = UNI(d.g.wk), wn = UNI(d.g.wn);
  auto lg = [](int x) { return x == 1 ? 0 : (x == 2 ? 1 : 2); };
  const int wk_id = wv & (wk - 1), wn_id = (wv >> lg(wk)) & (wn - 1), wm_id = wv >> (lg(wk) + lg(wn));
  const int N = UNI(d.g.N), C = UNI(d.C), flags = UNI(d.flags);
  const int tiles_n = UNI(d.g.tiles_n), tpp = UNI(d.g.tpp);
  const int qpart = UNI(fdiv(tile, frcp(tpp)));
  tile -= qpart * tpp;
  const int tm = UNI(fdiv(tile, frcp(tiles_n))), tn = tile - tm * tiles_n;
  const int m0 = tm * UNI(d.g.MT), n0 = tn * UNI(d.g.NT);
  const int SH = UNI(MODE == 1 ? d.H : d.OH), SW = UNI(MODE == 1 ? d.W : d.OW);
  const int PWd = UNI((MODE == 1 || S2) ? d.OW : d.W);            // row length of the pixel space
  const int st = MODE == 1 ? UNI(d.stride) : 1;
  const int CC = UNI(d.g.CC), PR = UNI(d.g.PR), Wp = UNI(d.g.Wp), plane = UNI(d.g.shw), W4 = UNI(d.g.sw);
  const int n_chunks = UNI(d.g.n_chunks), ch0 = qpart * UNI(d.g.cpp);
  const int ch_end = ch0 + UNI(d.g.cpp) < n_chunks ? ch0 + UNI(d.g.cpp) : n_chunks;
  const gfloat* Ag = GP(d.w);
  const gfloat* src = MODE == 2 ? (const gfloat*)at(d.dy, t) : (const gfloat*)at(d.x, t);

  // ---- patch: patch row 0 is source row row0, source column x lies at patch column 4 + x
  const float ipw = frcp(PWd);
  const int y0 = UNI(fdiv(n0, ipw)), row0 = S2 ? y0 : y0 * st - 1;
  const int tail = SW & 3;
  int pdst[DC_VU], psrc[DC_VU];
  {
    const float ichs = frcp(PR * W4), iw4 = frcp(W4);
#pragma unroll
    for (int u = 0; u < DC_VU; ++u) {
      const int i = tid + u * BLK, c = fdiv(i, ichs), rem = i - c * PR * W4, y = fdiv(rem, iw4), x = rem - y * W4;
      const int sy = row0 + y;
      const bool ok = c < CC && sy >= 0 && sy < SH;
      pdst[u] = ok ? (c * plane + y * Wp + 4 + 4 * x) | (x == W4 - 1 ? 1 : 0) : -1;
      psrc[u] = ok ? (c * SH + sy) * SW + 4 * x : 0;
    }
  }
  v4f pv[DC_VU];
  auto p_issue = [&](int ch) {
    const gfloat* s = src + (size_t)ch * (size_t)(CC * SH * SW);
#pragma unroll
    for (int u = 0; u < DC_VU; ++u)
      if (pdst[u] >= 0) pv[u] = *(const gv4u*)(s + (unsigned)psrc[u]);
  };
  auto p_commit = [&](lfloat* buf) {
#pragma unroll
    for (int u = 0; u < DC_VU; ++u)
      if (pdst[u] >= 0) {
        v4f v = pv[u];
        if (tail && (pdst[u] & 1)) {
          if (tail < 2) v[1] = 0.f;
          if (tail < 3) v[2] = 0.f;
          v[3] = 0.f;
        }
        *(lv4*)(buf + (pdst[u] & ~1)) = v;
      }
  };
  // ---- weights: lane (row li, channel kq of a block); 9 floats per block and row subtile.  Forward, the rows lie 36 C bytes
  // apart and a wave's load touches 16 of them, often on the same cache sets and memory channels; where the update of the
  // layer runs in its weight-gradient tiles they store the predicted weights in the order of the lanes instead.
  const bool perm = MODE == 1 && (flags & F_WHAT_PERM);
  const int acs = MODE == 1 ? (perm ? 144 : 9) : 9 * C;            // floats between a lane's weights of two channels 4 apart, / 4
  const unsigned lane_o = perm ? 9u * lane : (unsigned)(li * (MODE == 1 ? 9 * C : 9) + kq * acs);
  const int nsb = UNI(CC / (4 * UB * wk));                         // superblocks per chunk and wave
  const int g_end = (ch_end - ch0) * nsb;
  const unsigned a_i = (unsigned)(MODE == 1 ? 144 * C : 144);      // floats between two row subtiles
  const unsigned abase = lane_o + (unsigned)((m0 >> 4) + wm_id * MI) * a_i + (unsigned)((ch0 * CC + 4 * UB * wk_id) * acs);
  const unsigned a_ub = (unsigned)(4 * acs), a_sb = (unsigned)(4 * UB * wk * acs);
  float a[UB][MI][9];
  auto load_a = [&](float (&r)[UB][MI][9], int g) {
    const unsigned o = abase + (unsigned)g * a_sb;
#pragma unroll
    for (int ub = 0; ub < UB; ++ub)
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const gfloat* p = Ag + (o + (unsigned)ub * a_ub + (unsigned)i * a_i);
        const v4f x = *(const gv4u*)p, y = *(const gv4u*)(p + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) { r[ub][i][e] = x[e]; r[ub][i][4 + e] = y[e]; }
        r[ub][i][8] = p[8];
      }
  };
  p_issue(ch0);
  load_a(a, 0);
  // ---- lane offsets of the pixel subtiles' windows
  int poff[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    int n = n0 + (wn_id * NI + j) * 16 + li;
    n = n < N ? n : N - 1;
    const int y = fdiv(n, ipw), x = n - y * PWd;
    poff[j] = kq * plane + (S2 ? (y - row0) * Wp + x + 4 : (y * st - 1 - row0) * Wp + x * st + 3) + 4 * UB * wk_id * plane;
  }
  v4f acc[NC][MI][NI];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[c][i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  constexpr bool DUAL = MI * NI == 1 && !S2;   // (a second set: consecutive MFMAs would wait for each other)
  v4f acc2 = (v4f){0.f, 0.f, 0.f, 0.f};
  const int buf_fl = CC * plane;
  for (int i = tid; i < (2 * buf_fl) >> 2; i += BLK) *(lv4*)(smem + 4 * i) = (v4f){0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  p_commit(smem);
  __syncthreads();
  // Forward, a chunk's sum is formed by itself and added to the total.  Against float64, the gradients of 3x3 weights
  // (which carry the forward pass's error) are 0-5 % nearer than with one chain (2.52e-7 and 2.66e-7 at 128 and 256
  // channels, equal at 64); beside the patch-based tiles VGG-11, the wide network and ResNet-50 at 64 pixels stand at
  // 0.90, 0.72 and 0.98 of the error.
  constexpr bool BLOCKED = MODE == 1;
  v4f tot[BLOCKED ? MI : 1][BLOCKED ? NI : 1];
  if (BLOCKED) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) tot[BLOCKED ? i : 0][BLOCKED ? j : 0] = (v4f){0.f, 0.f, 0.f, 0.f};
  }
  const int sb_fl = 4 * UB * wk * plane;
  int g = 0;
  PB_TS(9);
  for (int ch = ch0; ch < ch_end; ++ch) {
    const lfloat* cur = smem + ((ch - ch0) & 1) * buf_fl;
    lfloat* nxt = smem + (((ch - ch0) & 1) ^ 1) * buf_fl;
    const bool more = ch + 1 < ch_end;
    if (more) p_issue(ch + 1);
    float b[2][NR][NI];
    auto load_b = [&](auto BI, const lfloat* base, int h) {
      constexpr int bi = decltype(BI)::value;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const lfloat* p = base + poff[j] + h * Wp;
#pragma unroll
        for (int x = 0; x < NR; ++x) b[bi][x][j] = p[x];
      }
    };
    auto mfmas = [&](auto BI, int ub, int h) {
      constexpr int bi = decltype(BI)::value;
      if constexpr (S2) {
        // window row h: gradient row y + h; taps kh = 0 (h 1, odd input row), 1 (h 0, even), 2 (h 0, odd)
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
          if ((kh == 0 ? 1 : 0) != h) continue;
#pragma unroll
          for (int kw = 0; kw < 3; ++kw) {
            const int cls = (kh == 1 ? 0 : 2) + (kw == 1 ? 0 : 1);
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
              for (int j = 0; j < NI; ++j)
                acc[cls][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ub][i][3 * kh + kw], b[bi][kw == 0 ? 1 : 0][j], acc[cls][i][j], 0, 0, 0);
          }
        }
      } else {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
          const int tap = MODE == 1 ? 3 * h + x : 8 - (3 * h + x);
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
              if (DUAL && ((h + x) & 1)) acc2 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ub][i][tap], b[bi][x][j], acc2, 0, 0, 0);
              else acc[0][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ub][i][tap], b[bi][x][j], acc[0][i][j], 0, 0, 0);
            }
        }
      }
    };
    load_b(IConst<0>(), cur, 0);
    const lfloat* base = cur;
    for (int s = 0; s < nsb; ++s, ++g) {
      float an[UB][MI][9];
      load_a(an, g + 1 < g_end ? g + 1 : g);
      const lfloat* next = s + 1 < nsb ? base + sb_fl : cur;
#pragma unroll
      for (int q = 0; q < UB * NR; ++q) {
        // the next window row comes from LDS while this one's MFMAs run
        const lfloat* nb = q + 1 < UB * NR ? base + ((q + 1) / NR) * 4 * plane : next;
        const int nh = q + 1 < UB * NR ? (q + 1) % NR : 0;
        if (q & 1) { load_b(IConst<0>(), nb, nh); __builtin_amdgcn_sched_barrier(0); mfmas(IConst<1>(), q / NR, q % NR); }
        else { load_b(IConst<1>(), nb, nh); __builtin_amdgcn_sched_barrier(0); mfmas(IConst<0>(), q / NR, q % NR); }
        __builtin_amdgcn_sched_barrier(0);
      }
      if ((UB * NR) & 1) {
#pragma unroll
        for (int x = 0; x < NR; ++x)
#pragma unroll
          for (int j = 0; j < NI; ++j) b[0][x][j] = b[1][x][j];
      }
#pragma unroll
      for (int ub = 0; ub < UB; ++ub)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int e = 0; e < 9; ++e) a[ub][i][e] = an[ub][i][e];
      base = next;
    }
    if (more) p_commit(nxt);
    if (BLOCKED) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          tot[BLOCKED ? i : 0][BLOCKED ? j : 0] += acc[0][i][j];
          acc[0][i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
        }
    }
    __syncthreads();
  }
  PB_TS(10);
  if (BLOCKED) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[0][i][j] = tot[BLOCKED ? i : 0][BLOCKED ? j : 0];
  }
  if (DUAL) acc[0][0][0] += acc2;
  // ---- the waves' shares of the reduction, in order
  if (wk > 1) {
    if (wk_id > 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) *(lv4*)(smem + (((wv * NC + c) * MI * NI + i * NI + j) * 64 + lane) * 4) = acc[c][i][j];
    }
    __syncthreads();
    if (wk_id != 0) return;
    for (int w2 = 1; w2 < wk; ++w2)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[c][i][j] += *(const lv4*)(smem + ((((wv + w2) * NC + c) * MI * NI + i * NI + j) * 64 + lane) * 4);
  }
  // ---- epilogue: lane holds rows 4 kq + r, column li of each 16x16 subtile
  int te = t;
  asm volatile("" : "+s"(te));
  const bool round = flags & F_BF16_OUT;
  gfloat* out = UNI(d.g.parts) > 1 ? GP(d.gw) + (size_t)qpart * (size_t)UNI(d.gpstride) : MODE == 2 ? at(d.dx, te) : at(d.y, te);
  if constexpr (S2) {
    const int H = UNI(d.H), W = UNI(d.W);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int n = n0 + (wn_id * NI + j) * 16 + li;
      if (n >= N) continue;
      const int y = fdiv(n, ipw), x = n - y * PWd;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gfloat* q = out + (size_t)(m0 + (wm_id * MI + i) * 16 + 4 * kq + r) * (size_t)(H * W) + 2 * y * W + 2 * x;
#pragma unroll
          for (int py = 0; py < 2; ++py) {
            if (2 * y + py >= H) continue;
            const float v0 = rbf_if(round, acc[2 * py][i][j][r]), v1 = rbf_if(round, acc[2 * py + 1][i][j][r]);
            if (!(W & 1)) *(gv2*)(q + py * W) = (v2f){v0, v1};
            else { q[py * W] = v0; if (2 * x + 1 < W) q[py * W + 1] = v1; }
          }
        }
    }
    return;
  } else {
    const gfloat* skip = (MODE == 1 && (flags & F_SKIP)) ? (const gfloat*)at(d.skip, te) : nullptr;
    const gfloat* bias = (MODE == 1 && (flags & F_BIAS) && qpart == 0) ? GP(d.b) : nullptr;
    const gfloat* xm = (MODE == 2 && (flags & F_MASK_X)) ? (const gfloat*)at(d.x, te) : nullptr;
    const gfloat* skg = (MODE == 2 && (flags & F_ADD_SKG)) ? (const gfloat*)at(d.skg, te) : nullptr;
    float add[MI][NI][4], msk[MI][NI][4];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) { add[i][j][r] = 0.f; msk[i][j][r] = 1.f; }
    auto epi_fetch = [&](const gfloat* s, float (&dst)[MI][NI][4]) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int n = n0 + (wn_id * NI + j) * 16 + li, nc = n < N ? n : N - 1;
#pragma unroll
          for (int r = 0; r < 4; ++r) dst[i][j][r] = s[(size_t)(m0 + (wm_id * MI + i) * 16 + 4 * kq + r) * N + nc];
        }
    };
    if (skip) epi_fetch(skip, add);
    if (skg) epi_fetch(skg, add);
    if (xm) epi_fetch(xm, msk);
    if (bias) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float bv = bias[m0 + (wm_id * MI + i) * 16 + 4 * kq + r];
#pragma unroll
          for (int j = 0; j < NI; ++j) add[i][j][r] += bv;
        }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n = n0 + (wn_id * NI + j) * 16 + li;
        if (n >= N) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float v = acc[0][i][j][r];
          if (MODE == 2 && !(msk[i][j][r] > 0.f)) v = 0.f;
          out[(size_t)(m0 + (wm_id * MI + i) * 16 + 4 * kq + r) * N + n] = rbf_if(round, v + add[i][j][r]);
        }
      }
  }
}

// Backward weights, stride S, MI row subtiles per wave.
// live: false before the layer's first gradient, when a step that updates the weights only carries them over.
template <int S, int MI>
__device__ __forceinline__ void step_dcw_t(const LDesc& d, int tile_, int t, lfloat* smem, bool live) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
  constexpr int NX = 3 * S + 3;              // map values of a window row that four pixels and three taps need
  const int tid = threadIdx.x, lane = tid & 63, wv = UNI(tid >> 6), li = lane & 15, kq = lane >> 4;
  const int wk = UNI(d.g.wk), wn = UNI(d.g.wn);
  auto lg = [](int x) { return x == 1 ? 0 : (x == 2 ? 1 : 2); };
  const int wk_id = wv & (wk - 1), wn_id = (wv >> lg(wk)) & (wn - 1), wm_id = wv >> (lg(wk) + lg(wn));
  const int C = UNI(d.C), H = UNI(d.H), W = UNI(d.W), OH = UNI(d.OH), OW = UNI(d.OW), P = OH * OW;
  const int tiles_n = UNI(d.g.tiles_n), tpp = UNI(d.g.tpp);
  const int qpart = UNI(fdiv(tile, frcp(tpp)));
  tile -= qpart * tpp;
  const int tm = UNI(fdiv(tile, frcp(tiles_n))), tn = tile - tm * tiles_n;
  const int m0 = tm * UNI(d.g.MT) + wm_id * MI * 16, CT = 16 * wn, c0 = tn * CT;
  const int PR = UNI(d.g.PR), Wp = UNI(d.g.Wp), plane = UNI(d.g.shw), W4 = UNI(d.g.sw), rows_c = UNI(d.g.rows_c);
  const int n_chunks = UNI(d.g.n_chunks), ch0 = qpart * UNI(d.g.cpp);
  const int ch_end = !live ? ch0 : ch0 + UNI(d.g.cpp) < n_chunks ? ch0 + UNI(d.g.cpp) : n_chunks;
  const int OWp = (OW + 3) & ~3;             // pixels of a row in the reduction
  const gfloat* dy = at(d.dy, t);
  const gfloat* src = (const gfloat*)at(d.x, t) + (size_t)c0 * (size_t)(H * W);
  const int tail = W & 3;
  int pdst[DC_VU], psrc[DC_VU], prow[DC_VU];
  {
    const float ichs = frcp(PR * W4), iw4 = frcp(W4);
#pragma unroll
    for (int u = 0; u < DC_VU; ++u) {
      const int i = tid + u * BLK, c = fdiv(i, ichs), rem = i - c * PR * W4, y = fdiv(rem, iw4), x = rem - y * W4;
      const bool ok = c < CT;
      pdst[u] = ok ? (c * plane + y * Wp + 4 + 4 * x) | (x == W4 - 1 ? 1 : 0) : -1;
      psrc[u] = (c * H - 1 + y) * W + 4 * x;
      prow[u] = y - 1;
    }
  }
  v4f pv[DC_VU];
  auto p_issue = [&](int ch) {
    const int r0 = ch * rows_c * S;
#pragma unroll
    for (int u = 0; u < DC_VU; ++u) {
      pv[u] = (v4f){0.f, 0.f, 0.f, 0.f};
      const int sy = r0 + prow[u];
      if (pdst[u] >= 0 && sy >= 0 && sy < H) pv[u] = *(const gv4u*)(src + (unsigned)(psrc[u] + r0 * W));
    }
  };
  auto p_commit = [&](lfloat* buf) {
#pragma unroll
    for (int u = 0; u < DC_VU; ++u)
      if (pdst[u] >= 0) {
        v4f v = pv[u];
        if (tail && (pdst[u] & 1)) {
          if (tail < 2) v[1] = 0.f;
          if (tail < 3) v[2] = 0.f;
          v[3] = 0.f;
        }
        *(lv4*)(buf + (pdst[u] & ~1)) = v;
      }
  };
  const float iow = frcp(OWp);
  const int nblk = (rows_c * OWp + 15) >> 4;                       // blocks of 16 pixels per chunk
  const int nmine = nblk > wk_id ? (nblk - wk_id + wk - 1) >> lg(wk) : 0;
  // block i of this wave in chunk ch: the lane's four gradient values per row subtile, zero outside the map
  auto load_a = [&](v4f (&r)[MI], int ch, int i) {
    const int e = 16 * (i * wk + wk_id) + 4 * kq, y = fdiv(e, iow), x = e - y * OWp, oy = ch * rows_c + y;
    const bool ok = y < rows_c && oy < OH;
    const unsigned o = (unsigned)((m0 + li) * P + (ok ? oy * OW + x : 0));
#pragma unroll
    for (int k = 0; k < MI; ++k) {
      const v4f v = *(const gv4u*)(dy + (o + (unsigned)(16 * k * P)));
#pragma unroll
      for (int u = 0; u < 4; ++u) r[k][u] = (ok && x + u < OW) ? v[u] : 0.f;
    }
  };
  auto b_off = [&](int i) {
    const int e = 16 * (i * wk + wk_id) + 4 * kq;
    int y = fdiv(e, iow);
    const int x = e - y * OWp;
    y = y < rows_c ? y : rows_c - 1;
    return (wn_id * 16 + li) * plane + y * S * Wp + x * S + 3;
  };
  v4f acc[MI][9];
#pragma unroll
  for (int k = 0; k < MI; ++k)
#pragma unroll
    for (int j = 0; j < 9; ++j) acc[k][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  p_issue(ch0);
  v4f a[MI];
  load_a(a, ch0, 0);
  const int buf_fl = CT * plane;
  for (int i = tid; i < (2 * buf_fl + 64) >> 2; i += BLK) *(lv4*)(smem + 4 * i) = (v4f){0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  p_commit(smem);
  __syncthreads();                           // (a step that is not live yet contracts nothing)
  PB_TS(9);
  for (int ch = ch0; ch < ch_end; ++ch) {
    const lfloat* cur = smem + ((ch - ch0) & 1) * buf_fl;
    lfloat* nxt = smem + (((ch - ch0) & 1) ^ 1) * buf_fl;
    const bool more = ch + 1 < ch_end;
    if (more) p_issue(ch + 1);
    float b[2][NX];
    auto load_b = [&](auto BI, const lfloat* p) {
      constexpr int bi = decltype(BI)::value;
#pragma unroll
      for (int x = 0; x < NX; ++x) b[bi][x] = p[x];
    };
    auto mfmas = [&](auto BI, int kh) {
      constexpr int bi = decltype(BI)::value;
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int kw = 0; kw < 3; ++kw)
#pragma unroll
          for (int k = 0; k < MI; ++k)
            acc[k][3 * kh + kw] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k][u], b[bi][u * S + kw], acc[k][3 * kh + kw], 0, 0, 0);
    };
    const lfloat* p = cur + b_off(0);
    load_b(IConst<0>(), p);
    for (int i = 0; i < nmine; ++i) {
      v4f an[MI];
      const bool end = i + 1 >= nmine;
      load_a(an, end && more ? ch + 1 : ch, end ? 0 : i + 1);
      const lfloat* pn = cur + b_off(end ? 0 : i + 1);
      load_b(IConst<1>(), p + Wp);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(IConst<0>(), 0);
      __builtin_amdgcn_sched_barrier(0);
      load_b(IConst<0>(), p + 2 * Wp);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(IConst<1>(), 1);
      __builtin_amdgcn_sched_barrier(0);
      load_b(IConst<1>(), pn);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(IConst<0>(), 2);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int x = 0; x < NX; ++x) b[0][x] = b[1][x];
#pragma unroll
      for (int k = 0; k < MI; ++k) a[k] = an[k];
      p = pn;
    }
    if (nmine == 0 && more) load_a(a, ch + 1, 0);
    if (more) p_commit(nxt);
    __syncthreads();
  }
  PB_TS(10);
  // ---- the waves' shares of the reduction, in order
  const int flags = UNI(d.flags), ch = c0 + wn_id * 16 + li;
  if (wk > 1) {
    if (wk_id > 0) {
#pragma unroll
      for (int k = 0; k < MI; ++k)
#pragma unroll
        for (int j = 0; j < 9; ++j) *(lv4*)(smem + (((wv - (wv >> lg(wk)) - 1) * MI * 9 + k * 9 + j) * 64 + lane) * 4) = acc[k][j];
    }
    __syncthreads();
  }
  if (wk > 1 && wk_id == 0) {
    for (int w2 = 1; w2 < wk; ++w2) {
      const int ow = wv + w2;
#pragma unroll
      for (int k = 0; k < MI; ++k)
#pragma unroll
        for (int j = 0; j < 9; ++j) acc[k][j] += *(const lv4*)(smem + (((ow - (ow >> lg(wk)) - 1) * MI * 9 + k * 9 + j) * 64 + lane) * 4);
    }
  }
  if (flags & F_UPD_W) {
    // the update of the tile's weights: no gradient in memory (8 bytes per weight and a launch's tail saved).  The tile lies
    // behind the waves' shares: 2304 MI floats for all four waves' shares and sums together, 4 more per row.
    const int pitch = 9 * CT + 4, MT = UNI(d.g.MT), mt0 = tm * MT;
    lfloat* T = smem + (wk > 1 ? (4 - (4 >> lg(wk))) * MI * 9 * 256 : 0);
    const bool perm = flags & F_WHAT_PERM;
    tile_update<4>(d, T, pitch, MT, 9 * CT / 4, (unsigned)(mt0 * C + c0) * 9u, 9u * (unsigned)C, perm, [&]() {
      if (wk_id != 0) return;
#pragma unroll
      for (int k = 0; k < MI; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lfloat* q = T + ((wm_id * MI + k) * 16 + 4 * kq + r) * pitch + (wn_id * 16 + li) * 9;
#pragma unroll
          for (int e = 0; e < 9; ++e) q[e] = acc[k][e][r];
        }
    });
    if (perm) {
      // the predicted weights in the order of the forward tiles' lanes: 16 threads per block of 16 rows x 4 channels
      __syncthreads();
      const int nb = (MT >> 4) * (CT >> 2), tl = tid & 15;
      int off[9][4];
#pragma unroll
      for (int i = 0; i < 9; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int x = 4 * (tl + 16 * i) + e, s = fdiv(x, 1.f / 9.f), row = s & 15;
          off[i][e] = row * pitch + (s >> 4) * 9 + x - 9 * s;
        }
      for (int b = tid >> 4; b < nb; b += 16) {
        const int rt = b >> (2 + lg(wn)), c4 = b & (4 * wn - 1);
        const lfloat* p = T + 16 * rt * pitch + 36 * c4;
        gfloat* q = GP(d.what) + (size_t)((unsigned)(((mt0 >> 4) + rt) * (C >> 2) + (c0 >> 2) + c4) * 576u) + 4 * tl;
#pragma unroll
        for (int i = 0; i < 9; ++i) *(gv4*)(q + 64 * i) = (v4f){p[off[i][0]], p[off[i][1]], p[off[i][2]], p[off[i][3]]};
      }
    }
    return;
  }
  if (wk_id != 0) return;
  // ---- lane holds, for rows 4 kq + r and channel li, the nine taps: 36 contiguous bytes
  gfloat* out = GP(d.gw) + (size_t)qpart * (size_t)UNI(d.gpstride);
#pragma unroll
  for (int k = 0; k < MI; ++k)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      gfloat* q = out + (size_t)((m0 + k * 16 + 4 * kq + r) * C + ch) * 9;
      v4f x, y;
#pragma unroll
      for (int e = 0; e < 4; ++e) { x[e] = acc[k][e][r]; y[e] = acc[k][4 + e][r]; }
      *(gv4u*)q = x;
      *(gv4u*)(q + 4) = y;
      q[8] = acc[k][8][r];
    }
}

// Forward (MODE 1) and backward data (MODE 2) of a 1x1 layer of stride 1 or 2 on a small map.  The reduction is walked in
// blocks of 16 channels, in MFMA u of a block lane group kq supplies channel 4 kq + u.  Forward, a lane's four weights of a
// block are 16 contiguous bytes; backward they lie in four rows of the weight matrix, and with MI = 4 the row subtiles
// interleave (subtile i holds rows 4 li + i) so that a lane's weights of one channel are 16 contiguous bytes there.  The
// requests of UB blocks are in flight while the UB before are contracted.
template <int MODE, int MI, int NI>
__device__ __forceinline__ void step_d1_t(const LDesc& d, int tile_, int t, lfloat* smem) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
  constexpr int UB = MI * NI == 1 ? 4 : MI * NI == 4 ? 2 : 1;
  const int tid = threadIdx.x, lane = tid & 63, wv = UNI(tid >> 6), li = lane & 15, kq = lane >> 4;
  const int wk = UNI(d.g.wk);
  auto lg = [](int x) { return x == 1 ? 0 : (x == 2 ? 1 : 2); };
  const int wk_id = wv & (wk - 1), wm_id = wv >> lg(wk);
  const int N = UNI(d.g.N), R = UNI(d.g.Q), M = UNI(d.g.M), flags = UNI(d.flags), ps = UNI(d.g.ps);
  const int tiles_n = UNI(d.g.tiles_n);
  const int tm = UNI(fdiv(tile, frcp(tiles_n))), tn = tile - tm * tiles_n;
  const int m0 = tm * UNI(d.g.MT) + wm_id * 16 * MI, n0 = tn * UNI(d.g.NT);
  const int H = UNI(d.H), W = UNI(d.W), OW = UNI(d.OW);
  const gfloat* Ag = GP(d.w);
  const gfloat* src = MODE == 2 ? (const gfloat*)at(d.dy, t) : (const gfloat*)at(d.x, t);
  const int plane = MODE == 2 ? N : H * W;                          // floats of a channel of the source
  const float iow = frcp(OW);
  unsigned boff[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    int n = n0 + 16 * j + li;
    n = n < N ? n : N - 1;
    if (MODE == 1 && ps == 2) { const int y = fdiv(n, iow); n = 2 * (y * W + n - y * OW); }
    boff[j] = (unsigned)(4 * kq * plane + n);
  }
  const unsigned aoff = MODE == 1 ? (unsigned)((m0 + li) * R + 4 * kq) : (unsigned)(4 * kq * M + m0 + (MI == 4 ? 4 * li : li));
  float a[UB][MI][4], b[UB][NI][4];
  auto load = [&](float (&ra)[UB][MI][4], float (&rb)[UB][NI][4], int g) {
#pragma unroll
    for (int ub = 0; ub < UB; ++ub) {
      const unsigned blk = (unsigned)((g * wk + wk_id) * UB + ub);
      if (MODE == 1) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          const v4f x = *(const gv4u*)(Ag + (aoff + 16u * blk + (unsigned)(16 * i * R)));
#pragma unroll
          for (int u = 0; u < 4; ++u) ra[ub][i][u] = x[u];
        }
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const gfloat* p = Ag + (aoff + (16u * blk + (unsigned)u) * (unsigned)M);
          if constexpr (MI == 4) {
            const v4f x = *(const gv4u*)p;
#pragma unroll
            for (int i = 0; i < 4; ++i) ra[ub][i][u] = x[i];
          } else {
            ra[ub][0][u] = *p;
          }
        }
      }
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int u = 0; u < 4; ++u) rb[ub][j][u] = src[boff[j] + (16u * blk + (unsigned)u) * (unsigned)plane];
    }
  };
  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  const int ng = UNI((R >> 4) / (UB * wk));                         // superblocks of this wave
  load(a, b, 0);
  for (int g = 0; g < ng; ++g) {
    float an[UB][MI][4], bn[UB][NI][4];
    load(an, bn, g + 1 < ng ? g + 1 : g);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ub = 0; ub < UB; ++ub)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ub][i][u], b[ub][j][u], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ub = 0; ub < UB; ++ub)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int i = 0; i < MI; ++i) a[ub][i][u] = an[ub][i][u];
#pragma unroll
        for (int j = 0; j < NI; ++j) b[ub][j][u] = bn[ub][j][u];
      }
  }
  if (wk > 1) {
    if (wk_id > 0) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) *(lv4*)(smem + ((wv * MI * NI + i * NI + j) * 64 + lane) * 4) = acc[i][j];
    }
    __syncthreads();
    if (wk_id != 0) return;
    for (int w2 = 1; w2 < wk; ++w2)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) acc[i][j] += *(const lv4*)(smem + (((wv + w2) * MI * NI + i * NI + j) * 64 + lane) * 4);
  }
  int te = t;
  asm volatile("" : "+s"(te));
  const bool round = flags & F_BF16_OUT;
  gfloat* out = MODE == 2 ? at(d.dx, te) : at(d.y, te);
  auto row_of = [&](int i, int r) { return m0 + (MODE == 2 && MI == 4 ? 4 * (4 * kq + r) + i : 16 * i + 4 * kq + r); };
  const gfloat* skip = (MODE == 1 && (flags & F_SKIP)) ? (const gfloat*)at(d.skip, te) : nullptr;
  const gfloat* bias = (MODE == 1 && (flags & F_BIAS)) ? GP(d.b) : nullptr;
  const gfloat* xm = (MODE == 2 && (flags & F_MASK_X)) ? (const gfloat*)at(d.x, te) : nullptr;
  const gfloat* skg = (MODE == 2 && (flags & F_ADD_SKG)) ? (const gfloat*)at(d.skg, te) : nullptr;
  float add[MI][NI][4], msk[MI][NI][4];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) { add[i][j][r] = 0.f; msk[i][j][r] = 1.f; }
  auto epi_fetch = [&](const gfloat* s, float (&dst)[MI][NI][4]) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int n = n0 + 16 * j + li, nc = n < N ? n : N - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[i][j][r] = s[(size_t)row_of(i, r) * N + nc];
      }
  };
  if (skip) epi_fetch(skip, add);
  if (skg) epi_fetch(skg, add);
  if (xm) epi_fetch(xm, msk);
  if (bias) {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float bv = bias[row_of(i, r)];
#pragma unroll
        for (int j = 0; j < NI; ++j) add[i][j][r] += bv;
      }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      const int n = n0 + 16 * j + li;
      if (n >= N) continue;
      if (MODE == 2 && ps == 2) {
        // the gradient of output pixel (oy, ox) belongs to input pixel (2 oy, 2 ox); its neighbours took no part
        const int y = fdiv(n, iow), x = n - y * OW;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          gfloat* q = out + (size_t)row_of(i, r) * (size_t)(H * W) + 2 * (y * W + x);
          *(gv2*)q = (v2f){rbf_if(round, acc[i][j][r]), 0.f};
          *(gv2*)(q + W) = (v2f){0.f, 0.f};
        }
        continue;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float v = acc[i][j][r];
        if (MODE == 2 && !(msk[i][j][r] > 0.f)) v = 0.f;
        out[(size_t)row_of(i, r) * N + n] = rbf_if(round, v + add[i][j][r]);
      }
    }
}

template <int MODE>
__device__ __forceinline__ void step_d1(const LDesc& d, int tile, int t, lfloat* smem) {
  const int mi = UNI(d.g.mi), ni = UNI(d.g.ni);
  if (mi == 4) {
    if (ni == 4) step_d1_t<MODE, 4, 4>(d, tile, t, smem);
    else step_d1_t<MODE, 4, 1>(d, tile, t, smem);
  } else {
    if (ni == 4) step_d1_t<MODE, 1, 4>(d, tile, t, smem);
    else step_d1_t<MODE, 1, 1>(d, tile, t, smem);
  }
}

__device__ __forceinline__ void step_dc(const LDesc& d, int tile, int t, lfloat* smem, bool live) {
  const int gm = UNI(d.g.gm), mi = UNI(d.g.mi), ni = UNI(d.g.ni), s = UNI(d.stride);
  if (UNI(d.g.dc) == 2) {
    if (gm == 1) step_d1<1>(d, tile, t, smem);
    else step_d1<2>(d, tile, t, smem);
    return;
  }
  if (gm == 1) {
    if (mi == 4) step_dc_t<1, false, 4, 2>(d, tile, t, smem);
    else if (mi == 2 && ni == 2) step_dc_t<1, false, 2, 2>(d, tile, t, smem);
    else if (mi == 2) step_dc_t<1, false, 2, 1>(d, tile, t, smem);
    else step_dc_t<1, false, 1, 1>(d, tile, t, smem);
  } else if (gm == 2 && s == 1) {
    if (mi == 4) step_dc_t<2, false, 4, 2>(d, tile, t, smem);
    else if (mi == 2 && ni == 2) step_dc_t<2, false, 2, 2>(d, tile, t, smem);
    else if (mi == 2) step_dc_t<2, false, 2, 1>(d, tile, t, smem);
    else step_dc_t<2, false, 1, 1>(d, tile, t, smem);
  } else if (gm == 2) {
    if (mi == 2 && ni == 2) step_dc_t<2, true, 2, 2>(d, tile, t, smem);
    else if (mi == 2) step_dc_t<2, true, 2, 1>(d, tile, t, smem);
    else step_dc_t<2, true, 1, 1>(d, tile, t, smem);
  } else if (s == 1) {
    if (mi == 2) step_dcw_t<1, 2>(d, tile, t, smem, live);
    else step_dcw_t<1, 1>(d, tile, t, smem, live);
  } else {
    if (mi == 2) step_dcw_t<2, 2>(d, tile, t, smem, live);
    else step_dcw_t<2, 1>(d, tile, t, smem, live);
  }
}

}  // namespace pb
