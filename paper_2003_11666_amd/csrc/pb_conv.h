// 3x3 layers (padding 1, stride 1 or 2) of networks tiled for throughput: all three passes without offset tables and
// without a staged weight operand.
//
// The patch-based tiles of pb_gemm.h spend 55-60 % of their time outside the MFMA loop (12 requests per thread
// and chunk, the stores of both operands into LDS, two barriers) and read LDS once per MFMA, offsets on top.
// Here weights go from memory straight into registers and map values are read from a zero-padded patch in LDS, three
// taps of a row at fixed offsets from one address; a window read from LDS feeds MI products and a weight NI.
//
// Forward and backward data of layers that contract a multiple of 32 channels on 16 pixels and more (step_ds_t), and all
// weight gradients (step_dw_t), run on the bf16 matrix pipes with operands split into three pieces (pb_split.h); other
// channel counts and smaller maps on v_mfma_f32_16x16x4_f32 (step_dc_t).  Measured with fp32 MFMAs for all and with this:
// 512 ticks of the wide network 61.9 and 50.2 ms, 256 of ResNet-50 at 224 pixels 142.0 and 125.6; the loops over the
// chunks at 62-72 % and 100-160 % of the fp32 pipes' rate; error of the gradients against float64 (two basic networks, fixed
// weights) 1.81e-7 and 1.43e-7, 1.97e-7 and 1.41e-7.
//
// step_dc_t walks the reduction in blocks of 4 channels x 9 taps: lane group kq = lane / 16 supplies channel
// 4 b + kq in all nine MFMAs of block b, so
//   * a lane's nine weights of a block are the nine taps of one (output, input) channel pair, 36 contiguous bytes
//     in memory, forward and backward alike: they go straight into registers, one superblock ahead;
//   * its nine map values are a 3x3 window at a fixed lane offset into the patch: three row addresses, the columns are
//     immediate offsets.
// The patch is double buffered, the next chunk's 16-byte requests (rows whose length is no multiple of 4 included:
// unaligned loads, the tail masked on its way into LDS) are in flight while this one is contracted; one barrier per chunk.
//
// Backward data of a stride-2 layer runs over the gradient's pixels: the nine taps of a gradient pixel's window
// fall into the four parity classes of the 2x2 input pixels it belongs to (4, 2, 2 and 1 taps), one accumulator
// set each -- a quarter of the work of a gradient spread out with zeros.
//
// 1x1 layers on maps of fewer than 64 pixels (step_d1_t): both operands go straight from memory into registers, no LDS
// and no barrier; such a layer streams its weights and is bound by their way from memory.
//
// Included by pb_gemm.h.
#pragma once
#include "pb_device.h"

namespace pb {

// The end of a forward or backward-data tile: the waves' shares of the reduction added up, then the outputs.
template <int MODE, bool S2, int MI, int NI>
__device__ __forceinline__ void dc_finish(const LDesc& d, int t, lfloat* smem, v4f (&acc)[S2 ? 4 : 1][MI][NI], int wv, int wk, int wk_id, int wm_id, int wn_id,
                                          int qpart, int m0, int n0) {
  constexpr int NC = S2 ? 4 : 1;
  const int lane = (int)here(threadIdx.x) & 63, li = lane & 15, kq = lane >> 4;   // (no pixel index kept across the contraction)
  const int N = UNI(d.g.N), flags = UNI(d.flags), PWd = UNI((MODE == 1 || S2) ? d.OW : d.W);
  const float ipw = frcp(PWd);
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
  dc_finish<MODE, S2, MI, NI>(d, t, smem, acc, wv, wk, wk_id, wm_id, wn_id, qpart, m0, n0);
}

// Forward (MODE 1) and backward data (MODE 2) on the bf16 matrix pipes (pb_split.h), layers whose reduction runs over a
// multiple of 32 channels.
//
// An MFMA contracts 32 channels of one tap: lane group kq supplies channels kq, kq + 4, .. kq + 28 of a block of 32.  The
// patch is split on its way into LDS, [piece][octet][pixel][8 channels], octet kq of a block holding those eight: a lane's
// map values of one tap are one 16-byte read per piece, 16 neighbouring pixels' reads one 256-byte run.  A lane's weights of
// a block are the nine taps of eight channel pairs, requested, split and contracted a kernel row at a time, the next row's
// requests in flight beside the MFMAs of this one.  As the layer stores them a row is a 12-byte piece of a 36-byte run;
// where the layer's weight-gradient tiles store weights and predicted weights for this (PERM) it comes in runs of 1 KB.  The three taps of a
// kernel row (96 entries) are added up from zero, then join the accumulators.  One chunk of the patch in LDS.
template <int MODE, bool S2, bool PERM, int MI, int NI>
__device__ __forceinline__ void step_ds_t(const LDesc& d, int tile_, int t, lfloat* smem) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
  constexpr int NC = S2 ? 4 : 1;           // accumulator sets
  const int tid = threadIdx.x, lane = tid & 63, wv = UNI(tid >> 6), li = lane & 15, kq = lane >> 4;
  const int wk = UNI(d.g.wk), wn = UNI(d.g.wn);
  auto lg = [](int x) { return x == 1 ? 0 : (x == 2 ? 1 : 2); };
  const int wk_id = wv & (wk - 1), wn_id = (wv >> lg(wk)) & (wn - 1), wm_id = wv >> (lg(wk) + lg(wn));
  const int N = UNI(d.g.N), C = UNI(d.C);
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

  // ---- patch: patch row 0 is source row row0, source column x lies at patch column x + PAD.  A unit of a thread is four
  // pixels of four channels (of one octet); units of a chunk: CC / 4 x PR x W4
  constexpr int PAD = S2 ? 0 : 1;
  const float ipw = frcp(PWd);
  const int y0 = UNI(fdiv(n0, ipw)), row0 = S2 ? y0 : y0 * st - 1;
  const int piece = CC * plane / 2 + 4;    // floats of a piece: 16 bytes per pixel and octet, and one pixel that nobody reads
  const int cs = 4 * SH * SW;              // floats between two channels of a unit
  // (worked out again for every request and store: kept, they would cost registers across the contraction)
  const float irow = frcp(2 * W4), ioct = frcp(2 * W4 * PR);
  const int units = (CC >> 2) * PR * W4, passes = UNI((units + DS_VU * BLK - 1) / (DS_VU * BLK));
  auto unit = [&](int i, int& o, int& h, int& y, int& x) {
    o = fdiv(i, ioct);
    const int rem = i - o * 2 * W4 * PR;
    y = fdiv(rem, irow);
    const int xh = rem - y * 2 * W4;
    x = 4 * (xh >> 1);
    h = xh & 1;
    return i < units && row0 + y >= 0 && row0 + y < SH;
  };
  v4f pv[DS_VU][4];
  auto p_issue = [&](int ch, int pass) {
    const gfloat* s = src + (size_t)ch * (size_t)(CC * SH * SW);
#pragma unroll
    for (int u = 0; u < DS_VU; ++u) {
      int o, h, y, x;
      const bool ok = unit((int)here(tid) + (pass * DS_VU + u) * BLK, o, h, y, x);
      const unsigned b = ok ? 4u * (unsigned)(((32 * (o >> 2) + 16 * h + (o & 3)) * SH + row0 + y) * SW + x) : 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) pv[u][e] = *(const gv4u*)((const gbyte*)(s + e * cs) + b);
    }
  };
  // (no branch per pixel: what lies outside the map goes to the pixel behind the piece)
  auto p_commit = [&](int pass) {
#pragma unroll
    for (int u = 0; u < DS_VU; ++u) {
      int o, h, y, x;
      const bool ok = unit((int)here(tid) + (pass * DS_VU + u) * BLK, o, h, y, x);
      const int cnt = ok ? SW - x : 0, dst = 4 * (o * plane + y * Wp + x + PAD) + 2 * h;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        unsigned a[2], m[2], l[2];
        split2(pv[u][0][p], pv[u][1][p], a[0], m[0], l[0]);
        split2(pv[u][2][p], pv[u][3][p], a[1], m[1], l[1]);
        lfloat* q = smem + (p < cnt ? dst + 4 * p : piece - 4);
        *(lw2*)q = (v2w){a[0], a[1]};
        *(lw2*)(q + piece) = (v2w){m[0], m[1]};
        *(lw2*)(q + 2 * piece) = (v2w){l[0], l[1]};
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // ---- weights of a block of 32 channels: element e of a lane is channel 4 e + kq, row li
  const int nsb = UNI(CC / (32 * wk));                             // blocks per chunk and wave: wk_id, wk_id + wk, ...
  const int g_end = (ch_end - ch0) * nsb;
  const int blk0 = ch0 * (CC >> 5) + wk_id;                        // block g of the wave is blk0 + g wk
  const int row_s = MODE == 1 ? 9 * C : 9, red_s = MODE == 1 ? 9 : 9 * C;
  // (a lane's share of the address in bytes, the rest is scalar)
  const unsigned lane_b = PERM ? 16u * lane : 4u * ((unsigned)(li * row_s) + (unsigned)(kq * red_s));
  const int nb32 = (MODE == 1 ? C : UNI(d.K)) >> 5;                // blocks of the whole reduction
  const gfloat* Aw = PERM ? Ag + (size_t)(((m0 >> 4) + wm_id * MI) * nb32) * 4608 : Ag + (size_t)(m0 + wm_id * MI * 16) * row_s;
  // the weights of a kernel row as requested: three taps of eight channels per row subtile
  v3f wn_[PERM ? 1 : MI][8];
  v4f wp[PERM ? MI : 1][3][2];
  auto load_row = [&](int g, int kh) {
    const unsigned lb = here(lane_b);
    if constexpr (PERM) {
      const gfloat* o = Aw + (size_t)(blk0 + g * wk) * 4608 + 1536 * kh;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int x = 0; x < 6; ++x) wp[i][x >> 1][x & 1] = *(const gv4*)((const gbyte*)(o + (size_t)(i * nb32) * 4608 + 256 * x) + lb);
    } else {
      const gfloat* o = Aw + (size_t)(32 * (blk0 + g * wk)) * red_s + 3 * kh;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) wn_[i][e] = *(const gv3u*)((const gbyte*)(o + (size_t)(16 * i * row_s + 4 * e * red_s)) + lb);
    }
  };
  auto load_tap = [&](int g, int kh, int kw) {
    const unsigned lb = here(lane_b);
    const gfloat* o = Aw + (size_t)(blk0 + g * wk) * 4608 + 1536 * kh + 512 * kw;
#pragma unroll
    for (int i = 0; i < (PERM ? MI : 0); ++i)
#pragma unroll
      for (int x = 0; x < 2; ++x) wp[i][kw][x] = *(const gv4*)((const gbyte*)(o + (size_t)(i * nb32) * 4608 + 256 * x) + lb);
  };
  auto weight = [&](int i, int kw, int e) -> float {
    if constexpr (PERM) return wp[i][kw][e >> 2][e & 3];
    else return wn_[i][e][kw];
  };
  auto split_tap = [&](bf8 (&a)[MI][3], int kw) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      v4w h, m, l;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        unsigned h_, m_, l_;
        split2(weight(i, kw, 2 * e), weight(i, kw, 2 * e + 1), h_, m_, l_);
        h[e] = h_; m[e] = m_; l[e] = l_;
      }
      a[i][0] = __builtin_bit_cast(bf8, h);
      a[i][1] = __builtin_bit_cast(bf8, m);
      a[i][2] = __builtin_bit_cast(bf8, l);
    }
  };
  p_issue(ch0, 0);
  load_row(0, 0);
  // ---- lane offsets of the pixel subtiles' windows
  int poff[NI];
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    int n = n0 + (wn_id * NI + j) * 16 + li;
    n = n < N ? n : N - 1;
    const int y = fdiv(n, ipw), x = n - y * PWd;
    poff[j] = 4 * (kq * plane + (S2 ? (y - row0) * Wp + x : (y * st - 1 - row0) * Wp + x * st));
  }
  v4f acc[NC][MI][NI];
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j) acc[c][i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int i = tid; i < (3 * piece) >> 2; i += BLK) *(lv4*)(smem + 4 * i) = (v4f){0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  PB_TS(9);
  int g = 0;
  bf8 at_[MI][3];                          // PERM: the pieces of the tap at hand
  for (int ch = ch0; ch < ch_end; ++ch) {
    if (ch > ch0) {
      p_issue(ch, 0);
      __syncthreads();                     // every wave has contracted the chunk before
    }
    p_commit(0);
    for (int q = 1; q < passes; ++q) {
      p_issue(ch, q);
      p_commit(q);
    }
    __syncthreads();
    if constexpr (PERM) {
      // tap by tap: between the MFMAs of one tap the next one's weights are split (an MFMA keeps its pipe busy for four vector
      // instructions, 11 of which split a pair), those three taps on and the next map values are requested
      constexpr int NJ = NI < 2 ? NI : 2, NH = NI / NJ, STEPS = 6 * NH;
      if (ch == ch0) split_tap(at_, 0);
      for (int s = 0; s < nsb; ++s, ++g) {
        const lfloat* base = smem + 16 * (s * wk + wk_id) * plane;
        const int gn = g + 1 < g_end ? g + 1 : g;
        v4f z[MI][NI];
        bf8 an[MI][3], b[2][NJ][3];
        auto window = [&](bf8 (&r)[NJ][3], int tap, int half) {
          const int kh = tap / 3, kw = tap % 3;
          const int wy = S2 ? (kh == 0 ? 1 : 0) : MODE == 1 ? kh : 2 - kh, wx = S2 ? (kw == 0 ? 1 : 0) : MODE == 1 ? kw : 2 - kw;
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const lfloat* q = base + (int)here(poff[half * NJ + j]);
#pragma unroll
            for (int p = 0; p < 3; ++p) r[j][p] = __builtin_bit_cast(bf8, *(const lw4*)(q + (wy * Wp + p * (piece >> 2)) * 4 + 4 * wx));
          }
        };
        window(b[0], 0, 0);
        auto one_tap = [&](auto TAP, bf8 (&a)[MI][3], bf8 (&nx)[MI][3]) {
          constexpr int tap = decltype(TAP)::value, kh = tap / 3, kw = tap % 3;
          load_tap(kh < 2 ? g : gn, kh < 2 ? kh + 1 : 0, kw);
          v4w nh[MI], nm[MI], nl[MI];
#pragma unroll
          for (int half = 0; half < NH; ++half) {
            constexpr int first = tap * NH;
            bf8 (&bc)[NJ][3] = b[(first + half) & 1];
            if (first + half + 1 < 9 * NH) window(b[(first + half + 1) & 1], half + 1 < NH ? tap : tap + 1, half + 1 < NH ? half + 1 : 0);
            if (S2 || kw == 0) {
#pragma unroll
              for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) z[i][half * NJ + j] = (v4f){0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int q = 0; q < 6; ++q) {
#pragma unroll
              for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                  z[i][half * NJ + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][split_pa(q)], bc[j][split_pb(q)], z[i][half * NJ + j], 0, 0, 0);
#pragma unroll
              for (int u = 4 * MI * (6 * half + q) / STEPS; u < 4 * MI * (6 * half + q + 1) / STEPS; ++u) {
                const int i = u >> 2, e = u & 3;
                unsigned h_, m_, l_;
                split2(weight(i, (kw + 1) % 3, 2 * e), weight(i, (kw + 1) % 3, 2 * e + 1), h_, m_, l_);
                nh[i][e] = h_; nm[i][e] = m_; nl[i][e] = l_;
              }
              __builtin_amdgcn_sched_barrier(0);
            }
            if (S2 || kw == 2) {
              constexpr int cls = S2 ? (kh == 1 ? 0 : 2) + (kw == 1 ? 0 : 1) : 0;
#pragma unroll
              for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j) acc[cls][i][half * NJ + j] += z[i][half * NJ + j];
            }
          }
#pragma unroll
          for (int i = 0; i < MI; ++i) {
            nx[i][0] = __builtin_bit_cast(bf8, nh[i]);
            nx[i][1] = __builtin_bit_cast(bf8, nm[i]);
            nx[i][2] = __builtin_bit_cast(bf8, nl[i]);
          }
        };
        one_tap(IConst<0>(), at_, an); one_tap(IConst<1>(), an, at_); one_tap(IConst<2>(), at_, an);
        one_tap(IConst<3>(), an, at_); one_tap(IConst<4>(), at_, an); one_tap(IConst<5>(), an, at_);
        one_tap(IConst<6>(), at_, an); one_tap(IConst<7>(), an, at_); one_tap(IConst<8>(), at_, an);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int p = 0; p < 3; ++p) at_[i][p] = an[i][p];
      }
      continue;
    }
    for (int s = 0; s < nsb; ++s, ++g) {
      const lfloat* base = smem + 16 * (s * wk + wk_id) * plane;
#pragma unroll
      for (int kh = 0; kh < 3; ++kh) {
        bf8 a[3][MI][3];
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) split_tap(a[kw], kw);
        __builtin_amdgcn_sched_barrier(0);
        // the next kernel row's weights (the last one's again at the end)
        if (kh < 2) load_row(g, kh + 1);
        else load_row(g + 1 < g_end ? g + 1 : g, 0);
        // window row of the kernel row (stride 2 backward: kh = 0 row 1, odd input row; 1 row 0, even; 2 row 0, odd)
        const int wy = S2 ? (kh == 0 ? 1 : 0) : MODE == 1 ? kh : 2 - kh;
        static_assert(PERM || NI <= 2, "no registers for the sums and map values of four pixel subtiles beside a row's requests");
        v4f z[MI][NI];
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
          const int wx = S2 ? (kw == 0 ? 1 : 0) : MODE == 1 ? kw : 2 - kw;
          bf8 b[NI][3];
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const lfloat* q = base + (int)here(poff[j]);
#pragma unroll
            for (int p = 0; p < 3; ++p) b[j][p] = __builtin_bit_cast(bf8, *(const lw4*)(q + (wy * Wp + p * (piece >> 2)) * 4 + 4 * wx));
          }
          if (S2 || kw == 0) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
              for (int j = 0; j < NI; ++j) z[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
          for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
              for (int j = 0; j < NI; ++j)
                z[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[kw][i][split_pa(q)], b[j][split_pb(q)], z[i][j], 0, 0, 0);
          if (S2 || kw == 2) {
            const int cls = S2 ? (kh == 1 ? 0 : 2) + (kw == 1 ? 0 : 1) : 0;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
              for (int j = 0; j < NI; ++j) acc[cls][i][j] += z[i][j];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  PB_TS(10);
  if (wk > 1) __syncthreads();             // the waves' shares go where the patch lies
  dc_finish<MODE, S2, MI, NI>(d, t, smem, acc, wv, wk, wk_id, wm_id, wn_id, qpart, m0, n0);
}

// Backward weights on the bf16 matrix pipes (pb_split.h), stride S, MI row subtiles per wave.
//
// MFMA rows are output channels, columns 16 input channels, the reduction runs over pixels, rows padded to octets: an MFMA
// contracts four octets, lane group kq the one it is at.  The output gradient's octets come from memory as they lie, once for
// all nine taps.  The patch lies in LDS as [piece][channel][row][column], split on the way in, column x at bf16 8 + x of its
// row: the octet of the middle tap is an aligned 16-byte read, those of its neighbours are shifted in registers by one
// value (v_alignbit).  Stride 2: a row is its even and its odd columns one after the other.  The patch is double buffered,
// the next chunk's requests are in flight while this one is contracted; every 32 pixels are added up from zero.
// live: false before the layer's first gradient, when a step that updates the weights only carries them over.
template <int S, int MI>
__device__ __forceinline__ void step_dw_t(const LDesc& d, int tile_, int t, lfloat* smem, bool live) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
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
  const int PR = UNI(d.g.PR), row_f = UNI(d.g.Wp), plane = UNI(d.g.shw), W4 = UNI(d.g.sw), rows_c = UNI(d.g.rows_c);   // row_f, plane: floats
  const int n_chunks = UNI(d.g.n_chunks), ch0 = qpart * UNI(d.g.cpp);
  const int ch_end = !live ? ch0 : ch0 + UNI(d.g.cpp) < n_chunks ? ch0 + UNI(d.g.cpp) : n_chunks;
  const int noc = UNI(d.g.pw) >> 3;          // octets of an output row
  const int piece = CT * plane;
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
      pdst[u] = ok ? 2 * (c * plane + y * row_f + 4 + (S == 1 ? 2 * x : x)) | (x == W4 - 1 ? 1 : 0) : -1;
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
        lfloat* q = buf + (pdst[u] >> 1);
        unsigned h[2], m[2], l[2];
        if constexpr (S == 1) {
          split2(v[0], v[1], h[0], m[0], l[0]);
          split2(v[2], v[3], h[1], m[1], l[1]);
          *(lw2*)q = (v2w){h[0], h[1]};
          *(lw2*)(q + piece) = (v2w){m[0], m[1]};
          *(lw2*)(q + 2 * piece) = (v2w){l[0], l[1]};
        } else {
          split2(v[0], v[2], h[0], m[0], l[0]);
          split2(v[1], v[3], h[1], m[1], l[1]);
#pragma unroll
          for (int o = 0; o < 2; ++o) {
            lfloat* r = q + o * (row_f >> 1);
            *(lw1*)r = h[o];
            *(lw1*)(r + piece) = m[o];
            *(lw1*)(r + 2 * piece) = l[o];
          }
        }
      }
  };
  const float inoc = frcp(noc);
  const int nblk = (rows_c * noc + 3) >> 2;                        // blocks of four octets per chunk
  const int nmine = nblk > wk_id ? (nblk - wk_id + wk - 1) >> lg(wk) : 0;
  // block i of this wave in chunk ch: the lane's octet of gradient values per row subtile, zero outside the map
  auto load_a = [&](v4f (&r)[MI][2], int ch, int i) {
    const int e = 4 * (i * wk + wk_id) + kq, y = fdiv(e, inoc), x = 8 * (e - y * noc), oy = ch * rows_c + y;
    const bool ok = y < rows_c && oy < OH;
    const unsigned o = (unsigned)((m0 + li) * P + (ok ? oy * OW + x : 0)), o2 = ok && x + 4 < OW ? o + 4u : o;
#pragma unroll
    for (int k = 0; k < MI; ++k) {
      r[k][0] = *(const gv4u*)(dy + (o + (unsigned)(16 * k * P)));
      r[k][1] = *(const gv4u*)(dy + (o2 + (unsigned)(16 * k * P)));
#pragma unroll
      for (int u = 0; u < 8; ++u) r[k][u >> 2][u & 3] = (ok && x + u < OW) ? r[k][u >> 2][u & 3] : 0.f;
    }
  };
  auto b_off = [&](int i) {
    const int e = 4 * (i * wk + wk_id) + kq;
    int y = fdiv(e, inoc);
    const int x = e - y * noc;
    y = y < rows_c ? y : rows_c - 1;
    return (wn_id * 16 + li) * plane + y * S * row_f + 4 * x + 4;  // floats: the octet of the middle column
  };
  v4f acc[MI][9];
#pragma unroll
  for (int k = 0; k < MI; ++k)
#pragma unroll
    for (int j = 0; j < 9; ++j) acc[k][j] = (v4f){0.f, 0.f, 0.f, 0.f};
  p_issue(ch0);
  v4f ar[MI][2];
  load_a(ar, ch0, 0);
  const int buf_fl = 3 * piece;
  for (int i = tid; i < (2 * buf_fl + 16) >> 2; i += BLK) *(lv4*)(smem + 4 * i) = (v4f){0.f, 0.f, 0.f, 0.f};
  __syncthreads();
  p_commit(smem);
  __syncthreads();                           // (a step that is not live yet contracts nothing)
  PB_TS(9);
  for (int ch = ch0; ch < ch_end; ++ch) {
    const lfloat* cur = smem + ((ch - ch0) & 1) * buf_fl;
    lfloat* nxt = smem + (((ch - ch0) & 1) ^ 1) * buf_fl;
    const bool more = ch + 1 < ch_end;
    if (more) p_issue(ch + 1);
    for (int i = 0; i < nmine; ++i) {
      bf8 a[MI][3];
#pragma unroll
      for (int k = 0; k < MI; ++k) {
        v4w h, m, l;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          unsigned h_, m_, l_;
          split2(ar[k][e >> 1][2 * (e & 1)], ar[k][e >> 1][2 * (e & 1) + 1], h_, m_, l_);
          h[e] = h_; m[e] = m_; l[e] = l_;
        }
        a[k][0] = __builtin_bit_cast(bf8, h);
        a[k][1] = __builtin_bit_cast(bf8, m);
        a[k][2] = __builtin_bit_cast(bf8, l);
      }
      const bool end = i + 1 >= nmine;
      load_a(ar, end && more ? ch + 1 : ch, end ? 0 : i + 1);
      const lfloat* p = cur + b_off(i);
#pragma unroll
      for (int kh = 0; kh < 3; ++kh) {
        bf8 b[3][3];                         // [column of the kernel][piece]
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const lfloat* r = p + (kh * row_f + q * piece);
          v4w lo, mid, hi;
          if constexpr (S == 1) {
            mid = *(const lw4*)r;
            const unsigned before = *(const lw1*)(r - 1), after = *(const lw1*)(r + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              lo[e] = __builtin_amdgcn_alignbit(mid[e], e == 0 ? before : mid[e > 0 ? e - 1 : 0], 16);
              hi[e] = __builtin_amdgcn_alignbit(e == 3 ? after : mid[e < 3 ? e + 1 : 3], mid[e], 16);
            }
          } else {
            mid = *(const lw4*)r;                                  // even columns
            hi = *(const lw4*)(r + (row_f >> 1));                  // odd columns
            const unsigned before = *(const lw1*)(r + (row_f >> 1) - 1);
#pragma unroll
            for (int e = 0; e < 4; ++e) lo[e] = __builtin_amdgcn_alignbit(hi[e], e == 0 ? before : hi[e > 0 ? e - 1 : 0], 16);
          }
          b[0][q] = __builtin_bit_cast(bf8, lo);
          b[1][q] = __builtin_bit_cast(bf8, mid);
          b[2][q] = __builtin_bit_cast(bf8, hi);
        }
        __builtin_amdgcn_sched_barrier(0);
        v4f z[MI][3];
#pragma unroll
        for (int k = 0; k < MI; ++k)
#pragma unroll
          for (int x = 0; x < 3; ++x) z[k][x] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
          for (int x = 0; x < 3; ++x)
#pragma unroll
            for (int k = 0; k < MI; ++k)
              z[k][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[k][split_pa(q)], b[x][split_pb(q)], z[k][x], 0, 0, 0);
#pragma unroll
        for (int k = 0; k < MI; ++k)
#pragma unroll
          for (int x = 0; x < 3; ++x) acc[k][3 * kh + x] += z[k][x];
      }
    }
    if (nmine == 0 && more) load_a(ar, ch + 1, 0);
    if (more) p_commit(nxt);
    __syncthreads();
  }
  PB_TS(10);
  // ---- the waves' shares of the reduction, in order
  const int flags = UNI(d.flags);
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
  // the tile's gradients go through LDS, behind the waves' shares: 2304 MI floats for all four waves' shares and sums
  // together, 4 more per row
  const int pitch = 9 * CT + 4, MT = UNI(d.g.MT), mt0 = tm * MT;
  lfloat* T = smem + (wk > 1 ? (4 - (4 >> lg(wk))) * MI * 9 * 256 : 0);
  auto stage = [&]() {
    if (wk_id != 0) return;
#pragma unroll
    for (int k = 0; k < MI; ++k)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lfloat* q = T + ((wm_id * MI + k) * 16 + 4 * kq + r) * pitch + (wn_id * 16 + li) * 9;
#pragma unroll
        for (int e = 0; e < 9; ++e) q[e] = acc[k][e][r];
      }
  };
  if (flags & F_UPD_W) {
    // the update of the tile's weights: no gradient in memory (8 bytes per weight and a launch's tail saved)
    const bool perm = flags & F_WHAT_PERM;
    if (flags & F_W_PERM) tile_update_lanes<4>(d, T, pitch, MT >> 4, lg(wn), mt0, c0, stage);
    else tile_update<4>(d, T, pitch, MT, 9 * CT / 4, (unsigned)(mt0 * C + c0) * 9u, 9u * (unsigned)C, perm, stage);
    if (perm) {
      // the predicted weights in the order of the forward tiles' lanes
      __syncthreads();
      if (flags & F_WHAT_P32) {
        // (step_ds_t: 64 lanes x 4 channels per tap, 16 rows and 16 channels)
        const int np = 9 * (MT >> 4) * wn;
        for (int p = wv; p < np; p += 4) {
          const int g = UNI(fdiv(p, 1.f / 9.f)), tap = p - 9 * g, rt = g >> lg(wn), cg = g & (wn - 1), ca = c0 + 16 * cg;
          const lfloat* q = T + (16 * rt + li) * pitch + (16 * cg + kq) * 9 + tap;
          gfloat* o = GP(d.what) + (size_t)((((unsigned)((mt0 >> 4) + rt) * (unsigned)(C >> 5) + (unsigned)(ca >> 5)) * 9u + (unsigned)tap) * 2u + (unsigned)((ca >> 4) & 1)) * 256u + 4 * lane;
          *(gv4*)o = (v4f){q[0], q[36], q[72], q[108]};
        }
      } else {
        // (step_dc_t: 16 threads per block of 16 rows x 4 channels)
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
    }
    return;
  }
  // the gradients, by the same way through LDS: whole vectors instead of 36-byte segments
  stage();
  __syncthreads();
  gfloat* out = GP(d.gw) + (size_t)qpart * (size_t)UNI(d.gpstride);
  const int cv = 9 * CT / 4, total = MT * cv;
  const float icv = frcp(cv);
  for (int i = tid; i < total; i += BLK) {
    const int r = fdiv(i, icv), c = i - r * cv;
    *(gv4*)(out + (unsigned)((mt0 + r) * C + c0) * 9u + (unsigned)(4 * c)) = *(const lv4*)(T + r * pitch + 4 * c);
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

template <int MODE, bool S2, bool PERM>
__device__ __forceinline__ void step_ds_mn(const LDesc& d, int tile, int t, lfloat* smem) {
  const int mi = UNI(d.g.mi), ni = UNI(d.g.ni);
  if constexpr (!S2) {                       // (stride 2 backward has four accumulator sets)
    if (mi == 2) {
      if constexpr (PERM) {
        if (ni == 4) { step_ds_t<MODE, S2, PERM, 2, 4>(d, tile, t, smem); return; }
      }
      if (ni == 2) step_ds_t<MODE, S2, PERM, 2, 2>(d, tile, t, smem);
      else step_ds_t<MODE, S2, PERM, 2, 1>(d, tile, t, smem);
      return;
    }
  }
  if (ni == 2) step_ds_t<MODE, S2, PERM, 1, 2>(d, tile, t, smem);
  else step_ds_t<MODE, S2, PERM, 1, 1>(d, tile, t, smem);
}

__device__ __forceinline__ void step_dc(const LDesc& d, int tile, int t, lfloat* smem, bool live) {
  const int gm = UNI(d.g.gm), mi = UNI(d.g.mi), ni = UNI(d.g.ni), s = UNI(d.stride);
  if (UNI(d.g.dc) == 2) {
    if (gm == 1) step_d1<1>(d, tile, t, smem);
    else step_d1<2>(d, tile, t, smem);
    return;
  }
  if (gm == 3) {
    if (s == 1) {
      if (mi == 2) step_dw_t<1, 2>(d, tile, t, smem, live);
      else step_dw_t<1, 1>(d, tile, t, smem, live);
    } else {
      if (mi == 2) step_dw_t<2, 2>(d, tile, t, smem, live);
      else step_dw_t<2, 1>(d, tile, t, smem, live);
    }
    return;
  }
  if (UNI(d.g.dc) == 3) {
    if (gm == 1) {
      if (UNI(d.flags) & F_WHAT_PERM) step_ds_mn<1, false, true>(d, tile, t, smem);
      else step_ds_mn<1, false, false>(d, tile, t, smem);
    } else if (s == 1) {
      if (UNI(d.flags) & F_W_PERM) step_ds_mn<2, false, true>(d, tile, t, smem);
      else step_ds_mn<2, false, false>(d, tile, t, smem);
    } else {
      if (UNI(d.flags) & F_W_PERM) step_ds_mn<2, true, true>(d, tile, t, smem);
      else step_ds_mn<2, true, false>(d, tile, t, smem);
    }
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
  }
}

}  // namespace pb
