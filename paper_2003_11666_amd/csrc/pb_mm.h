// Dense matrix-product core for the 1x1 layers of networks tiled for
// throughput (fp32 operands and results, split for the bf16 matrix pipes: pb_split.h).
//
// A 1x1 layer of stride 1 on one sample is a plain matrix product over the flattened map:
//   forward           Y[K x P]  = W[K x C] * X[C x P]
//   backward data     dX[C x P] = W^T[C x K] * dY[K x P]
//   backward weights  gW[K x C] = dY[K x P] * X^T[P x C]
// with P pixels and all three matrices row-major in memory.  There is no patch
// and no offset table: the operands of a chunk of 32 reduction entries are split
// into their three pieces on the way into LDS, [piece][row or column][32 entries],
// once per workgroup, and a wave keeps a register tile of MI x NI 16x16 accumulators
// (a workgroup of 2 x 2 waves: 32 MI rows, 32 NI columns), so that an operand read
// from LDS feeds MI or NI products and a float fetched from memory is used 32 MI
// (32 NI) times.  A lane's eight entries of an MFMA are one 16-byte LDS read; the
// 16-byte units of a row are exchanged by (row / 4) mod 4, so that 16 rows lie on
// different banks.  The requests of chunk c + 1 are in flight while chunk c is
// contracted; LDS holds two chunks, or one where the tile is 128 x 128 (48 KB).
// Measured with the tiles of the fp32 pipes before and these: 256 ticks of ResNet-50 at 224 pixels 151.7 and 142.0 ms, 384
// of its stages at 64 pixels 88.6 and 85.4; the gradients' error against float64 (two networks of bottleneck blocks, fixed
// weights) 5.8e-7 and 4.7e-7, 4.3e-7 and 3.6e-7.
//
// An operand whose rows run along the reduction (W forward, dY and X backward
// weights) goes into LDS as it is requested, four entries of a row per thread.  One
// whose rows run along rows or columns of the result is transposed in registers: a
// thread requests four columns (rows) of four consecutive entries.  These columns go
// to LDS rows 32 apart, so that the writes spread over the banks, and so that a lane
// of the result holds NI neighbouring columns (MI neighbouring rows backward data).
//
// Operands that cannot be copied 16 bytes at a time -- the input of a projection of
// stride 2 -- are gathered element by element; the geometry is that of a general k x k
// layer (reduction or columns over (channel, tap)), which the planner uses for k > 1
// only on request: a tap-by-tap gather fetches nine times what a patch in LDS serves once.
// Rows of no multiple of 4 pixels are requested with unaligned vectors that reach up to
// three floats past the last row.
//
// Included by pb_gemm.h.
#pragma once
#include "pb_device.h"

namespace pb {

template <int MODE, int MI, int NI>
__device__ __forceinline__ void step_mm_t(const LDesc& d, int tile_, int t, lfloat* smem, bool live) {
  int tile = tile_;
  asm volatile("" : "+s"(tile));
  constexpr int MT = 32 * MI, NT = 32 * NI;
  constexpr int NBUF = mm_buffers(MT, NT), CHUNK = mm_chunk_floats(MT, NT);
  constexpr int APL = 16 * MT, BPL = 16 * NT;      // floats (pairs of bf16) per piece
  constexpr bool A_ALONG = MODE != 2, B_ALONG = MODE == 3;   // the operand's rows run along the reduction
  const int tid = threadIdx.x, lane = tid & 63, wv = UNI(tid >> 6);
  const int wr = wv >> 1, wc = wv & 1, li = lane & 15, kq = lane >> 4;
  const int M = UNI(d.g.M), N = UNI(d.g.N), Q = UNI(d.g.Q);
  const int flags = UNI(d.flags);
  const int tiles_n = UNI(d.g.tiles_n);
  int qpart = 0;
  if (MODE == 3) {
    const int tpp = UNI(d.g.tpp);
    qpart = UNI(fdiv(tile, frcp(tpp)));
    tile -= qpart * tpp;
  }
  const int tm = UNI(fdiv(tile, frcp(tiles_n))), tn = tile - tm * tiles_n;
  const int m0 = tm * MT, n0 = tn * NT;
  const int n_chunks = UNI(d.g.n_chunks);
  const int ch0 = MODE == 3 ? qpart * UNI(d.g.cpp) : 0;
  // (live: false before the layer's first gradient, when a step that updates the weights only carries them over)
  const int ch_end = (MODE == 3 && !live) ? ch0 : (MODE == 3 && ch0 + UNI(d.g.cpp) < n_chunks) ? ch0 + UNI(d.g.cpp) : n_chunks;

  // forward: A = W[M][Q] rows m0.., B = X[Q][N] columns n0..
  // backward data: A^T = W[Q][M] columns m0.., B = dY[Q][N] columns n0..
  // backward weights: A = dY[M][Q] rows m0.., B^T = X[N][Q] rows n0..
  const gfloat* Ag = MODE == 3 ? (const gfloat*)at(d.dy, t) : GP(d.w);
  const gfloat* Bg = MODE == 2 ? (const gfloat*)at(d.dy, t) : (const gfloat*)at(d.x, t);
  // Gathered operands: dense pixel p lies at poff(p) inside its channel's map, channels shw floats apart.
  const int gather = UNI(d.g.gather), ps = UNI(d.g.ps), pw = UNI(d.g.pw), sw = UNI(d.g.sw), shw = UNI(d.g.shw);
  const float ipw = frcp(pw);
  constexpr int AV = MT * MM_QC / 4 / BLK;     // 16-byte requests per thread and chunk: A
  constexpr int BV = NT * MM_QC / 4 / BLK;     //                                        B
  v4f ra[AV], rb[BV];
  // Convolution geometry of the gathered operands.  A k x k layer is the same product with the reduction (forward)
  // or the columns (backward weights) running over (channel, tap): the element for tap (kh, kw) and pixel (y, x) of the
  // output lies at row ps y + kh - pad, column ps x + kw - pad of the source map, and is zero outside the map.
  const int ck = UNI(d.g.ck), kk = ck * ck, cpad = UNI(d.g.cpad), srcH = UNI(d.g.sh);
  const float ikk = frcp(kk), ick = frcp(ck);
  auto tap_of = [&](int q, int& c, int& dy, int& dx) {
    c = fdiv(q, ikk);
    const int tap = q - c * kk, kh = fdiv(tap, ick);
    dy = kh - cpad;
    dx = tap - kh * ck - cpad;
  };
  auto pix_of = [&](int p, int& y, int& x) {
    y = fdiv(p, ipw);
    x = (p - y * pw) * ps;
    y *= ps;
  };
  // (a load from a clamped position and a select: no branch between two loads)
  auto src_at = [&](const gfloat* base, int c, int y, int x, bool ok) -> float {
    const bool in = ok && y >= 0 && y < srcH && x >= 0 && x < sw;
    const float v = base[(unsigned)(in ? c * shw + y * sw + x : 0)];   // (unsigned: a 32-bit offset from a scalar base)
    return in ? v : 0.f;
  };
  // rows along the reduction: vector v of a thread is entries 4 (v mod 8) .. + 3 of row v / 8
  auto issue_along = [&](const gfloat* g, auto& r, int row0, int q0) {
    constexpr int V = sizeof(r) / sizeof(r[0]);
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int v = tid + u * BLK, row = v >> 3, q = q0 + 4 * (v & 7);
      r[u] = (v4f){0.f, 0.f, 0.f, 0.f};
      if (q < Q) r[u] = *(const gv4u*)(g + (unsigned)((row0 + row) * Q + q));
    }
  };
  // Entries past the end of a row belong to the next one.  They are cleared on the way into LDS, in the last chunk: a select
  // behind each request waits for it before the next one goes out (529 pixels, tile of 128 x 64: 17 chunks in 61 us).
  auto clear_tail = [&](auto& r, int q0) {
    constexpr int V = sizeof(r) / sizeof(r[0]);
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int q = q0 + 4 * ((tid + u * BLK) & 7);
#pragma unroll
      for (int e = 1; e < 4; ++e) r[u][e] = q + e < Q ? r[u][e] : 0.f;
    }
  };
  // rows along the result: vector u of a thread is four columns of entry V kb + u
  auto issue_across = [&](const gfloat* g, auto& r, int col0, int cols, int q0) {
    constexpr int V = sizeof(r) / sizeof(r[0]), C4 = 8 * V;
    const int col = col0 + 4 * (tid % C4), k0 = V * (tid / C4);
#pragma unroll
    for (int u = 0; u < V; ++u) {
      r[u] = (v4f){0.f, 0.f, 0.f, 0.f};
      if (col < cols) r[u] = *(const gv4u*)(g + (unsigned)((q0 + k0 + u) * cols + col));
    }
  };
  auto issue = [&](int ch) {
    const int q0 = ch * MM_QC;
    if (A_ALONG) issue_along(Ag, ra, m0, q0);
    else issue_across(Ag, ra, m0, M, q0);
    if (!gather) {
      if (B_ALONG) issue_along(Bg, rb, n0, q0);
      else issue_across(Bg, rb, n0, N, q0);
    } else if (MODE == 3) {
#pragma unroll
      for (int u = 0; u < BV; ++u) {
        const int v = tid + u * BLK, p = q0 + 4 * (v & 7);
        int c, dy, dx;
        tap_of(n0 + (v >> 3), c, dy, dx);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          int y, x;
          pix_of(p + e < Q ? p + e : 0, y, x);
          rb[u][e] = src_at(Bg, c, y + dy, x + dx, p + e < Q);
        }
      }
    } else {
      // a thread keeps one column: neighbouring lanes read neighbouring pixels
      const int p = n0 + tid % NT, k0 = 4 * BV * (tid / NT);
      int y, x;
      pix_of(p < N ? p : 0, y, x);
#pragma unroll
      for (int i = 0; i < 4 * BV; ++i) {
        int c, dy, dx;
        tap_of(q0 + k0 + i, c, dy, dx);
        rb[i >> 2][i & 3] = src_at(Bg, c, y + dy, x + dx, p < N);
      }
    }
  };
  // LDS: A pieces | B pieces; entries 4 q .. 4 q + 3 of a row
  auto at_quad = [&](lfloat* op, int row, int q) { return op + 16 * row + 4 * ((q >> 1) ^ ((row >> 2) & 3)) + 2 * (q & 1); };
  auto put_quad = [&](lfloat* op, int pl, int row, int q, v4f x) {
    unsigned h[2], m[2], l[2];
    split2(x[0], x[1], h[0], m[0], l[0]);
    split2(x[2], x[3], h[1], m[1], l[1]);
    lfloat* p = at_quad(op, row, q);
    *(lw2*)p = (v2w){h[0], h[1]};
    *(lw2*)(p + pl) = (v2w){m[0], m[1]};
    *(lw2*)(p + 2 * pl) = (v2w){l[0], l[1]};
  };
  auto commit_along = [&](lfloat* op, int pl, auto& r) {
    constexpr int V = sizeof(r) / sizeof(r[0]);
#pragma unroll
    for (int u = 0; u < V; ++u) {
      const int v = tid + u * BLK;
      put_quad(op, pl, v >> 3, v & 7, r[u]);
    }
  };
  // column c of the tile goes to LDS row 32 (c mod V) + c / V  (V = NI, or MI)
  auto commit_across = [&](lfloat* op, int pl, auto& r) {
    constexpr int V = sizeof(r) / sizeof(r[0]), C4 = 8 * V;
    const int c4 = tid % C4, kb = tid / C4;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int row = 32 * (j % V) + (4 * c4 + j) / V;
      if constexpr (V == 4) {
        put_quad(op, pl, row, kb, (v4f){r[0][j], r[1][j], r[2][j], r[3][j]});
      } else {
        unsigned h, m, l;
        split2(r[0][j], r[1][j], h, m, l);
        lfloat* p = at_quad(op, row, kb >> 1) + (kb & 1);
        *(lw1*)p = h;
        *(lw1*)(p + pl) = m;
        *(lw1*)(p + 2 * pl) = l;
      }
    }
  };
  auto commit = [&](lfloat* buf) {
    lfloat* Bl = buf + 3 * APL;
    if (A_ALONG) commit_along(buf, APL, ra);
    else commit_across(buf, APL, ra);
    if (B_ALONG) {
      commit_along(Bl, BPL, rb);
    } else if (gather) {
      const int c = tid % NT;
#pragma unroll
      for (int u = 0; u < BV; ++u) put_quad(Bl, BPL, 32 * (c % NI) + c / NI, BV * (tid / NT) + u, rb[u]);
    } else {
      commit_across(Bl, BPL, rb);
    }
  };

  v4f acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = (v4f){0.f, 0.f, 0.f, 0.f};

  // LDS rows of the wave's subtiles: 16 consecutive ones each
  auto sub_a = [&](int i) { return A_ALONG ? 16 * (wr * MI + i) : 32 * i + 16 * wr; };
  auto sub_b = [&](int j) { return B_ALONG ? 16 * (wc * NI + j) : 32 * j + 16 * wc; };
  const int un = 4 * (kq ^ ((li >> 2) & 3));       // (16 rows: the exchange of units depends on the lane alone)
  issue(ch0);
  for (int ch = ch0; ch < ch_end; ++ch) {
    lfloat* buf = smem + (NBUF > 1 ? ((ch - ch0) & 1) * CHUNK : 0);
    if (NBUF == 1) __syncthreads();                // every wave has contracted the chunk before
    if (MODE == 3 && (Q & 3) && (ch + 1) * MM_QC > Q) {
      clear_tail(ra, ch * MM_QC);
      if (!gather) clear_tail(rb, ch * MM_QC);
    }
    commit(buf);
    __syncthreads();
    if (ch + 1 < ch_end) issue(ch + 1);
    __builtin_amdgcn_sched_barrier(0);
    const lfloat* Al = buf + 16 * li + un;
    const lfloat* Bl = Al + 3 * APL;
    bf8 a[MI][3], b[2][3];
#pragma unroll
    for (int p = 0; p < 3; ++p) b[0][p] = __builtin_bit_cast(bf8, *(const lw4*)(Bl + p * BPL + 16 * sub_b(0)));
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int p = 0; p < 3; ++p) a[i][p] = __builtin_bit_cast(bf8, *(const lw4*)(Al + p * APL + 16 * sub_a(i)));
#pragma unroll
    for (int j = 0; j < NI; ++j) {
      if (j + 1 < NI) {
#pragma unroll
        for (int p = 0; p < 3; ++p) b[(j + 1) & 1][p] = __builtin_bit_cast(bf8, *(const lw4*)(Bl + p * BPL + 16 * sub_b(j + 1)));
      }
      __builtin_amdgcn_sched_barrier(0);
      v4f z[MI];
      split_products<MI>(z, a, b[j & 1]);
#pragma unroll
      for (int i = 0; i < MI; ++i) acc[i][j] += z[i];
    }
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- epilogue: accumulator element r of subtile (i, j) is row row_of(i, r), column col0 + j
  // (backward weights: columns 16 apart)
  int te = t;
  asm volatile("" : "+s"(te));
  gfloat* out = MODE == 3 ? GP(d.gw) + (size_t)qpart * (size_t)UNI(d.gpstride) : MODE == 2 ? at(d.dx, te) : at(d.y, te);
  auto row_of = [&](int i, int r) { return m0 + (A_ALONG ? 16 * (wr * MI + i) + 4 * kq + r : MI * (16 * wr + 4 * kq + r) + i); };
  if constexpr (MODE == 3) {
    if (flags & F_UPD_W) {
      // the update of the tile's weights: no gradient in memory
      constexpr int pitch = NT + 4;
      __syncthreads();                             // every wave is done with its operands
      tile_update<4>(d, smem, pitch, MT, NT / 4, (unsigned)m0 * (unsigned)N + (unsigned)n0, (unsigned)N, false, [&]() {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) smem[(row_of(i, r) - m0) * pitch + 16 * (wc * NI + j) + li] = acc[i][j][r];
      });
      return;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NI; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(unsigned)(row_of(i, r) * N + n0 + 16 * (wc * NI + j) + li)] = acc[i][j][r];
    return;
  } else {
    typedef float vn __attribute__((ext_vector_type(NI), aligned(4)));
    typedef __attribute__((address_space(1))) vn gvn;
    const int col0 = n0 + NI * (16 * wc + li);
    const gfloat* skip = (MODE == 1 && (flags & F_SKIP)) ? (const gfloat*)at(d.skip, te) : nullptr;
    const gfloat* bias = (MODE == 1 && (flags & F_BIAS)) ? GP(d.b) : nullptr;
    const gfloat* xm = (MODE == 2 && (flags & F_MASK_X)) ? (const gfloat*)at(d.x, te) : nullptr;
    const gfloat* skg = (MODE == 2 && (flags & F_ADD_SKG)) ? (const gfloat*)at(d.skg, te) : nullptr;
    const bool round = flags & F_BF16_OUT;
    // every operand of the epilogue is requested before the first one is used (the registers of the
    // contraction's operands are free by now): one memory round trip for the whole tile.  Straight-line loads from
    // clamped addresses: a branch per element would make every load wait for the one before.
    const bool whole = N % NI == 0;                // a lane's columns all lie in the map or all outside
    const int colc = col0 < N ? col0 : 0;
    float add[MI][4][NI], msk[MI][4][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < NI; ++j) { add[i][r][j] = 0.f; msk[i][r][j] = 1.f; }
    auto epi_fetch = [&](const gfloat* src, float (&dst)[MI][4][NI]) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const gfloat* p = src + (unsigned)(row_of(i, r) * N);
          if (whole) {
            const vn x = *(const gvn*)(p + colc);
#pragma unroll
            for (int j = 0; j < NI; ++j) dst[i][r][j] = x[j];
          } else {
#pragma unroll
            for (int j = 0; j < NI; ++j) dst[i][r][j] = p[colc + j < N ? colc + j : N - 1];
          }
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
          for (int j = 0; j < NI; ++j) add[i][r][j] += bv;
        }
    }
    if (MODE == 2 && ps == 2) {
      // backward data of a layer of stride 2: the gradient of dense pixel (oy, ox) belongs to input pixel (2 oy, 2 ox);
      // its three neighbours in the 2 x 2 block took no part in the forward pass
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int col = col0 + j, oy = fdiv(col, ipw), o = (oy * sw + (col - oy * pw)) * ps;
        if (col >= N) continue;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            gfloat* q = out + (size_t)row_of(i, r) * shw + o;
            *(gv2*)q = (v2f){rbf_if(round, acc[i][j][r]), 0.f};
            *(gv2*)(q + sw) = (v2f){0.f, 0.f};
          }
      }
      return;
    }
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        gfloat* p = out + (unsigned)(row_of(i, r) * N);
        vn x;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          float v = acc[i][j][r];
          if (MODE == 2 && !(msk[i][r][j] > 0.f)) v = 0.f;
          x[j] = rbf_if(round, v + add[i][r][j]);
        }
        if (whole) {
          if (col0 < N) *(gvn*)(p + col0) = x;
        } else {
#pragma unroll
          for (int j = 0; j < NI; ++j)
            if (col0 + j < N) p[col0 + j] = x[j];
        }
      }
  }
}

__device__ __forceinline__ void step_mm(const LDesc& d, int tile, int t, lfloat* smem, bool live) {
  // forward and backward data: tiles of 128 x 128, 64 x 128 (layers of 64 channels) or 128 x 64 (maps of at most 64 pixels)
  const int gm = UNI(d.g.gm), mi = UNI(d.g.mi), ni = UNI(d.g.ni);
  if (gm == 1) {
    if (mi == 4 && ni == 4) step_mm_t<1, 4, 4>(d, tile, t, smem, live);
    else if (mi == 4) step_mm_t<1, 4, 2>(d, tile, t, smem, live);
    else step_mm_t<1, 2, 4>(d, tile, t, smem, live);
  } else if (gm == 2) {
    if (mi == 4 && ni == 4) step_mm_t<2, 4, 4>(d, tile, t, smem, live);
    else if (mi == 4) step_mm_t<2, 4, 2>(d, tile, t, smem, live);
    else step_mm_t<2, 2, 4>(d, tile, t, smem, live);
  } else {
    if (mi == 4 && ni == 4) step_mm_t<3, 4, 4>(d, tile, t, smem, live);
    else if (mi == 4) step_mm_t<3, 4, 2>(d, tile, t, smem, live);
    else if (ni == 4) step_mm_t<3, 2, 4>(d, tile, t, smem, live);
    else step_mm_t<3, 2, 2>(d, tile, t, smem, live);
  }
}

}  // namespace pb
