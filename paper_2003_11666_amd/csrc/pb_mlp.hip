// A perceptron's pipeline with the parameters in registers.
//
// Every stage of a perceptron is a matrix-vector layer on one sample: a tick moves each weight and velocity once and
// multiplies it three times, so as launches of the phase kernel it is bound by what surrounds the arithmetic -- launches,
// descriptors, memory round trips (14.9 us a tick for 64-128-128-128-10) -- or, with wide layers, by the memory traffic of
// weights, velocities, gradients and predicted weights (89 us a tick for four 1024 x 1024 layers).  But the weights and
// velocities of such a network fit the register files: 512 KB per compute unit.  Here a workgroup owns 8 RW consecutive
// rows of one stage for the whole launch, wavefront w the rows w RW .. w RW + RW - 1, lane l the columns l, l + 64, ...;
// parameters are read when the launch starts and written when it ends, and between the ticks only activations and
// gradients move: a few KB.  Measured: 1000 ticks of 64-128-128-128-10 15.3 -> 2.1 ms; 256 ticks of 1024-1024-1024-1024-1024-100
// with the read-back of 34 MB 28.3 -> 3.0 ms; 16 ticks of the small one fed by the host, one launch each, 0.48 -> 0.19 ms.
// A small tick is a chain of dependent instructions between two messages (a hop takes 0.35-0.5 us of its 2.1): no division
// by a run-time value in it, labels in LDS, the softmax in registers, the loss after the messages, and only wavefronts that
// take messages wait for them (with all that inside the chain the 1000 ticks took 3.1 ms).
//
// A tick of a workgroup: take the stage's input (from all workgroups of the previous stage) and the gradient of its own
// rows (one partial value from every workgroup of the next stage, added in order), forward rows out, backward columns out,
// then the update, which overlaps the messages' way.  The last stage runs forward, loss and backward in the same tick.
//
// Messages are 8-byte words (value, tick + 1) written and read with agent-scope atomics: the word is its own flag, so one
// hop costs one store and one load through memory, without cache-wide releases.  Two words per value, by parity of the
// tick, are enough: a workgroup finishes tick t only after every workgroup of both neighbours has published tick t - 1,
// i.e. has consumed what it was sent for tick t - 1.  (They publish in every tick, zeros while the pipeline fills.)
// The waits need all workgroups resident: one per compute unit, never more than the GPU has, and the host keeps launches
// of several contexts and processes apart (WaitDevice in pb_host.cpp).  A wait is bounded by the clock (4 s); on expiry the error word is set and the grid drains.
#include "pb_device.h"
#include "pb_mlp.h"
#include "pb_wave.h"

#include <type_traits>

namespace pb {

typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) uint64_t gmsg;
typedef __attribute__((address_space(1))) int32_t gint;
typedef __attribute__((address_space(1))) unsigned char gbyte;
// an opaque copy: what is derived from it is worked out where it is used instead of being kept in registers
__device__ __forceinline__ unsigned here(unsigned x) { asm volatile("" : "+v"(x)); return x; }
#define MLP_UNI(x) __builtin_amdgcn_readfirstlane(x)

__device__ __forceinline__ uint64_t msg_load(const gmsg* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void msg_store(gmsg* p, float v, uint32_t tag) {
  __hip_atomic_store(p, ((uint64_t)tag << 32) | (uint64_t)__float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float msg_value(uint64_t m) { return __uint_as_float((uint32_t)m); }
__device__ __forceinline__ uint32_t msg_tag(uint64_t m) { return (uint32_t)(m >> 32); }

// Bound of a wait: looked at every 256 polls.
struct MlpWait {
  uint32_t polls = 0;
  uint64_t start = 0;
  __device__ bool expired(int32_t* sync) {
    __builtin_amdgcn_s_sleep(1);
    if ((++polls & 255u) != 0) return false;
    const uint64_t now = __builtin_amdgcn_s_memrealtime();   // 100 MHz
    if (polls == 256u) start = now;
    if (now - start > 400000000ull || __hip_atomic_load(sync + SYNC_ERR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
      __hip_atomic_fetch_or(sync + SYNC_ERR, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return true;
    }
    return false;
  }
};

// NQ: columns per lane; RW: rows per wavefront; WF: weight-difference form of the prediction (the predicted weights are
// then state of their own: w' + T (w' - w); in the velocity form they are w - lr T v, worked out when used).
// ONE: a launch of one tick (fed by the host): its instructions are fetched anew for that tick, so it holds no loop over ticks.
template <int NQ, int RW, bool WF, bool ONE>
__global__ void __launch_bounds__(MLP_BLK) __attribute__((amdgpu_waves_per_eu(2, 2))) k_mlp(MlpArgs A) {
  constexpr int CP = 64 * NQ, R = MLP_WAVES * RW, SLOTS = mlp_hist_slots(NQ);
  constexpr int XU = (CP + MLP_BLK - 1) / MLP_BLK, DU = MLP_DYB / MLP_BLK;
  __shared__ float hist[SLOTS * CP];        // the stage's inputs of the last D + 2 ticks
  __shared__ float red[MLP_WAVES * CP];     // gradient of the input, one partial sum per wavefront
  __shared__ float dyb[MLP_DYB];            // partial gradients [part][row]
  __shared__ float lg[MLP_MAX_K];
  __shared__ int lab[ONE ? 1 : mlp_launch_ticks(NQ)];
  __shared__ int stop;
  const MlpRec P = A.recs[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63, wv = MLP_UNI(tid >> 6);
  const int S = A.S, K = P.K, C = P.C, D = P.D, depth = D + 2, s = P.stage, r0 = P.r0, n = ONE ? 1 : A.n_ticks, t0 = A.t0;
  const bool first = s == 0, last = s == S - 1;
  const int parts = P.parts;
  const float fa = P.fa, fb = P.fb, lrT = P.flrT, lr = P.flr, fm = P.fm;
  const int row0 = r0 + wv * RW;

  // ---- parameters into registers (rows and columns beyond the matrix are zero and stay so)
  float w[RW][NQ], v[RW][NQ], h[WF ? RW : 1][WF ? NQ : 1], wb[RW], vb[RW], hb[WF ? RW : 1];
  {
    const gfloat* hs = (const gfloat*)P.what + (size_t)(t0 & 1) * P.what_stride;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      const int row = row0 + i;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const int col = lane + 64 * q;
        const bool ok = row < K && col < C;
        const size_t o = ok ? (size_t)row * C + col : 0;
        const float w_ = ((const gfloat*)P.w)[o], v_ = ((const gfloat*)P.v)[o];
        w[i][q] = ok ? w_ : 0.f;
        v[i][q] = ok ? v_ : 0.f;
        if (WF) { const float h_ = hs[o]; h[i][q] = ok ? h_ : 0.f; }
      }
      const bool okb = P.bias && row < K;
      wb[i] = okb ? ((const gfloat*)P.b)[row] : 0.f;
      vb[i] = okb ? ((const gfloat*)P.vb)[row] : 0.f;
      if (WF) hb[i] = okb ? ((const gfloat*)P.hb + (size_t)(t0 & 1) * P.what_stride)[row] : 0.f;
    }
  }
  // ---- inputs of earlier ticks whose backward pass falls into this launch, and the first tick's input
  const int n_old = n < D ? n : D;
  for (int j = 0; j < n_old; ++j) {
    const int tt = t0 - D + j;
    const int sl = (tt + depth * 8) % depth;       // (tt >= -D)
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int c = tid + u * MLP_BLK;
      if (c < CP) hist[sl * CP + c] = (tt >= 0 && c < C) ? ((const gfloat*)P.xring)[(size_t)sl * C + c] : 0.f;
    }
  }
  // (pool items, ring slots and the like are counted up from tick to tick: a division by a run-time value is some forty
  // dependent instructions, with 64 bits some hundred more, all of them fetched anew in a launch of one tick)
  int item = A.item0;
  auto sample_of = [&](int it) { return (const gfloat*)(A.sample ? A.sample : A.pool + (size_t)it * C); };
  float xs[XU];
  auto fetch_input = [&](const gfloat* src) {
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int c = tid + u * MLP_BLK;
      xs[u] = c < C ? src[c] : 0.f;
    }
  };
  fetch_input(first ? sample_of(item) : (const gfloat*)P.xring + (size_t)(t0 % depth) * C);
  // the launch's labels into LDS: in the last stage, whose tick is the longest, a request and its index arithmetic would stand
  // between the logits and their gradient.  Samples that entered before this launch have theirs in the label ring (whose
  // slots are overwritten when the launch ends).
  int loss_at = 0;
  if (last) {
    const int j0 = t0 - (S - 1);
    loss_at = j0 > 0 ? j0 % A.loss_cap : 0;
    for (int i = tid; i < n; i += MLP_BLK) {
      const int j = j0 + i;
      lab[i] = j >= t0 ? ((const gint*)A.pool_labels)[((unsigned)A.item0 + (unsigned)(j - t0)) % (unsigned)A.n_pool] : j >= 0 ? ((const gint*)A.labels)[j % S] : 0;
    }
  }
  int yslot = last ? 0 : (t0 + 1) % D;
  if (tid == 0) stop = 0;
  __syncthreads();

  int slot = t0 % depth;
  bool ok_all = true;
  for (int it = 0; it < n; ++it) {
    const int t = t0 + it, par = t & 1, slot_old = slot + 2 >= depth ? slot + 2 - depth : slot + 2;
    const uint32_t tag = (uint32_t)t + 1u;
    const bool live_f = t >= P.t_f, live_b = t >= P.t_b;
    float* hx = hist + slot * CP;
    float sm = 0.f, lmx = 0.f;
    // ---- the tick's input and the gradient of the workgroup's rows.  NU: messages per thread the latter take.  (Where one is
    // enough the bookkeeping of up to eight -- guards, addresses, checks -- was half of the time between two ticks.)
    auto take = [&](auto NU_) {
      constexpr int NU = decltype(NU_)::value;
      const bool plain_dy = it == 0 && A.dy_plain;
      const bool poll_x = !first && it > 0;
      const int nd = (last || (it == 0 && (!live_b || plain_dy))) ? 0 : parts * R;
      const gbyte* xb = (const gbyte*)P.xbox + (size_t)(par * C) * 8;
      const gbyte* db = (const gbyte*)P.dybox + (size_t)(par * parts * K) * 8;
      const unsigned tl = here((unsigned)tid);
      unsigned xof[XU], dof[NU];
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        const unsigned c = tl + u * MLP_BLK;
        xof[u] = c < (unsigned)C ? 8u * c : 0u;
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const unsigned i = tl + u * MLP_BLK, q = i / R, row = (unsigned)r0 + i % R;
        dof[u] = (i < (unsigned)nd && row < (unsigned)K) ? 8u * (q * (unsigned)K + row) : 0u;
      }
      uint64_t xm[XU], dm[NU];
      MlpWait wait;
      // (only wavefronts that take something: with few columns the first ones do, which have no messages of their own on
      // their way -- a wait for a load is one for the stores before it, too)
      while ((poll_x && wv * 64 < C) || wv * 64 < nd) {
        bool ok = true;
        if (poll_x) {
#pragma unroll
          for (int u = 0; u < XU; ++u) xm[u] = msg_load((const gmsg*)(xb + xof[u]));
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
          if (u * MLP_BLK < nd) dm[u] = msg_load((const gmsg*)(db + dof[u]));
        if (poll_x) {
#pragma unroll
          for (int u = 0; u < XU; ++u) ok = ok && msg_tag(xm[u]) == tag;
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
          if (u * MLP_BLK < nd) ok = ok && msg_tag(dm[u]) == tag;
        if (__ballot(!ok) == 0) break;
        if (wait.expired(A.sync)) { stop = 1; break; }
      }
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        const int c = tid + u * MLP_BLK;
        if (c < CP) hx[c] = c < C ? (poll_x ? msg_value(xm[u]) : xs[u]) : 0.f;
        if (first && P.me == 0 && c < C) ((gfloat*)P.xring)[(size_t)slot * C + c] = xs[u];
      }
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int i = tid + u * MLP_BLK;
        if (u * MLP_BLK < nd && i < nd) dyb[i] = r0 + i % R < K ? msg_value(dm[u]) : 0.f;
      }
      if (nd == 0 && !last && tid < R) {
        const int row = r0 + tid;
        const float g = (plain_dy && live_b && row < K) ? ((const gfloat*)P.gradbox)[(size_t)par * K + row] : 0.f;
        for (int p = 0; p < parts; ++p) dyb[p * R + tid] = p == 0 ? g : 0.f;
      }
    };
    if (parts * R <= MLP_BLK) take(std::integral_constant<int, 1>());
    else take(std::integral_constant<int, DU>());
    __syncthreads();
    if (stop) { ok_all = false; break; }
    float xn[NQ], xo[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float a = hx[lane + 64 * q], b = hist[slot_old * CP + lane + 64 * q];
      if (P.relu) { a = fmaxf(a, 0.f); b = fmaxf(b, 0.f); }
      xn[q] = live_f ? a : 0.f;
      xo[q] = live_b ? b : 0.f;
    }
    float dy[RW];
    if (!last) {
#pragma unroll
      for (int i = 0; i < RW; ++i) {
        float a = lane < parts ? dyb[lane * R + wv * RW + i] : 0.f;
        for (int p = lane + 64; p < parts; p += 64) a += dyb[p * R + wv * RW + i];
        dy[i] = wave_sum(a);
      }
    }
    // ---- forward
    float y[RW];
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      float a0 = 0.f, a1 = 0.f;
#pragma unroll
      for (int q = 0; q < NQ; q += 2) {
        a0 = fmaf(WF ? h[WF ? i : 0][WF ? q : 0] : fmaf(-lrT, v[i][q], w[i][q]), xn[q], a0);
        a1 = fmaf(WF ? h[WF ? i : 0][WF ? q + 1 : 0] : fmaf(-lrT, v[i][q + 1], w[i][q + 1]), xn[q + 1], a1);
      }
      y[i] = wave_sum(a0 + a1);
      if (P.bias) y[i] += WF ? hb[WF ? i : 0] : fmaf(-lrT, vb[i], wb[i]);
      if (!live_f) y[i] = 0.f;
    }
    float ysel = y[0];
#pragma unroll
    for (int i = 1; i < RW; ++i) ysel = lane == i ? y[i] : ysel;
    const bool mine = lane < RW && row0 + lane < K;
    if (!last) {
      if (mine) {
        msg_store((gmsg*)P.ybox + (size_t)(par ^ 1) * K + row0 + lane, ysel, tag + 1u);
        if (live_f) ((gfloat*)P.yring)[(size_t)yslot * K + row0 + lane] = ysel;
      }
    } else {
      if (P.n_wg == 1) {
        if (mine) lg[row0 + lane] = ysel;
      } else if (live_f) {
        if (mine) msg_store((gmsg*)A.lbox + (size_t)par * K + row0 + lane, ysel, tag);
        for (int k = tid; k < K; k += MLP_BLK) {
          MlpWait wait;
          uint64_t m;
          while (msg_tag(m = msg_load((const gmsg*)A.lbox + (size_t)par * K + k)) != tag)
            if (wait.expired(A.sync)) { stop = 1; break; }
          lg[k] = msg_value(m);
        }
      }
      __syncthreads();
      if (stop) { ok_all = false; break; }
#pragma unroll
      for (int i = 0; i < RW; ++i) dy[i] = 0.f;
      if (live_f) {
        // softmax cross-entropy, by every wavefront for itself; up to 64 classes stay in a register
        const int label = lab[it];
        float mx = -3.0e38f, l0 = -3.0e38f;
        if (lane < K) l0 = lg[lane];
        mx = l0;
        for (int k = lane + 64; k < K; k += 64) mx = fmaxf(mx, lg[k]);
        mx = wave_max_dpp(mx);
        const float e0 = lane < K ? expf(l0 - mx) : 0.f;
        sm = e0;
        for (int k = lane + 64; k < K; k += 64) sm += expf(lg[k] - mx);
        sm = wave_sum(sm);
        lmx = mx;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
          const int r = row0 + i;
          if (r < K) {
            const float e = r < 64 ? __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e0), MLP_UNI(r))) : expf(lg[r] - mx);
            dy[i] = e / sm - (r == label ? 1.f : 0.f);
          }
        }
      }
    }
    // ---- gradient of the input: this workgroup's rows' share of every column
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      float a = 0.f;
#pragma unroll
      for (int i = 0; i < RW; ++i) a = fmaf(w[i][q], dy[i], a);
      if (!first) red[wv * CP + lane + 64 * q] = a;
    }
    if (first && it + 1 < n) {
      if (!A.sample) item = item + 1 == A.n_pool ? 0 : item + 1;
      fetch_input(sample_of(item));
    }
    __syncthreads();
    if (!first) {
#pragma unroll
      for (int u = 0; u < XU; ++u) {
        // (with up to 256 columns the other half of the workgroup sends, where the first waits for another tick's messages)
        const int c = (ONE ? tid : tid ^ (MLP_BLK / 2)) + u * MLP_BLK;
        if (c < C) {
          float a = 0.f;
#pragma unroll
          for (int k = 0; k < MLP_WAVES; ++k) a += red[k * CP + c];
          if (P.relu && !(hist[slot_old * CP + c] > 0.f)) a = 0.f;
          msg_store((gmsg*)P.dxbox + ((size_t)(par ^ 1) * P.n_wg + P.me) * C + c, a, tag + 1u);
        }
      }
    }
    if (last) {
      if (live_f) {
        if (P.me == 0 && tid == MLP_BLK - 64) ((gfloat*)A.loss)[loss_at] = logf(sm) + lmx - lg[lab[it]];
        loss_at = loss_at + 1 == A.loss_cap ? 0 : loss_at + 1;
      }
    }
    yslot = yslot + 1 == D ? 0 : yslot + 1;
    // ---- update (Eqs. gscv, gscw, lwp_v_form / lwp_w_form) while the messages are on their way
#pragma unroll
    for (int i = 0; i < RW; ++i) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float g = dy[i] * xo[q], w_old = w[i][q];
        v[i][q] = fmaf(fm, v[i][q], g);
        w[i][q] = fmaf(-lr, fmaf(fa, v[i][q], fb * g), w_old);
        if (WF) h[WF ? i : 0][WF ? q : 0] = fmaf(lrT, w[i][q] - w_old, w[i][q]);
      }
      const float g = dy[i], b_old = wb[i];
      vb[i] = fmaf(fm, vb[i], g);
      wb[i] = fmaf(-lr, fmaf(fa, vb[i], fb * g), b_old);
      if (WF) hb[WF ? i : 0] = fmaf(lrT, wb[i] - b_old, wb[i]);
    }
    slot = slot + 1 == depth ? 0 : slot + 1;
  }
  if (!ok_all) return;
  // ---- parameters back to memory
  {
    const size_t ho = (size_t)((t0 + n) & 1) * P.what_stride;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
      const int row = row0 + i;
      if (row < K) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const int col = lane + 64 * q;
          if (col < C) {
            const size_t o = (size_t)row * C + col;
            ((gfloat*)P.w)[o] = w[i][q];
            ((gfloat*)P.v)[o] = v[i][q];
            if (WF) ((gfloat*)P.what + ho)[o] = h[WF ? i : 0][WF ? q : 0];
          }
        }
        if (P.bias && lane == 0) {
          P.b[row] = wb[i];
          P.vb[row] = vb[i];
          if (WF) (P.hb + ho)[row] = hb[WF ? i : 0];
        }
      }
    }
  }
  if (last && P.me == 0 && tid < S) {
    // label ring: the samples that entered in this launch
    const int j = t0 + n - 1 - tid;
    if (j >= t0) A.labels[j % S] = A.sample ? A.label : A.pool_labels[((unsigned)A.item0 + (unsigned)(j - t0)) % (unsigned)A.n_pool];
  }
}

// One workgroup per workgroup of k_mlp: predicted weights of tick t (velocity form; the other form keeps them in memory
// already) and the sums of the partial gradients, for steps of the phase kernel.
__global__ void __launch_bounds__(256) k_mlp_flush(const MlpRec* __restrict__ recs, int rows, int t) {
  const MlpRec P = recs[blockIdx.x];
  const int hi = P.r0 + rows < P.K ? P.r0 + rows : P.K;
  if (!P.lwp_w) {
    float* hw = P.what + (size_t)(t & 1) * P.what_stride;
    for (int64_t i = (int64_t)P.r0 * P.C + threadIdx.x; i < (int64_t)hi * P.C; i += 256) hw[i] = fmaf(-P.flrT, P.v[i], P.w[i]);
    if (P.bias) {
      float* hb = P.hb + (size_t)(t & 1) * P.what_stride;
      for (int i = P.r0 + (int)threadIdx.x; i < hi; i += 256) hb[i] = fmaf(-P.flrT, P.vb[i], P.b[i]);
    }
  }
  if (P.parts > 0 && t >= P.t_b)
    for (int i = P.r0 + (int)threadIdx.x; i < hi; i += 256) {
      float a = 0.f;
      for (int p = 0; p < P.parts; ++p) a += msg_value(P.dybox[((size_t)(t & 1) * P.parts + p) * P.K + i]);
      P.gradbox[(size_t)(t & 1) * P.K + i] = a;
    }
}

template <int NQ, bool ONE>
static void launch_nq(const MlpArgs& a, int grid, int rw, bool wf, hipStream_t s) {
#define PB_MLP(RW, WF) hipLaunchKernelGGL((k_mlp<NQ, RW, WF, ONE>), dim3(grid), dim3(MLP_BLK), 0, s, a)
  if (rw == 2) { if (wf) PB_MLP(2, true); else PB_MLP(2, false); return; }
  if constexpr (NQ == 16) {
    if (!wf) PB_MLP(3, false);
  } else {
    if (rw == 3) { if (wf) PB_MLP(3, true); else PB_MLP(3, false); }
    else { if (wf) PB_MLP(4, true); else PB_MLP(4, false); }
  }
#undef PB_MLP
}

void launch_mlp(const MlpArgs& a, int grid, int nq, int rw, bool lwp_w, hipStream_t s) {
  auto launch = [&](auto ONE) {
    constexpr bool one = decltype(ONE)::value;
    if (nq == 2) launch_nq<2, one>(a, grid, rw, lwp_w, s);
    else if (nq == 4) launch_nq<4, one>(a, grid, rw, lwp_w, s);
    else if (nq == 8) launch_nq<8, one>(a, grid, rw, lwp_w, s);
    else launch_nq<16, one>(a, grid, rw, lwp_w, s);
  };
  if (a.n_ticks == 1) launch(std::true_type());
  else launch(std::false_type());
}

void launch_mlp_flush(const MlpRec* recs, int grid, int rows, int t, hipStream_t s) {
  hipLaunchKernelGGL(k_mlp_flush, dim3(grid), dim3(256), 0, s, recs, rows, t);
}

}  // namespace pb
