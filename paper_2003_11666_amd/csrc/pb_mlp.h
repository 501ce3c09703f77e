// Shared between the host runtime and the kernel that runs a perceptron with its
// parameters held in registers (pb_mlp.hip).  Plain data only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pb {

constexpr int MLP_BLK = 512;             // threads of a workgroup: 8 wavefronts, two per SIMD (256 registers each)
constexpr int MLP_WAVES = MLP_BLK / 64;
constexpr int MLP_MAX_STAGES = 12;
constexpr int MLP_MAX_C = 1024;          // inputs of a stage: 16 per lane
constexpr int MLP_MAX_K = 1024;          // classes (logits in LDS)
constexpr int MLP_DYB = 4096;            // LDS floats for the partial gradients of a workgroup's rows
// Ticks one launch runs at most: a launch may hold every compute unit, which are closed to other streams meanwhile, so it
// is bounded by time.  Measured per tick: 2.1-2.3 us up to 256 inputs per stage (nq 2 and 4), 2.9 us at 512 (nq 8),
// 4.1-6.5 us at 1024 (nq 16), i.e. 1.5-3.3 ms a launch; the way from one launch to the next costs 8 us.
constexpr int mlp_launch_ticks(int nq) { return nq <= 4 ? 1024 : 512; }
constexpr int mlp_hist_slots(int nq) { return nq >= 16 ? 12 : 24; }   // input history of a stage in LDS (its delay + 2)

// One workgroup of the launch: `rows` consecutive output rows of one stage.
struct MlpRec {
  int32_t stage, me, n_wg, r0;           // stage; the workgroup's index in it, their number; first row
  int32_t K, C, D;                       // rows, columns, ticks between forward and backward pass
  int32_t relu, bias, lwp_w;
  int32_t t_f, t_b;                      // first tick with a forward / a backward pass
  int32_t parts;                         // partial gradients that arrive per row: workgroups of the next stage
  float fa, fb, flrT, flr, fm;           // see K_UPDATE
  float *w, *v, *b, *vb;                 // master weights and bias with their velocities
  float *what, *hb;                      // slot 0 of the ring (2 slots, what_stride apart) of predicted weights
  int64_t what_stride;
  float* xring;                          // the stage's input ring [D + 2][C]
  float* yring;                          // the next stage's [D][K] (depth D - 2 + 2), nullptr in the last stage
  float* gradbox;                        // [2][K]: gradient of the stage's output when the phase kernels wrote it
  uint64_t* xbox;                        // [2][C] messages: input of the next tick, by parity of that tick
  uint64_t* ybox;                        // the next stage's xbox
  uint64_t* dybox;                       // [2][parts][K]: partial gradients of the stage's output
  uint64_t* dxbox;                       // the previous stage's dybox, nullptr in the first stage
};

struct MlpArgs {
  const MlpRec* recs;
  int32_t S, n_ticks, t0;
  int32_t dy_plain;                      // the first tick's gradients lie in gradbox
  const float* pool;                     // samples; tick t takes item (item0 + t - t0) mod n_pool
  const int32_t* pool_labels;
  int32_t n_pool, item0;
  const float* sample;                   // one tick fed by the host: its sample and label
  int32_t label, loss_cap;
  float* loss;
  int32_t* labels;                       // label ring [S]
  int32_t* sync;                         // error word
  uint64_t* lbox;                        // [2][K of the last stage]: logits of a last stage of several workgroups
};

// rows per wavefront rw (2, 3, 4), inputs per lane nq (2, 4, 8, 16), see mlp_plan
void launch_mlp(const MlpArgs& a, int grid, int nq, int rw, bool lwp_w, hipStream_t s);
// leaves the state a launch of phase kernels expects: predicted weights of tick t and whole gradients
void launch_mlp_flush(const MlpRec* recs, int grid, int rows, int t, hipStream_t s);

}  // namespace pb
