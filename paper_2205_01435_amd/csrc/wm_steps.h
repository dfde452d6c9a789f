// Arguments and launchers of the per-step kernels of the multi-launch path.
// Internal to libwm.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wm_gemm.h"
#include "wm_layout.h"

namespace wm {

struct GatesArgs {
  const void* Wg;
  const void* WaT;
  const float* bg;
  long ldk, ldx;
  int H, A, Z, M;
  const void* x_in;  // X_t [M, ldx] DT
  void* x_out;       // X_t+1 [M, ldx] DT: h_t+1 goes to columns Z .. Z+H-1
  float* c;          // [M, H] fp32, updated in place
  const int32_t* act;
  float* h_trace;  // [M, H] fp32 or null
  float* c_trace;
  int nll_mode;
  int runs;  // slices per run of the sum over K (KSum::Runs)
  TileMap map;
};

// The mixture head.
struct MdnArgs {
  const void* Wm;
  const float* bm;
  long ldh, ldx;
  int H, Z, K, Nm, M;
  // [M, ldx] DT activation rows: the head reads h at columns Z ..; the
  // rollout writes q(z_t+1) to columns 0 .. Z-1
  void* x;
  // rollout
  const int32_t* act;
  const float* z_prev;  // [M, Z]
  float* z_next;        // [M, Z]
  uint32_t k0, k1, step, traj0;
  float tau;
  float sig;  // scale of the normal deviate: sqrt(tau) with the sigma temperature, else 1
  // nll
  const float* z_tgt;  // [M, Z]
  float* part;         // [M, ntd]
  float* head;         // [M, 2]
  int ntd;
  int nll_mode;
  int runs;  // slices per run of the sum over K (KSum::Runs)
  // rollout, with lh: tiles past the zt groups of four latent dims compute the
  // next step's controller logits' h part, lh[m][n] = W_c[n][Z ..] . h_t+1
  // (bias not added), fp32, Nc of each row of ldl; zt = 0: only those
  int zt;
  const void* Wc;
  long ldk;
  int Nc;
  float* lh;
  long ldl;
  TileMap map;
};

// The controller.
struct CtrlArgs {
  const void* Wc;
  const float* bc;
  long ldk;
  int Z, H, A, Nc, M;
  const void* x;   // rollout: X_t [M, ldx] DT
  long ldx;
  const float* z;  // controller step: z [M, Z] and h [M, H], fp32
  const float* h;
  const uint8_t* mask;
  uint32_t k0, k1, step, traj0;
  int mode;
  // mode 0
  float* probs;
  int32_t* action;
  // mode 1/2
  int32_t* act_t;       // [M]
  const int32_t* act_prev;  // [M] or null (t == 0)
  float* rew_prev;
  uint8_t* done_prev;
  float* rew_t;
  uint8_t* done_t;
  int32_t* done_state;
  int use_done;
  // per-trajectory horizons (null: T for all): a step t >= lengths[m] is padding
  const int32_t* lengths;
  int t;
  // two-level controller (N > 0): mask holds the xfer masks [M, N+1]
  // followed by the location masks [M, N, Lc]; the logits are the N+1 xfer
  // rows then the Lc location rows
  int N, Lc;
  // logits stored instead of picked (k_ctrl_logits, k_ctrl_wide): columns [0, ncol) of each
  // row, bias not added, at logits_out + m ldl; k_ctrl_rows then picks
  float* logits_out;
  long ldl;
  int ncol;
  const float* lh;  // rollout: the logits' h part (k_ctrl_z), Nc of each row of ldlh, null: zero
  long ldlh;
  float* lg_ws;  // rollout workspace [M, Nc] for those logits (wide two-level controllers)
  TileMap map;   // of k_ctrl_logits
};

// One launch each on `s`, the tile chosen from the call's sizes; defined for
// float and bf16_t (launch_ctrl also for the standalone step's two-tensor
// activation source).
template <typename DT>
hipError_t launch_gates(GatesArgs a, hipStream_t s);
template <typename DT>
hipError_t launch_mdn(const MdnArgs& a, int Q, int ntiles, hipStream_t s);
template <class S>
hipError_t launch_ctrl(const CtrlArgs& a, hipStream_t s);
// Whether a rollout computes the controller's h part beside the mixture: fp32
// only (it sums the logits' h columns before their z columns, and a bf16
// rollout's sums keep one order, KSum), the matrix rows of W_c need to be
// readable Z + ldh wide, the logits to fit the z and h columns of an activation
// row (where they wait for the next step), the two-level controller's to fit
// k_ctrl_z's staged rows, and the extra tiles to cost the mixture launch less
// than the deeper product costs the controller.
bool ctrl_h_wanted(const Layout& L, int B);
// The controller's h part alone (MdnArgs::lh, zt = 0), and the rollout's
// decision from it.
hipError_t launch_ctrl_h(MdnArgs a, int Q, hipStream_t s);
hipError_t launch_ctrl_z(const CtrlArgs& a, hipStream_t s);

}  // namespace wm
