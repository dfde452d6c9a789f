// The controller of the per-step path and the standalone controller step.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "wm_device.h"
#include "wm_gemm.h"
#include "wm_kernels.h"
#include "wm_profile.h"
#include "wm_steps.h"

namespace wm {

// ===========================================================================
// k_ctrl: controller logits for BM = 16*MBW rows (all Nc outputs in one
// block; four waves take interleaved 16-output slices), weights read
// straight from global memory, activations staged through LDS in K chunks.
//   mode 0: controller step (probs + action)
//   mode 1: rollout step t: resolve transition t-1, choose a_t
//   mode 2: rollout tail: resolve transition T-1 only
// ===========================================================================
// What the bookkeeping of row m reads: its done state, the action of the
// previous transition (-1 at the first step) and whether step t is padding.
// Kernels load it ahead of their product.
struct RowState {
  int ds, prev, pad;
};
__device__ __forceinline__ RowState row_state(const CtrlArgs& p, int m) {
  RowState r;
  r.ds = p.done_state[m];
  r.prev = p.act_prev ? p.act_prev[m] : -1;
  r.pad = p.lengths && p.t >= p.lengths[m];
  return r;
}

// Rollout bookkeeping of row m at step t (modes 1 and 2 of the controller
// kernels).  First the previous transition t-1 is resolved if the row was
// live then: its reward is the reward head on h_t and it is done when
// sigmoid(done head) exceeds the stream-3 uniform of step t-1.  Then (mode 1)
// the row takes action `a` (the masked Gumbel-max, -1 if no action is valid)
// or, if done, the frozen outputs; a row without a valid action ends here.
// A step past the row's horizon is padding: no action, reward 0, done 0 (its
// state is kept like a frozen row's; the latent is zeroed afterwards).
__device__ __forceinline__ void ctrl_row_commit(const CtrlArgs& p, const Rng& rng, int m, int a,
                                                float rr, float rd, const RowState& r) {
  int ds = r.ds;
  if (r.prev >= 0) {
    p.rew_prev[m] = rr;
    int d = 0;
    if (p.use_done) {
      const uint4 w = rng.block(0, p.step - 1u, p.traj0 + (uint32_t)m, STREAM_DONE);
      d = sigmoidf(rd) > word_to_uniform(w.x);
    }
    p.done_prev[m] = (uint8_t)d;
    if (d) ds = 1;
  }
  if (p.mode == 1) {
    if (ds || r.pad) a = -1;
    else if (a < 0) ds = 1;
    p.act_t[m] = a;
    if (a < 0) {
      p.rew_t[m] = 0.f;
      p.done_t[m] = r.pad ? 0 : 1;
    }
  }
  p.done_state[m] = ds;
}

// Two-level pick of row m (section 3.1.3) by its TPR threads (thread q of
// the row), from its logits lg (bias not yet added): an xfer among the valid
// ones (stream 0, index x; x = N is the NO-OP), then a location valid for
// that xfer (stream 4, index l).  two_level_xfer returns x (-1 when none is
// valid), two_level_loc the location of xfer x < N (-1 when none is valid),
// two_level_pick the flat action x Lc + l, -2 for the NO-OP, -1 when nothing
// is valid; the same value in every thread of the row.  Ties go to the
// lowest index.  LMAX bounds Lc.
template <int TPR>
__device__ __forceinline__ void row_argmax(float& best, int& bidx) {
#pragma unroll
  for (int off = 1; off < TPR; off <<= 1) {
    const float ob = __shfl_xor(best, off);
    const int oi = __shfl_xor(bidx, off);
    if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
  }
}

template <int TPR>
__device__ __forceinline__ int two_level_xfer(const CtrlArgs& p, const Rng& rng, const float* lg, int m,
                                              bool on, int q, uint32_t traj) {
  const int NX = p.N + 1;
  float best = -INFINITY;
  int x = -1;
  if (on) {
    for (int i = q; i < NX; i += TPR) {
      if (!p.mask[(long)m * NX + i]) continue;
      const uint4 w = rng.block((uint32_t)i >> 2, p.step, traj, STREAM_CONTROLLER);
      const float sc = lg[i] + p.bc[i] + gumbel(word_to_uniform(word_of(w, i & 3)));
      if (sc > best) { best = sc; x = i; }
    }
  }
  row_argmax<TPR>(best, x);
  return x;
}

template <int TPR, int LMAX>
__device__ __forceinline__ int two_level_loc(const CtrlArgs& p, const Rng& rng, const float* lg, int m,
                                             bool on, int q, uint32_t traj, int x) {
  const int N = p.N, NX = N + 1, Lc = p.Lc;
  const uint8_t* lm = p.mask + (long)p.M * NX + ((long)m * N + x) * Lc;
  // thread q takes the contiguous locations [l0, l1) (a multiple of four:
  // one Philox block each); their mask bytes are all loaded before the
  // first is used, instead of one dependent load per location
  constexpr int MAXW = (((LMAX + TPR - 1) / TPR + 3) & ~3) / 4;
  const int cpt = ((Lc + TPR - 1) / TPR + 3) & ~3;
  const int l0 = q * cpt, l1 = min(l0 + cpt, Lc);
  uint32_t mw[MAXW];
#pragma unroll
  for (int k = 0; k < MAXW; ++k) {
    uint32_t wv = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = l0 + 4 * k + v;
      if (on && i < l1 && lm[i]) wv |= 1u << (8 * v);
    }
    mw[k] = wv;
  }
  float best = -INFINITY;
  int l = -1;
#pragma unroll
  for (int k = 0; k < MAXW; ++k) {
    if (mw[k] == 0) continue;
    const int b = l0 + 4 * k;
    const uint4 w = rng.block((uint32_t)b >> 2, p.step, traj, STREAM_LOCATION);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if ((mw[k] >> (8 * v)) & 1u) {
        const float sc = lg[NX + b + v] + p.bc[NX + b + v] + gumbel(word_to_uniform(word_of(w, v)));
        if (sc > best) { best = sc; l = b + v; }
      }
    }
  }
  row_argmax<TPR>(best, l);
  return l;
}

template <int TPR, int LMAX = 316>
__device__ __forceinline__ int two_level_pick(const CtrlArgs& p, const Rng& rng, const float* lg,
                                              int m, bool on, int q, uint32_t traj) {
  const int x = two_level_xfer<TPR>(p, rng, lg, m, on, q, traj);
  if (x < 0) return -1;
  if (x == p.N) return -2;
  const int l = two_level_loc<TPR, LMAX>(p, rng, lg, m, on, q, traj, x);
  return l < 0 ? -1 : x * p.Lc + l;
}

// One lane's share of a pick by a whole wave over n scores: the NB blocks of
// four consecutive indices lane, lane + 64, ... (one Philox block each; 256 NB
// scores at most), whose logits and biases are all loaded before the first is
// used.
constexpr int kRowBlk = 4;  // N + 1 and Lc go up to 1024
template <int NB>
struct RowLogits {
  float v[NB][4];
};

// logits + biases of indices [0, n) at byte offset o0 of both rows
template <int NB>
__device__ __forceinline__ void row_logits(RowLogits<NB>& r, rsrc_t rl, rsrc_t rb, uint32_t o0, int n, int lane) {
  float b[NB][4];
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * (lane + 64 * k) + v;
      const uint32_t o = i < n ? o0 + 4u * (uint32_t)i : kOffNone;
      r.v[k][v] = __uint_as_float(bload4(rl, o));
      b[k][v] = __uint_as_float(bload4(rb, o));
    }
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) r.v[k][v] += b[k][v];
}

// mask bytes m[o0 .. o0 + n) of the lane's blocks, one bit per index
template <int NB>
__device__ __forceinline__ uint32_t row_mask(rsrc_t rm, uint32_t o0, int n, int lane) {
  uint32_t by[NB][4], bits = 0;
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = 4 * (lane + 64 * k) + v;
      by[k][v] = bload1(rm, i < n ? o0 + (uint32_t)i : kOffNone);
    }
#pragma unroll
  for (int k = 0; k < NB; ++k)
#pragma unroll
    for (int v = 0; v < 4; ++v) bits |= by[k][v] ? 1u << (4 * k + v) : 0u;
  return bits;
}

// Gumbel-max over the valid indices, lowest index on ties; the wave's lanes
// all return it (-1: none valid).
template <int NB>
__device__ __forceinline__ int row_pick(const RowLogits<NB>& r, uint32_t bits, const Rng& rng, uint32_t step,
                                        uint32_t traj, uint32_t stream, int lane) {
  float best = -INFINITY;
  int bi = -1;
#pragma unroll
  for (int k = 0; k < NB; ++k) {
    const uint32_t m4 = (bits >> (4 * k)) & 15u;
    if (!m4) continue;
    const uint32_t blk = (uint32_t)(lane + 64 * k);
    const uint4 w = rng.block(blk, step, traj, stream);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if ((m4 >> v) & 1u) {
        const float sc = r.v[k][v] + gumbel(word_to_uniform(word_of(w, v)));
        if (sc > best) { best = sc; bi = (int)(4 * blk) + v; }
      }
    }
  }
  row_argmax<64>(best, bi);
  return bi;
}

// The two-level controller from stored logits (k_ctrl_logits, k_ctrl_wide),
// one wave per row, for controllers too wide for the staged tiles and for
// the controller step.  Rollout modes: the pick and the row's commit (the
// reward and done logits are columns Ac, Ac + 1).  Mode 0: the action and,
// over the row's logits in place, the probabilities: the softmax of the
// valid xfers' logits [N+1], then the softmax of the valid locations of the
// picked xfer [Lc] (0 after a NO-OP or when nothing is valid).
// Bound by the latency of its loads: everything but the chosen xfer's
// location mask is in flight before the first value is used, and a lane
// takes four consecutive indices per Philox block.  (One xfer index per
// block and a load at a time before: 11.8 us per step at B 4096, N 288,
// L 200.)
template <int XB, int LB>
__global__ void __launch_bounds__(256) k_ctrl_rows(const CtrlArgs p) {
  const int lane = threadIdx.x & 63;
  const int m = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (m >= p.M) return;  // the whole wave
  float* lg = p.logits_out + (long)m * p.ldl;
  const Rng rng{p.k0, p.k1};
  const uint32_t traj = p.traj0 + (uint32_t)m;
  const int N = p.N, NX = N + 1, Lc = p.Lc, Ar = NX + Lc;
  const int ncol = p.mode == 0 ? Ar : Ar + 2;
  const rsrc_t rl = uniform_rsrc(lg, (uint32_t)ncol * 4u);
  const rsrc_t rb = uniform_rsrc(p.bc, (uint32_t)p.Nc * 4u);
  const rsrc_t rx = uniform_rsrc(p.mask + (long)m * NX, (uint32_t)NX);
  // location masks of the row's xfers (N Lc bytes; below 2^20)
  const rsrc_t rlm = uniform_rsrc(p.mask + (long)p.M * NX + (long)m * N * Lc, (uint32_t)(N * Lc));
  int x = -1, a = -1;
  RowLogits<XB> lx{};
  RowLogits<LB> ll{};
  uint32_t mx = 0, ml = 0;
  float rr = 0.f, rd = 0.f;
  RowState rs{};
  if (p.mode != 0) {
    rs = row_state(p, m);
    rr = __uint_as_float(bload4(rl, 4u * (uint32_t)Ar)) + __uint_as_float(bload4(rb, 4u * (uint32_t)Ar));
    rd = __uint_as_float(bload4(rl, 4u * (uint32_t)(Ar + 1))) + __uint_as_float(bload4(rb, 4u * (uint32_t)(Ar + 1)));
  }
  if (p.mode != 2) {
    mx = row_mask<XB>(rx, 0u, NX, lane);
    row_logits(lx, rl, rb, 0u, NX, lane);
    row_logits(ll, rl, rb, 4u * (uint32_t)NX, Lc, lane);
    x = row_pick(lx, mx, rng, p.step, traj, STREAM_CONTROLLER, lane);
    if (x == N) a = -2;
    else if (x >= 0) {
      ml = row_mask<LB>(rlm, (uint32_t)(x * Lc), Lc, lane);
      const int l = row_pick(ll, ml, rng, p.step, traj, STREAM_LOCATION, lane);
      a = l < 0 ? -1 : x * Lc + l;
    }
  }
  if (p.mode != 0) {
    if (lane == 0) ctrl_row_commit(p, rng, m, a, rr, rd, rs);
    return;
  }
  float mxx = -INFINITY, mxl = -INFINITY;
  auto each = [](auto nb, auto f) {
#pragma unroll
    for (int k = 0; k < decltype(nb)::value; ++k)
#pragma unroll
      for (int v = 0; v < 4; ++v) f(k, v);
  };
  constexpr std::integral_constant<int, XB> xb;
  constexpr std::integral_constant<int, LB> lb;
  each(xb, [&](int k, int v) { if ((mx >> (4 * k + v)) & 1u) mxx = fmaxf(mxx, lx.v[k][v]); });
  each(lb, [&](int k, int v) { if ((ml >> (4 * k + v)) & 1u) mxl = fmaxf(mxl, ll.v[k][v]); });
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    mxx = fmaxf(mxx, __shfl_xor(mxx, off));
    mxl = fmaxf(mxl, __shfl_xor(mxl, off));
  }
  float sx = 0.f, sl = 0.f;
  // (a logit of -inf has no probability, also where all of a row's are)
  each(xb, [&](int k, int v) {
    lx.v[k][v] = (mx >> (4 * k + v)) & 1u && lx.v[k][v] != -INFINITY ? expf(lx.v[k][v] - mxx) : 0.f;
    sx += lx.v[k][v];
  });
  each(lb, [&](int k, int v) {
    ll.v[k][v] = (ml >> (4 * k + v)) & 1u && ll.v[k][v] != -INFINITY ? expf(ll.v[k][v] - mxl) : 0.f;
    sl += ll.v[k][v];
  });
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    sx += __shfl_xor(sx, off);
    sl += __shfl_xor(sl, off);
  }
  const float ix = sx > 0.f ? 1.0f / sx : 0.f, il = sl > 0.f ? 1.0f / sl : 0.f;
  each(xb, [&](int k, int v) {
    const int i = 4 * (lane + 64 * k) + v;
    if (i < NX) lg[i] = lx.v[k][v] * ix;
  });
  each(lb, [&](int k, int v) {
    const int i = 4 * (lane + 64 * k) + v;
    if (i < Lc) lg[NX + i] = ll.v[k][v] * il;
  });
  if (lane == 0) p.action[m] = a;
}

// Activation source of the controller kernels for rows m0 .. m0+rows-1.
template <class S>
__device__ __forceinline__ S ctrl_src(const CtrlArgs& p, int m0, int rows) {
  using DT = typename S::DT;
  if constexpr (S::kTwo) return S(p.z, p.h, p.Z, p.H, m0, rows, p.M);
  else return S(reinterpret_cast<const DT*>(p.x), p.ldx, p.ldx, m0, rows, p.M);
}

// Logits of a rollout's wide two-level controller (more rows than the staged
// tiles hold): lg[m][n] = W_c row n . X_t row m, bias not added, for
// k_ctrl_rows.  One many-tile GEMM launch: every W_c row block is read once
// per 64 or 128 trajectories (k_ctrl_wide, which ran here before, read all of
// W_c once per 16 or 32: 50.6 us per step at B 4096, 489 logits, bf16).
template <class C>
__global__ void __launch_bounds__(C::NT) k_ctrl_logits(const CtrlArgs p) {
  using DT = typename C::DT;
  __shared__ __attribute__((aligned(16))) char lds_raw[C::LDS_BYTES];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int n0 = nt * C::BN, m0 = mt * C::BM;
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wc), p.ldk, p.ldk, n0, C::BN, p.Nc);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x), p.ldx, p.ldx, m0, C::BM, p.M);
  f32x4 acc[C::NBW][C::MBW];
  C::run(acc, w, x, (int)p.ldk, reinterpret_cast<DT*>(lds_raw));
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wn = C::wn(), wmi = C::wm();
#pragma unroll
  for (int j = 0; j < C::MBW; ++j) {
    const int m = m0 + (wmi * C::MBW + j) * 16 + r16;
    if (m >= p.M) continue;
#pragma unroll
    for (int i = 0; i < C::NBW; ++i) {
      const int n = n0 + (wn * C::NBW + i) * 16 + 4 * g;
      if (n < p.Nc)  // Nc and ldl are multiples of 16
        *reinterpret_cast<f32x4*>(p.logits_out + (long)m * p.ldl + n) = acc[i][j];
    }
  }
}

template <class S, int NBW, int MBW, int BKC>
__global__ void __launch_bounds__(256) k_ctrl_wide(const CtrlArgs p) {
  using DT = typename S::DT;
  constexpr int VEC = DType<DT>::VEC;
  constexpr int BM = 16 * MBW;
  constexpr int LDL = BKC + 2 * VEC;
  __shared__ __attribute__((aligned(16))) DT xl[BM * LDL];
  __shared__ float s_best[4][BM];
  __shared__ int s_idx[4][BM];
  __shared__ float s_max[4][BM];
  __shared__ float s_rho[BM][2];
  __shared__ float s_fin[BM][2];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int m0 = blockIdx.x * BM;
  const int nbtot = p.Nc / 16;
  const DT* W = reinterpret_cast<const DT*>(p.Wc);
  const S src = ctrl_src<S>(p, m0, BM);

  f32x4 acc[NBW][MBW];
#pragma unroll
  for (int i = 0; i < NBW; ++i)
#pragma unroll
    for (int j = 0; j < MBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int kc = 0; kc < (int)p.ldk; kc += BKC) {
    __syncthreads();
    for (int v = tid; v < BM * (BKC / VEC); v += 256) {
      const int r = v / (BKC / VEC), kv = v % (BKC / VEC);
      *reinterpret_cast<uint4*>(xl + r * LDL + kv * VEC) = src.load(src.row(r), kc + kv * VEC, (int)p.ldk);
    }
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < BKC; ks += Mfma<DT>::KSLICE) {
      if (kc + ks >= (int)p.ldk) break;  // last chunk may overhang the padded K
      // the slice's weight fragments are loaded in groups of GW, one group
      // ahead of its MFMAs, from rows clamped into the matrix (blocks past
      // nbtot are loaded but not used). Unguarded loads let each MFMA wait
      // for its own fragment only; under the guard it waited for all of them.
      constexpr int GW = 8, NG = (NBW + GW - 1) / GW;
      uint4 a[2][GW];
      auto load_group = [&](int gi, uint4(&dst)[GW]) {
#pragma unroll
        for (int q = 0; q < GW; ++q) {
          const int i = gi * GW + q;
          if (i < NBW) {
            const int nb = min(wave + 4 * i, nbtot - 1);
            dst[q] = *reinterpret_cast<const uint4*>(W + (long)(nb * 16 + r16) * p.ldk + kc + ks + g * VEC);
          }
        }
      };
      load_group(0, a[0]);
      uint4 b[MBW];
#pragma unroll
      for (int j = 0; j < MBW; ++j)
        b[j] = *reinterpret_cast<const uint4*>(xl + (j * 16 + r16) * LDL + ks + g * VEC);
#pragma unroll
      for (int gi = 0; gi < NG; ++gi) {
        if (gi + 1 < NG) load_group(gi + 1, a[(gi + 1) & 1]);
#pragma unroll
        for (int q = 0; q < GW; ++q) {
          const int i = gi * GW + q;
          if (i < NBW && wave + 4 * i < nbtot) {
#pragma unroll
            for (int j = 0; j < MBW; ++j) Mfma<DT>::step(acc[i][j], a[gi & 1][q], b[j]);
          }
        }
      }
    }
  }

  // ---- epilogue ----
  if (p.logits_out) {  // logits only (bias not added); k_ctrl_rows picks
#pragma unroll
    for (int j = 0; j < MBW; ++j) {
      const int m = m0 + j * 16 + r16;
      if (m >= p.M) continue;
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const int nb = wave + 4 * i;
        const int n = nb * 16 + 4 * g;
        if (nb >= nbtot) continue;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (n + v < p.ncol) p.logits_out[(long)m * p.ldl + n + v] = acc[i][j][v];
      }
    }
    return;
  }
  const Rng rng{p.k0, p.k1};
  const int A = p.A;
  const bool want_action = p.mode != 2;
  // the mask bytes of this lane's actions (n .. n+3 of each block, each
  // row), all loaded before the first is used
  uint32_t mk[NBW][MBW];
#pragma unroll
  for (int j = 0; j < MBW; ++j) {
    const int m = m0 + j * 16 + r16;
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int n = (wave + 4 * i) * 16 + 4 * g;
      uint32_t wv = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (m < p.M && wave + 4 * i < nbtot && n + v < A && p.mask[(long)m * A + n + v]) wv |= 1u << (8 * v);
      mk[i][j] = wv;
    }
  }
#pragma unroll
  for (int j = 0; j < MBW; ++j) {
    const int ml = j * 16 + r16;
    const int m = m0 + ml;
    float best = -INFINITY, mx = -INFINITY;
    int bidx = -1;
    if (m < p.M) {
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const int nb = wave + 4 * i;
        if (nb >= nbtot) continue;
        const int n = nb * 16 + 4 * g;
        const float4 b4 = *reinterpret_cast<const float4*>(p.bc + n);
        const float lg[4] = {acc[i][j][0] + b4.x, acc[i][j][1] + b4.y, acc[i][j][2] + b4.z,
                             acc[i][j][3] + b4.w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (n + v == A) s_rho[ml][0] = lg[v];
          if (n + v == A + 1) s_rho[ml][1] = lg[v];
        }
        if (want_action && n < A) {
          const uint4 w = rng.block((uint32_t)(n >> 2), p.step, p.traj0 + (uint32_t)m, STREAM_CONTROLLER);
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if ((mk[i][j] >> (8 * v)) & 1u) {
              mx = fmaxf(mx, lg[v]);
              const float s = lg[v] + gumbel(word_to_uniform(word_of(w, v)));
              if (s > best) { best = s; bidx = n + v; }
            }
          }
        }
      }
    }
    // reduce over the four lane groups (same row), lowest index on ties
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float ob = __shfl_xor(best, off);
      const int oi = __shfl_xor(bidx, off);
      const float om = __shfl_xor(mx, off);
      if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
      mx = fmaxf(mx, om);
    }
    if (g == 0) {
      s_best[wave][ml] = best;
      s_idx[wave][ml] = bidx;
      s_max[wave][ml] = mx;
    }
  }
  __syncthreads();

  if (p.mode == 0) {
    // combine waves; then probabilities
    if (tid < BM) {
      float best = -INFINITY, mx = -INFINITY;
      int bidx = -1;
      for (int w = 0; w < 4; ++w) {
        const float ob = s_best[w][tid];
        const int oi = s_idx[w][tid];
        if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
        mx = fmaxf(mx, s_max[w][tid]);
      }
      s_fin[tid][0] = mx;
      const int m = m0 + tid;
      if (m < p.M) p.action[m] = bidx;
    }
    __syncthreads();
    if (p.probs) {
      // sum of exp(l - max) over valid actions
#pragma unroll
      for (int j = 0; j < MBW; ++j) {
        const int ml = j * 16 + r16;
        const int m = m0 + ml;
        float se = 0.f;
        if (m < p.M) {
          const float mx = s_fin[ml][0];
#pragma unroll
          for (int i = 0; i < NBW; ++i) {
            const int nb = wave + 4 * i;
            if (nb >= nbtot) continue;
            const int n = nb * 16 + 4 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if ((mk[i][j] >> (8 * v)) & 1u) se += expf(acc[i][j][v] + p.bc[n + v] - mx);
          }
        }
        se += __shfl_xor(se, 16);
        se += __shfl_xor(se, 32);
        if (g == 0) s_best[wave][ml] = se;
      }
      __syncthreads();
      if (tid < BM) s_fin[tid][1] = s_best[0][tid] + s_best[1][tid] + s_best[2][tid] + s_best[3][tid];
      __syncthreads();
#pragma unroll
      for (int j = 0; j < MBW; ++j) {
        const int ml = j * 16 + r16;
        const int m = m0 + ml;
        if (m >= p.M) continue;
        const float mx = s_fin[ml][0], inv = s_fin[ml][1] > 0.f ? 1.0f / s_fin[ml][1] : 0.f;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          const int nb = wave + 4 * i;
          if (nb >= nbtot) continue;
          const int n = nb * 16 + 4 * g;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            if (n + v < A) {
              const bool ok = (mk[i][j] >> (8 * v)) & 1u;
              p.probs[(long)m * A + n + v] = ok ? expf(acc[i][j][v] + p.bc[n + v] - mx) * inv : 0.f;
            }
          }
        }
      }
    }
    return;
  }

  // rollout modes: one thread per row
  if (tid < BM) {
    const int m = m0 + tid;
    if (m < p.M) {
      float best = -INFINITY;
      int a = -1;
      for (int w = 0; w < 4; ++w) {
        const float ob = s_best[w][tid];
        const int oi = s_idx[w][tid];
        if (oi >= 0 && (a < 0 || ob > best || (ob == best && oi < a))) { best = ob; a = oi; }
      }
      ctrl_row_commit(p, rng, m, a, s_rho[tid][0], s_rho[tid][1], row_state(p, m));
    }
  }
}

// k_ctrl: controller on the pipelined GEMM core for A + 2 <= 64 * NBW
// outputs (all Nc weight rows of a row block in one tile).  The logit tile
// is staged through LDS as E[row][output]; each row is then handled by TPR
// adjacent threads, thread q taking the contiguous actions
// [q * APT, (q + 1) * APT) (APT a multiple of 4: one Philox block per four
// actions).  The mask bytes of those actions are fetched as 32-bit words
// before the GEMM when A % 4 == 0 (byte loads otherwise).
template <class C, class S>
__global__ void __launch_bounds__(C::NT) k_ctrl(const CtrlArgs p) {
  using DT = typename C::DT;
  constexpr int NBW = C::NBW, MBW = C::MBW, BM = C::BM;
  constexpr int TPR = C::NT / BM;               // threads per row
  constexpr int MAXB = (C::BN / TPR + 3) / 4;  // Philox blocks per thread
  constexpr int ELD = C::BN + 4;
  constexpr int E_BYTES = BM * ELD * 4;
  constexpr int LDS = C::LDS_BYTES > E_BYTES ? C::LDS_BYTES : E_BYTES;
  static_assert(C::NT % BM == 0 && (TPR & (TPR - 1)) == 0 && TPR <= 16, "row groups inside a wave");
  __shared__ __attribute__((aligned(16))) char lds_raw[LDS];

  const int m0 = blockIdx.x * BM;
  const int r = threadIdx.x / TPR, q = threadIdx.x % TPR;
  const int m = m0 + r;
  const bool row_ok = m < p.M;
  const int A = p.A;
  const int apt = (A + 4 * TPR - 1) / (4 * TPR) * 4;  // actions per thread
  const int a0 = q * apt;
  const bool want_action = p.mode != 2;

  // mask words of this thread's actions, ahead of the GEMM
  uint32_t mk[MAXB];
  const rsrc_t rmask = uniform_rsrc(p.mask + (long)m0 * A, (uint32_t)(max(0, min(BM, p.M - m0)) * A));
  const bool words = (A & 3) == 0 && (reinterpret_cast<uintptr_t>(p.mask) & 3) == 0;
#pragma unroll
  for (int b = 0; b < MAXB; ++b) {
    const int a = a0 + 4 * b;
    const bool ok = want_action && row_ok && p.N == 0 && 4 * b < apt && a < A;
    const uint32_t off = (uint32_t)(r * A + a);
    if (words) {
      mk[b] = bload4(rmask, ok ? off : kOffNone);
    } else {
      mk[b] = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        mk[b] |= bload1(rmask, ok && a + v < A ? off + v : kOffNone) << (8 * v);
    }
  }

  const Rng rng{p.k0, p.k1};
  const uint32_t traj = p.traj0 + (uint32_t)m;
  const bool flat_pick = want_action && row_ok && p.N == 0;
  // On the sixteen-wave direct tile, the Gumbel noise of all of the thread's
  // actions is drawn while the GEMM's first chunks load (it does not depend
  // on the logits).  It is drawn whatever the mask: the mask words are still
  // in flight there, and waiting for them would wait for the chunks too.
  // (On the four-wave 32-row tiles of the large rollout the same draw made
  // the controller slower, 12.0 -> 12.8 us per step.)
  constexpr bool kPre = IsGemmD<C>::value && C::NT >= 1024 && MAXB <= 5;
  float gq[kPre ? MAXB : 1][4];
  auto draw = [&]() {
    if constexpr (kPre) {
#pragma unroll
      for (int b = 0; b < MAXB; ++b) {
        if (flat_pick && 4 * b < apt && a0 + 4 * b < A) {
          const uint4 wd = rng.block((uint32_t)((a0 + 4 * b) >> 2), p.step, traj, STREAM_CONTROLLER);
#pragma unroll
          for (int v = 0; v < 4; ++v) gq[b][v] = gumbel(word_to_uniform(word_of(wd, v)));
        }
      }
    }
  };

  f32x4 acc[NBW][MBW];
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wc), p.ldk, p.ldk, 0, p.Nc, p.Nc);
  if constexpr (kPre)
    C::run(acc, w, ctrl_src<S>(p, m0, BM), (int)p.ldk, reinterpret_cast<DT*>(lds_raw), draw);
  else
    C::run(acc, w, ctrl_src<S>(p, m0, BM), (int)p.ldk, reinterpret_cast<DT*>(lds_raw));
  float* E = reinterpret_cast<float*>(lds_raw);
  if (C::kw() == 0) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const int wn = C::wn(), wmi = C::wm();
#pragma unroll
    for (int j = 0; j < MBW; ++j)
#pragma unroll
      for (int i = 0; i < NBW; ++i)
        *reinterpret_cast<f32x4*>(E + ((wmi * MBW + j) * 16 + r16) * ELD + (wn * NBW + i) * 16 + 4 * g) =
            acc[i][j];
  }
  __syncthreads();

  const float* lg = E + r * ELD;
  float best = -INFINITY, mx = -INFINITY;
  int bidx = -1;
  if (flat_pick) {
#pragma unroll
    for (int b = 0; b < MAXB; ++b) {
      if (mk[b] == 0) continue;  // no valid action in the block (or outside the range)
      const int a = a0 + 4 * b;
      uint4 wd = make_uint4(0u, 0u, 0u, 0u);
      if constexpr (!kPre) wd = rng.block((uint32_t)(a >> 2), p.step, traj, STREAM_CONTROLLER);
      const float4 l4 = *reinterpret_cast<const float4*>(lg + a);
      const float4 b4 = *reinterpret_cast<const float4*>(p.bc + a);
      const float lv[4] = {l4.x + b4.x, l4.y + b4.y, l4.z + b4.z, l4.w + b4.w};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if ((mk[b] >> (8 * v)) & 0xffu) {
          mx = fmaxf(mx, lv[v]);
          float gv;
          if constexpr (kPre) gv = gq[b][v];
          else gv = gumbel(word_to_uniform(word_of(wd, v)));
          const float sc = lv[v] + gv;
          if (sc > best) { best = sc; bidx = a + v; }
        }
      }
    }
  }
  // reduce over the TPR threads of the row, lowest index on ties
#pragma unroll
  for (int off = 1; off < TPR; off <<= 1) {
    const float ob = __shfl_xor(best, off);
    const int oi = __shfl_xor(bidx, off);
    const float om = __shfl_xor(mx, off);
    if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
    mx = fmaxf(mx, om);
  }
  if (p.mode == 0) {
    if (row_ok && q == 0) p.action[m] = bidx;
    if (p.probs) {
      float se = 0.f;
#pragma unroll
      for (int b = 0; b < MAXB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if ((mk[b] >> (8 * v)) & 0xffu) se += expf(lg[a0 + 4 * b + v] + p.bc[a0 + 4 * b + v] - mx);
#pragma unroll
      for (int off = 1; off < TPR; off <<= 1) se += __shfl_xor(se, off);
      const float inv = se > 0.f ? 1.0f / se : 0.f;
      if (row_ok) {
#pragma unroll
        for (int b = 0; b < MAXB; ++b)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int a = a0 + 4 * b + v;
            if (4 * b + v < apt && a < A)
              p.probs[(long)m * A + a] = ((mk[b] >> (8 * v)) & 0xffu) ? expf(lg[a] + p.bc[a] - mx) * inv : 0.f;
          }
      }
    }
    return;
  }
  if (p.N > 0) bidx = two_level_pick<TPR>(p, rng, lg, m, want_action && row_ok, q, traj);
  const int Ar = p.N > 0 ? p.N + 1 + p.Lc : A;  // the reward and done logit rows
  if (row_ok && q == 0)
    ctrl_row_commit(p, rng, m, bidx, lg[Ar] + p.bc[Ar], lg[Ar + 1] + p.bc[Ar + 1], row_state(p, m));
}

// Controller on the register-direct core: all Nc outputs x 16 rows.  Each row
// is handled by 16 lanes of one wave (four waves, four rows per wave), each
// lane taking the action blocks sub + 16 h, h < 4 (four actions and one
// Philox block each).  Requires A <= 256.  A small call is one chain of
// latencies, so everything the epilogue needs (mask bytes, biases, the row's
// bookkeeping) is loaded unconditionally before the product's operands, and
// the noise is drawn while those are in flight.  (Mask bytes read one at a
// time behind their range checks, and again with the biases for the
// probabilities, made a step for one state take 11.3 us.)
template <class R, class S>
__global__ void __launch_bounds__(R::MAXT) k_ctrl_rd(const CtrlArgs p) {
  using DT = typename R::DT;
  extern __shared__ __attribute__((aligned(16))) float lds_dyn[];
  const int m0 = blockIdx.x * R::BM;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ml = 4 * wave + (lane >> 4), sub = lane & 15;
  const int m = m0 + ml;
  const bool row_ok = wave < 4 && m < p.M;
  const int A = p.A;
  constexpr int NH = (R::BN + 63) / 64;  // blocks of four actions per lane
  const rsrc_t rm = uniform_rsrc(p.mask + (long)m0 * A, (uint32_t)(min(R::BM, p.M - m0) * A));
  const rsrc_t rb = uniform_rsrc(p.bc, (uint32_t)p.Nc * 4u);
  const bool pick = row_ok && p.mode != 2;
  uint32_t mb[NH][4];
  float4 bias[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const int a = 4 * (sub + 16 * h);
#pragma unroll
    for (int v = 0; v < 4; ++v) mb[h][v] = bload1(rm, pick && a + v < A ? (uint32_t)(ml * A + a + v) : kOffNone);
    bias[h] = as_float4(bload16(rb, pick ? 4u * (uint32_t)a : kOffNone));
  }
  RowState rs{};
  float br = 0.f, bd = 0.f;
  if (p.mode != 0 && row_ok && sub == 0) {
    rs = row_state(p, m);
    br = p.bc[A];
    bd = p.bc[A + 1];
  }
  const Rng rng{p.k0, p.k1};
  float gn[NH][4];
  auto noise = [&]() {
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int b = sub + 16 * h;
      if (pick && 4 * b < A) {
        const uint4 w = rng.block((uint32_t)b, p.step, p.traj0 + (uint32_t)m, STREAM_CONTROLLER);
#pragma unroll
        for (int v = 0; v < 4; ++v) gn[h][v] = gumbel(word_to_uniform(word_of(w, v)));
      }
    }
  };
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wc), p.ldk, p.ldk, 0, R::BN, p.Nc);
  R::run(lds_dyn, w, ctrl_src<S>(p, m0, R::BM), (int)p.ldk, noise);
  if (wave >= 4) return;  // rows live in the first four waves; no barrier below
  const float* lg = R::E(lds_dyn) + ml * R::ELD;
  float best = -INFINITY, mx = -INFINITY;
  int bidx = -1;
  float l[NH][4];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    const float bv[4] = {bias[h].x, bias[h].y, bias[h].z, bias[h].w};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 4 * (sub + 16 * h) + v;
      l[h][v] = -INFINITY;
      if (mb[h][v]) {
        l[h][v] = lg[a] + bv[v];
        mx = fmaxf(mx, l[h][v]);
        const float sc = l[h][v] + gn[h][v];
        if (sc > best) { best = sc; bidx = a; }
      }
    }
  }
  // reduce over the 16 lanes of the row, lowest index on ties
#pragma unroll
  for (int off = 8; off >= 1; off >>= 1) {
    const float ob = __shfl_xor(best, off);
    const int oi = __shfl_xor(bidx, off);
    const float om = __shfl_xor(mx, off);
    if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
    mx = fmaxf(mx, om);
  }
  if (p.mode == 0) {
    if (row_ok && sub == 0) p.action[m] = bidx;
    if (p.probs) {
      float se = 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          l[h][v] = mb[h][v] ? expf(l[h][v] - mx) : 0.f;
          se += l[h][v];
        }
#pragma unroll
      for (int off = 8; off >= 1; off >>= 1) se += __shfl_xor(se, off);
      const float inv = se > 0.f ? 1.0f / se : 0.f;
#pragma unroll
      for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int a = 4 * (sub + 16 * h) + v;
          if (row_ok && a < A) p.probs[(long)m * A + a] = l[h][v] * inv;
        }
    }
    return;
  }
  if (row_ok && sub == 0) ctrl_row_commit(p, rng, m, bidx, lg[A] + br, lg[A + 1] + bd, rs);
}

// The rollout's decision where the mixture kernel of the step before has
// computed the logits' h part (MdnArgs::lh): 16 rows per work-group, logits =
// lh + W_c[:, 0 .. Z-1] q(z) + b_c, so that the product is Z deep instead of
// Z + H, and four waves of interleaved 16-output blocks, U at a time, pick from
// their accumulators.  A chain of latencies: every load of a group of blocks
// is issued before the first is used, the noise is drawn meanwhile.  TL: the
// two-level controller, whose picks need whole rows, goes through LDS.
// fp32 only (ctrl_h_wanted).  At B 301, A 50, H 368, Z 40 5.1 us per step,
// against 9.8 for the whole product.
template <int U, bool TL>
__global__ void __launch_bounds__(256) k_ctrl_z(const CtrlArgs p) {
  using DT = float;
  constexpr int VEC = DType<DT>::VEC, KS = Mfma<DT>::KSLICE;
  constexpr int SL = 4;  // K slices loaded together
  constexpr int ELD = 324;                     // staged row (at most 320 logits)
  __shared__ float s_best[4][16];
  __shared__ int s_idx[4][16];
  __shared__ float s_rho[2][16];
  __shared__ __attribute__((aligned(16))) float E[TL ? 16 * ELD : 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int m0 = blockIdx.x * 16, m = m0 + r16, rows = min(16, p.M - m0);
  const int A = p.A, Ar = TL ? p.N + 1 + p.Lc : A;  // the reward logit's row
  const bool pick = p.mode != 2;
  const int nbtot = p.Nc / 16, nb0 = pick ? 0 : Ar / 16;  // the tail step: the reward and done rows only
  RowState rs{};
  if (tid < 16 && m < p.M) rs = row_state(p, m);
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wc), p.ldk, p.ldk, 0, p.Nc, p.Nc);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x), p.ldx, p.ldx, m0, 16, p.M);
  const uint32_t ldl = (uint32_t)p.ldlh;
  const rsrc_t rl = uniform_rsrc(p.lh ? p.lh + (long)m0 * p.ldlh : nullptr,
                                 p.lh ? ((uint32_t)(rows - 1) * ldl + (uint32_t)p.Nc) * 4u : 0u);
  const rsrc_t rb = uniform_rsrc(p.bc, (uint32_t)p.Nc * 4u);
  const rsrc_t rm = uniform_rsrc(p.mask + (long)m0 * A, (uint32_t)(rows * A));
  const Rng rng{p.k0, p.k1};
  const uint32_t traj = p.traj0 + (uint32_t)m;
  const int ns = (p.Z + KS - 1) / KS;
  float best = -INFINITY;
  int bidx = -1;
  for (int i0 = nb0 + wave; i0 < nbtot; i0 += 4 * U) {
    uint32_t mb[U][4];
    f32x4 acc[U];
    float4 bias[U];
    uint4 wf[U][SL], xf[SL];
    auto load = [&](int s0) {
#pragma unroll
      for (int s = 0; s < SL; ++s) {
        const int k = (s0 + s) * KS + g * VEC;
        xf[s] = x.load(x.row(r16), k, p.Z);
#pragma unroll
        for (int i = 0; i < U; ++i) {
          const int nb = i0 + 4 * i;
          wf[i][s] = w.load(w.row(nb * 16 + r16), nb < nbtot ? k : p.Z, p.Z);
        }
      }
    };
    load(0);
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int n = (i0 + 4 * i) * 16 + 4 * g;
      const bool in = i0 + 4 * i < nbtot;
      const uint4 h = bload16(rl, in && m < p.M ? ((uint32_t)r16 * ldl + (uint32_t)n) * 4u : kOffNone);
      acc[i] = f32x4{__uint_as_float(h.x), __uint_as_float(h.y), __uint_as_float(h.z), __uint_as_float(h.w)};
      bias[i] = as_float4(bload16(rb, in ? (uint32_t)n * 4u : kOffNone));
#pragma unroll
      for (int v = 0; v < 4; ++v)
        mb[i][v] = !TL && pick ? bload1(rm, in && m < p.M && n + v < A ? (uint32_t)(r16 * A + n + v) : kOffNone) : 0u;
    }
    float gn[U][4];
    if (!TL && pick) {
#pragma unroll
      for (int i = 0; i < U; ++i) {
        const int n = (i0 + 4 * i) * 16 + 4 * g;
        if (n < A) {
          const uint4 wd = rng.block((uint32_t)(n >> 2), p.step, traj, STREAM_CONTROLLER);
#pragma unroll
          for (int v = 0; v < 4; ++v) gn[i][v] = gumbel(word_to_uniform(word_of(wd, v)));
        }
      }
    }
    for (int s0 = 0; s0 < ns; s0 += SL) {
      if (s0 > 0) load(s0);
#pragma unroll
      for (int s = 0; s < SL; ++s)
#pragma unroll
        for (int i = 0; i < U; ++i) Mfma<DT>::step(acc[i], wf[i][s], xf[s]);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int n = (i0 + 4 * i) * 16 + 4 * g;
      if (i0 + 4 * i >= nbtot) continue;
      const float lv[4] = {acc[i][0] + bias[i].x, acc[i][1] + bias[i].y, acc[i][2] + bias[i].z, acc[i][3] + bias[i].w};
      if constexpr (TL) *reinterpret_cast<f32x4*>(E + r16 * ELD + n) = acc[i];  // the picks add the bias
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (n + v == Ar) s_rho[0][r16] = lv[v];
        if (n + v == Ar + 1) s_rho[1][r16] = lv[v];
        if (!TL && mb[i][v]) {
          const float sc = lv[v] + gn[i][v];
          if (sc > best) { best = sc; bidx = n + v; }
        }
      }
    }
  }
  if constexpr (TL) {
    __syncthreads();
    const int r = tid >> 4, q = tid & 15;
    const int a = two_level_pick<16>(p, rng, E + r * ELD, m0 + r, pick && m0 + r < p.M, q, p.traj0 + (uint32_t)(m0 + r));
    if (q == 0) s_idx[0][r] = a;
    __syncthreads();
    if (tid < 16 && m < p.M) ctrl_row_commit(p, rng, m, s_idx[0][tid], s_rho[0][tid], s_rho[1][tid], rs);
    return;
  }
  // reduce over the four lane groups (same row), then the waves, lowest index
  // on ties
#pragma unroll
  for (int off = 16; off <= 32; off <<= 1) {
    const float ob = __shfl_xor(best, off);
    const int oi = __shfl_xor(bidx, off);
    if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
  }
  if (g == 0) {
    s_best[wave][r16] = best;
    s_idx[wave][r16] = bidx;
  }
  __syncthreads();
  if (tid < 16 && m < p.M) {
    best = -INFINITY;
    bidx = -1;
#pragma unroll
    for (int w4 = 0; w4 < 4; ++w4) {
      const float ob = s_best[w4][tid];
      const int oi = s_idx[w4][tid];
      if (oi >= 0 && (bidx < 0 || ob > best || (ob == best && oi < bidx))) { best = ob; bidx = oi; }
    }
    ctrl_row_commit(p, rng, m, bidx, s_rho[0][tid], s_rho[1][tid], rs);
  }
}

namespace {

// Controller tiles by dtype.
template <typename DT> struct Cfgs;
template <> struct Cfgs<float> {
  static constexpr bool kXL = false;  // fp32 calls this large take the 32-row controller tiles
  template <int NB> using CtrlLarge = Gemm<float, NB, 4, 4, 1, 1, 32, 3>;  // 64NB x 64
  template <int NB> using CtrlLargeX = GemmD<float, NB, 2, 4, 1, 3>;      // 64NB x 32
  template <int NB> using CtrlXL = CtrlLargeX<NB>;
  static constexpr int WIDE_BKC = 64;
};
template <> struct Cfgs<bf16_t> {
  static constexpr bool kXL = true;
  template <int NB> using CtrlLarge = Gemm<bf16_t, NB, 4, 4, 1, 1, 64, 2>;
  template <int NB> using CtrlLargeX = GemmD<bf16_t, NB, 2, 4, 1, 3>;
  // 64-row controller tiles, three stages: half the weight re-reads of the
  // 32-row tiles.  With five 64-output blocks (A up to 318) sixteen waves of
  // one 16-row block each, which hide more of the chunk loads' latency than
  // eight waves of two (xlarge controller 23.9 -> 22.6 us per step; four
  // waves of four blocks: 32 us)
  template <int NB> using CtrlXL = std::conditional_t<NB == 5, GemmD<bf16_t, NB, 1, 4, 4, 3>,
                                                      GemmD<bf16_t, NB, 2, 4, 2, 3>>;
  static constexpr int WIDE_BKC = 128;
};

// The 64-row controller tiles serve calls that give every CU at least one.
constexpr long kXLTiles = 256;

// The register-direct controller serves calls with at most this many rows,
// when the K slices fit SMAX per wave on the compiled block size.
constexpr int kRdCtrlRows = 1024;
template <class C, class S>
hipError_t launch_ctrl_cfg(const CtrlArgs& a, hipStream_t s) {
  static const char* const names[2][5] = {{"ctrl/32x64", "ctrl/32x128", "ctrl/32x192", "", "ctrl/32x320"},
                                          {"ctrl/64x64", "ctrl/64x128", "ctrl/64x192", "", "ctrl/64x320"}};
  static_assert(C::BM == 32 || C::BM == 64, "named tiles");
  return launch(names[C::BM / 64][C::BN / 64 - 1], k_ctrl<C, S>, dim3((a.M + C::BM - 1) / C::BM), dim3(C::NT), 0, s, a);
}

template <class S, int NBW, int MBW>
hipError_t launch_ctrl_wide(const CtrlArgs& a, hipStream_t s) {
  constexpr int BM = 16 * MBW;
  return launch("ctrl/wide", k_ctrl_wide<S, NBW, MBW, Cfgs<typename S::DT>::WIDE_BKC>,
                dim3((a.M + BM - 1) / BM), dim3(256), 0, s, a);
}

template <class R, class S>
hipError_t launch_ctrl_rd(const CtrlArgs& a, int nw, hipStream_t s) {
  const size_t lds = R::lds_bytes(nw);
  hipError_t e = allow_lds(k_ctrl_rd<R, S>, lds);
  if (e != hipSuccess) return e;
  return launch("ctrl/rd", k_ctrl_rd<R, S>, dim3((a.M + R::BM - 1) / R::BM), dim3(64 * nw), lds, s, a);
}

template <class C>
hipError_t launch_ctrl_logits_cfg(CtrlArgs a, hipStream_t s) {
  a.map = tile_map((a.Nc + C::BN - 1) / C::BN, (a.M + C::BM - 1) / C::BM,
                   (size_t)a.Nc * a.ldk * sizeof(typename C::DT));
  return launch("ctrl/logits", k_ctrl_logits<C>, dim3(grid_of(a.map)), dim3(C::NT), 0, s, a);
}

// The largest tile that still gives every CU one, else the smallest (the
// same product shape as the gates', whose tiles' times per CU order so).
template <typename DT>
hipError_t launch_ctrl_logits(const CtrlArgs& a, hipStream_t s) {
  auto tiles = [&](int bn, int bm) { return (long)((a.Nc + bn - 1) / bn) * ((a.M + bm - 1) / bm); };
  if (tiles(128, 128) >= kCUs) return launch_ctrl_logits_cfg<GemmD<DT, 4, 2, 2, 4, 2>>(a, s);
  if (tiles(128, 64) >= kCUs) return launch_ctrl_logits_cfg<GemmD<DT, 4, 2, 2, 2, 2>>(a, s);
  return launch_ctrl_logits_cfg<GemmD<DT, 4, 1, 1, 4, 4>>(a, s);
}

}  // namespace

// S: activation source (SrcX for the rollout's X_t, SrcZH for the step).
template <class S>
hipError_t launch_ctrl(const CtrlArgs& a, hipStream_t s) {
  using DT = typename S::DT;
  using Cf = Cfgs<DT>;
  const int nbtot = a.Nc / 16;
  const int nbw = (nbtot + 3) / 4;  // output blocks per wave over four waves
  // the two-level controller of the controller step, and in rollouts where
  // its logit rows do not fit the staged tiles: the logits are stored (into
  // probs for the step, the workspace in a rollout), then picked per row
  if (a.N > 0 && (a.mode == 0 || nbw > 5)) {
    CtrlArgs g = a;
    g.logits_out = a.mode == 0 ? a.probs : a.lg_ws;
    g.ldl = a.mode == 0 ? a.N + 1 + a.Lc : a.Nc;
    g.ncol = a.mode == 0 ? a.N + 1 + a.Lc : a.Nc;
    if (!g.logits_out) return hipErrorInvalidValue;
    hipError_t e;
    if constexpr (!S::kTwo) e = launch_ctrl_logits<DT>(g, s);
    else if (nbw <= 8) e = launch_ctrl_wide<S, 8, 2>(g, s);
    else if (nbw <= 12) e = launch_ctrl_wide<S, 12, 2>(g, s);
    else if (nbw <= 17) e = launch_ctrl_wide<S, 17, 1>(g, s);
    else if (nbw <= 24) e = launch_ctrl_wide<S, 24, 1>(g, s);
    else if (nbw <= 33) e = launch_ctrl_wide<S, 33, 1>(g, s);
    else return hipErrorInvalidValue;
    if (e != hipSuccess) return e;
    // one block per lane of either row where it fits, two of the xfers', else
    // four of both: a load that only reads past the row takes as long as the
    // others (B 4096, N 288, L 200: a step of the rollout 90.8 -> 88.5 us
    // against four blocks of each)
    const dim3 grid((unsigned)((a.M + 3) / 4));
    const bool x1 = a.N + 1 <= 256, x2 = a.N + 1 <= 512, l1 = a.Lc <= 256;
    if (x1 && l1) return launch("ctrl/rows", k_ctrl_rows<1, 1>, grid, dim3(256), 0, s, g);
    if (x2 && l1) return launch("ctrl/rows", k_ctrl_rows<2, 1>, grid, dim3(256), 0, s, g);
    return launch("ctrl/rows", k_ctrl_rows<kRowBlk, kRowBlk>, grid, dim3(256), 0, s, g);
  }
  // (otherwise the two-level controller runs on the kernels that stage whole logit rows)
  if (a.M <= kRdCtrlRows && nbtot <= 9 && a.N == 0) {
    const int nb = nbtot <= 1 ? 1 : nbtot <= 2 ? 2 : nbtot <= 3 ? 3 : nbtot <= 5 ? 5 : 9;
    const int smax = nb <= 5 ? 8 : 4;  // register budget
    // eight waves where their partial tiles fit the LDS: the K slices of a
    // wave are a serial chain (a step for one state, K 288: 9.3 us on four).
    // A bf16 rollout, whose sums keep one order (KSum), takes four, and where
    // K needs more than six the staged tiles.
    constexpr bool kOrder = sizeof(DT) == 2 && !S::kTwo;
    const int nw = rd_waves((int)a.ldk, Mfma<DT>::KSLICE, smax, nb <= 5 && !kOrder ? 8 : 4);
    const bool fits9 = GemmRD<DT, 9, 1, 4, 512>::lds_bytes(nw) <= kRdLdsMax;
    if (nw <= 8 && (fits9 || (nb <= 5 && !kOrder))) {
      switch (nb) {
        case 1: return launch_ctrl_rd<GemmRD<DT, 1, 1, 8, 512>, S>(a, nw, s);
        case 2: return launch_ctrl_rd<GemmRD<DT, 2, 1, 8, 512>, S>(a, nw, s);
        case 3: return launch_ctrl_rd<GemmRD<DT, 3, 1, 8, 512>, S>(a, nw, s);
        case 5: return launch_ctrl_rd<GemmRD<DT, 5, 1, 8, 512>, S>(a, nw, s);
        default: return launch_ctrl_rd<GemmRD<DT, 9, 1, 4, 512>, S>(a, nw, s);
      }
    }
  }
  const int nb = nbw;
  if constexpr (S::kTwo) {
    if (nb <= 1) return launch_ctrl_cfg<typename Cf::template CtrlLarge<1>, S>(a, s);
    if (nb <= 2) return launch_ctrl_cfg<typename Cf::template CtrlLarge<2>, S>(a, s);
    if (nb <= 3) return launch_ctrl_cfg<typename Cf::template CtrlLarge<3>, S>(a, s);
    if (nb <= 5) return launch_ctrl_cfg<typename Cf::template CtrlLarge<5>, S>(a, s);
  } else {
    // 64-row tiles once they still give every CU one, 32-row tiles below
    if (Cf::kXL && (long)(a.M + 63) / 64 >= kXLTiles) {
      if (nb <= 1) return launch_ctrl_cfg<typename Cf::template CtrlXL<1>, S>(a, s);
      if (nb <= 2) return launch_ctrl_cfg<typename Cf::template CtrlXL<2>, S>(a, s);
      if (nb <= 3) return launch_ctrl_cfg<typename Cf::template CtrlXL<3>, S>(a, s);
      if (nb <= 5) return launch_ctrl_cfg<typename Cf::template CtrlXL<5>, S>(a, s);
    }
    if (nb <= 1) return launch_ctrl_cfg<typename Cf::template CtrlLargeX<1>, S>(a, s);
    if (nb <= 2) return launch_ctrl_cfg<typename Cf::template CtrlLargeX<2>, S>(a, s);
    if (nb <= 3) return launch_ctrl_cfg<typename Cf::template CtrlLargeX<3>, S>(a, s);
    if (nb <= 5) return launch_ctrl_cfg<typename Cf::template CtrlLargeX<5>, S>(a, s);
  }
  if (nb <= 8) return launch_ctrl_wide<S, 8, 2>(a, s);
  if (nb <= 12) return launch_ctrl_wide<S, 12, 2>(a, s);
  if (nb <= 17) return launch_ctrl_wide<S, 17, 1>(a, s);
  if (nb <= 24) return launch_ctrl_wide<S, 24, 1>(a, s);
  if (nb <= 33) return launch_ctrl_wide<S, 33, 1>(a, s);
  return hipErrorInvalidValue;
}

hipError_t launch_ctrl_z(const CtrlArgs& a, hipStream_t s) {
  const dim3 grid((unsigned)((a.M + 15) / 16));
  const int nbw = (a.Nc / 16 + 3) / 4;
  if (a.N > 0) return launch("ctrl/z", k_ctrl_z<3, true>, grid, dim3(256), 0, s, a);
  if (nbw <= 1) return launch("ctrl/z", k_ctrl_z<1, false>, grid, dim3(256), 0, s, a);
  if (nbw <= 2) return launch("ctrl/z", k_ctrl_z<2, false>, grid, dim3(256), 0, s, a);
  return launch("ctrl/z", k_ctrl_z<3, false>, grid, dim3(256), 0, s, a);
}

template hipError_t launch_ctrl<SrcX<float>>(const CtrlArgs&, hipStream_t);
template hipError_t launch_ctrl<SrcX<bf16_t>>(const CtrlArgs&, hipStream_t);

hipError_t launch_controller_step(const Packed& P, int B, uint32_t traj0, const float* z,
                                  const float* h, const uint8_t* mask, uint32_t k0, uint32_t k1,
                                  uint32_t step, float* probs, int32_t* action, hipStream_t s) {
  const Layout& L = P.L;
  const char* base = reinterpret_cast<const char*>(P.base);
  CtrlArgs ca{};
  ca.Wc = base + L.off_Wc;
  ca.bc = reinterpret_cast<const float*>(base + L.off_bc);
  ca.ldk = L.ldk;
  ca.Z = L.Z; ca.H = L.H; ca.A = L.A; ca.Nc = L.Nc; ca.M = B;
  ca.z = z;
  ca.h = h;
  ca.mask = mask;
  ca.k0 = k0; ca.k1 = k1; ca.step = step; ca.traj0 = traj0;
  ca.mode = 0;
  ca.probs = probs;
  ca.action = action;
  ca.N = L.N;
  ca.Lc = L.Lc;
  if (L.dt == 0) return launch_ctrl<SrcZH<float>>(ca, s);
  return launch_ctrl<SrcZH<bf16_t>>(ca, s);
}

}  // namespace wm
