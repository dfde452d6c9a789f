// HIP kernels of libwm for gfx950 (MI355X).
//
// The dream rollout runs three kernels per step, each a GEMM on the MFMA
// units with the step's arithmetic fused into its epilogue:
//   k_ctrl   controller logits W_c [z_t, h_t] (+ reward/done rows on h_t),
//            masked Gumbel-max action, resolution of the previous
//            transition's reward and done flag;
//   k_gates  gate GEMM [z_t, h_t] x W^T plus the gathered one-hot column,
//            LSTM cell, state commit (frozen rows copy their state);
//   k_mdn    mixture head on h_{t+1}, Gumbel-max component pick per latent
//            dim, Box-Muller draw, z_{t+1} commit.
// The activations of step t are one matrix X_t = [q(z_t) | h_t | 0] in the
// compute type (q: round to the compute type), so every GEMM streams a
// single K-contiguous operand: the gate and controller GEMMs read X_t from
// column 0, the mixture head reads X_{t+1} from column Z, k_gates writes h_{t+1}
// and k_mdn q(z_{t+1}) into X_{t+1}.
// The NLL pass runs k_gates once per step (teacher-forced), then one k_mdn
// over all T*B rows with a log-likelihood epilogue, then a deterministic
// reduction.  Nothing here allocates memory.
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
// Packing (one-time): canonical fp32 -> kernel layout, rounded to DT.
// ===========================================================================
template <typename DT>
__global__ void k_pack(const Layout L, char* base, const float* __restrict__ W_g,
                       const float* __restrict__ b_g, const float* __restrict__ W_m,
                       const float* __restrict__ b_m, const float* __restrict__ w_r,
                       const float* __restrict__ b_r, const float* __restrict__ w_d,
                       const float* __restrict__ b_d, const float* __restrict__ W_c,
                       const float* __restrict__ b_c) {
  const int Z = L.Z, H = L.H, A = L.A, K = L.K, Q = L.Q;
  const long cg = Z + A + H;  // canonical W_g row length
  const int section = blockIdx.y;
  const long stride = (long)gridDim.x * blockDim.x;
  const long i0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  DT* Wg = reinterpret_cast<DT*>(base + L.off_Wg);
  DT* WaT = reinterpret_cast<DT*>(base + L.off_WaT);
  float* bg = reinterpret_cast<float*>(base + L.off_bg);
  DT* Wm = reinterpret_cast<DT*>(base + L.off_Wm);
  float* bm = reinterpret_cast<float*>(base + L.off_bm);
  DT* Wc = reinterpret_cast<DT*>(base + L.off_Wc);
  float* bc = reinterpret_cast<float*>(base + L.off_bc);
  const int head0 = 16 * Q * (Z / 4);
  if (section == 0) {
    for (long idx = i0; idx < (long)4 * H * L.ldk; idx += stride) {
      const int r = (int)(idx / L.ldk), col = (int)(idx % L.ldk);
      const long crow = (long)(r % 4) * H + r / 4;
      float v = 0.f;
      if (col < Z) v = W_g[crow * cg + col];
      else if (col < Z + H) v = W_g[crow * cg + A + col];
      DType<DT>::store(Wg, idx, v);
    }
  } else if (section == 1) {
    for (long idx = i0; idx < (long)A * 4 * H; idx += stride) {
      const int a = (int)(idx / (4 * H)), r = (int)(idx % (4 * H));
      const long crow = (long)(r % 4) * H + r / 4;
      DType<DT>::store(WaT, idx, W_g[crow * cg + Z + a]);
    }
  } else if (section == 2) {
    for (long idx = i0; idx < 4 * H; idx += stride) bg[idx] = b_g[(idx % 4) * H + idx / 4];
  } else if (section == 3 || section == 4) {
    const long n = section == 3 ? (long)L.Nm * L.ldh : (long)L.Nm;
    for (long idx = i0; idx < n; idx += stride) {
      const int row = section == 3 ? (int)(idx / L.ldh) : (int)idx;
      const int col = section == 3 ? (int)(idx % L.ldh) : 0;
      float v = 0.f;
      if (col < H) {
        if (row >= head0) {
          const int hr = row - head0;
          if (section == 3) v = hr == 0 ? w_r[col] : (hr == 1 ? w_d[col] : 0.f);
          else v = hr == 0 ? b_r[0] : (hr == 1 ? b_d[0] : 0.f);
        } else {
          const int J = row / (16 * Q), rem = row % (16 * Q);
          const int q = rem / 16, g = (rem % 16) / 4, vv = rem % 4;
          const int j = 4 * J + g, f = 4 * q + vv;
          long canon = -1;
          if (f < K) canon = (long)j * K + f;
          else if (f < 2 * K) canon = (long)Z * K + (long)j * K + (f - K);
          else if (f < 3 * K) canon = 2L * Z * K + (long)j * K + (f - 2 * K);
          if (canon >= 0) v = section == 3 ? W_m[canon * H + col] : b_m[canon];
        }
      }
      if (section == 3) DType<DT>::store(Wm, idx, v);
      else bm[idx] = v;
    }
  } else if (section == 5) {
    for (long idx = i0; idx < (long)L.Nc * L.ldk; idx += stride) {
      const int row = (int)(idx / L.ldk), col = (int)(idx % L.ldk);
      float v = 0.f;
      if (col < Z + H) {
        const int Ac = L.Ac;
        if (row < Ac) v = W_c[(long)row * (Z + H) + col];
        else if (row == Ac && col >= Z) v = w_r[col - Z];
        else if (row == Ac + 1 && col >= Z) v = w_d[col - Z];
      }
      DType<DT>::store(Wc, idx, v);
    }
  } else if (section == 6) {
    for (long idx = i0; idx < L.Nc; idx += stride)
      bc[idx] = idx < L.Ac ? b_c[idx] : (idx == L.Ac ? b_r[0] : (idx == L.Ac + 1 ? b_d[0] : 0.f));
  } else if constexpr (sizeof(DT) == 4) {
    if (section == 7) {  // WhT[i][r] = Wg[r][Z + i]
      float* WhT = reinterpret_cast<float*>(base + L.off_WhT);
      for (long idx = i0; idx < (long)H * 4 * H; idx += stride) {
        const int i = (int)(idx / (4 * H)), r = (int)(idx % (4 * H));
        WhT[idx] = W_g[((long)(r % 4) * H + r / 4) * cg + A + Z + i];
      }
    } else if (section == 8) {  // WmT[i][r] = Wm[r][i], zero past Nm
      float* WmT = reinterpret_cast<float*>(base + L.off_WmT);
      for (long idx = i0; idx < (long)H * L.NmP; idx += stride) {
        const int i = (int)(idx / L.NmP), row = (int)(idx % L.NmP);
        float v = 0.f;
        if (row >= head0 && row < L.Nm) {
          const int hr = row - head0;
          v = hr == 0 ? w_r[i] : (hr == 1 ? w_d[i] : 0.f);
        } else if (row < head0) {
          const int J = row / (16 * Q), rem = row % (16 * Q);
          const int q = rem / 16, g = (rem % 16) / 4, vv = rem % 4;
          const int j = 4 * J + g, f = 4 * q + vv;
          long canon = -1;
          if (f < K) canon = (long)j * K + f;
          else if (f < 2 * K) canon = (long)Z * K + (long)j * K + (f - K);
          else if (f < 3 * K) canon = 2L * Z * K + (long)j * K + (f - 2 * K);
          if (canon >= 0) v = W_m[canon * H + i];
        }
        WmT[idx] = v;
      }
    }
  }
}

// ===========================================================================
// k_gates: g = W [q(z) | h]^T + WaT[a] + b, LSTM cell, commit.
// Rollout mode: a < 0 marks a frozen row, whose state is copied forward.
// NLL mode: every row is live; a outside [0, A) adds no column.
// ===========================================================================
// Element-wise side of the gate kernels for rows m0 .. m0+rows-1 of a tile.
// Every access goes through a range-checked buffer resource and elements
// that must not be touched get the offset kOffNone, so that the loads are
// straight-line code issued together, before any of their values is used.
// load() fetches what the cell needs besides the GEMM (bias plus the
// gathered one-hot column, cell state, and for a frozen row its h);
// commit() runs the LSTM cell on the four gate pre-activations i, f, g, o
// and stores h_t+1 into X_t+1 and c (a frozen rollout row keeps its state).
struct GateIn {
  float4 add;  // bias + one-hot column, per gate
  float c;     // cell state c_t
  float hprev; // h_t (frozen rows only)
  bool live;
};

template <typename DT>
struct GateIO {
  rsrc_t rc, rxi, rxo, rw, rb, rht, rct;
  int H, A;
  uint32_t ldxb;  // X row stride in bytes
  bool nll;

  __device__ GateIO(const GatesArgs& p, int m0, int rows) {
    H = p.H;
    A = p.A;
    nll = p.nll_mode != 0;
    const long mval = max(0, min(rows, p.M - m0));
    const uint32_t hb = (uint32_t)(mval * H * 4);
    ldxb = (uint32_t)(p.ldx * (long)sizeof(DT));
    const uint32_t xb = mval ? (uint32_t)(((mval - 1) * p.ldx + H) * (long)sizeof(DT)) : 0u;
    rc = make_rsrc(p.c + (long)m0 * H, hb);
    rxi = make_rsrc(reinterpret_cast<const DT*>(p.x_in) + (long)m0 * p.ldx + p.Z, xb);
    rxo = make_rsrc(reinterpret_cast<DT*>(p.x_out) + (long)m0 * p.ldx + p.Z, xb);
    rw = make_rsrc(p.WaT, (uint32_t)((long)A * 4 * H * (long)sizeof(DT)));
    rb = make_rsrc(p.bg, (uint32_t)(16 * H));
    rht = make_rsrc(p.h_trace ? p.h_trace + (long)m0 * H : nullptr, p.h_trace ? hb : 0u);
    rct = make_rsrc(p.c_trace ? p.c_trace + (long)m0 * H : nullptr, p.c_trace ? hb : 0u);
  }

  // tile row ml, hidden unit u, action a of the row; ok: inside the call
  __device__ __forceinline__ GateIn load(int ml, int u, int a, bool ok) const {
    GateIn in;
    in.live = nll || a >= 0;
    const uint32_t ec = ((uint32_t)ml * H + u) * 4u;
    const uint4 b = bload16(rb, ok ? (uint32_t)u * 16u : kOffNone);
    const bool gather = ok && a >= 0 && a < A;
    const uint32_t ew = ((uint32_t)a * 4u * H + 4u * u) * (uint32_t)sizeof(DT);
    float4 w;
    if constexpr (sizeof(DT) == 4) {
      const uint4 v = bload16(rw, gather ? ew : kOffNone);
      w = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    } else {
      const uint2 v = bload8(rw, gather ? ew : kOffNone);
      w = make_float4(bf16_bits_to_f32(v.x & 0xffffu), bf16_bits_to_f32(v.x >> 16),
                      bf16_bits_to_f32(v.y & 0xffffu), bf16_bits_to_f32(v.y >> 16));
    }
    in.add = make_float4(__uint_as_float(b.x) + w.x, __uint_as_float(b.y) + w.y,
                         __uint_as_float(b.z) + w.z, __uint_as_float(b.w) + w.w);
    in.c = __uint_as_float(bload4(rc, ok ? ec : kOffNone));
    const uint32_t ex = (uint32_t)ml * ldxb + (uint32_t)u * (uint32_t)sizeof(DT);
    const uint32_t ox = ok && !in.live ? ex : kOffNone;
    if constexpr (sizeof(DT) == 4) in.hprev = __uint_as_float(bload4(rxi, ox));
    else in.hprev = bf16_bits_to_f32(bload2(rxi, ox));
    return in;
  }

  __device__ __forceinline__ void commit(int ml, int u, bool ok, const GateIn& in, float pi, float pf,
                                         float pg, float po) const {
    const float cn = fsigmoid(pf + in.add.y) * in.c + fsigmoid(pi + in.add.x) * ftanh_cell<DT>(pg + in.add.z);
    const float hn = DType<DT>::round(fsigmoid(po + in.add.w) * ftanh_cell<DT>(cn));
    const float cv = in.live ? cn : in.c;
    const float hv = in.live ? hn : in.hprev;
    const uint32_t ec = ((uint32_t)ml * H + u) * 4u;
    const uint32_t ex = (uint32_t)ml * ldxb + (uint32_t)u * (uint32_t)sizeof(DT);
    bstore4(rc, ok && in.live ? ec : kOffNone, __float_as_uint(cv));
    if constexpr (sizeof(DT) == 4) bstore4(rxo, ok ? ex : kOffNone, __float_as_uint(hv));
    else bstore2(rxo, ok ? ex : kOffNone, f32_to_bf16_bits(hv));
    bstore4(rht, ok ? ec : kOffNone, __float_as_uint(hv));  // dropped without traces
    bstore4(rct, ok ? ec : kOffNone, __float_as_uint(cv));
  }
};

// Element-wise side of the pipelined gate kernels for four consecutive hidden
// units u0 .. u0+3 of one tile row, so that cell state, h, traces and the
// gathered one-hot columns move in 16-byte (8-byte for bf16 h) pieces.
// Same masking scheme as GateIO: range-checked buffer accesses, kOffNone for
// elements that must not be touched.
struct Gate4In {
  float4 add[4];  // bias + one-hot column of unit u0 + t, per gate
  float4 c;       // cell states of the four units
  float4 hprev;   // h_t of the four units (frozen rows only)
  bool live;
};

template <typename DT>
struct Gate4IO {
  rsrc_t rc, rxi, rxo, rw, rb, rht, rct;
  int H, A;
  uint32_t ldxb;
  bool nll, trace;

  __device__ Gate4IO(const GatesArgs& p, int m0, int rows) {
    H = p.H;
    A = p.A;
    nll = p.nll_mode != 0;
    trace = p.h_trace != nullptr;
    const long mval = max(0, min(rows, p.M - m0));
    const uint32_t hb = (uint32_t)(mval * H * 4);
    ldxb = (uint32_t)(p.ldx * (long)sizeof(DT));
    const uint32_t xb = mval ? (uint32_t)(((mval - 1) * p.ldx + H) * (long)sizeof(DT)) : 0u;
    rc = make_rsrc(p.c + (long)m0 * H, hb);
    rxi = make_rsrc(reinterpret_cast<const DT*>(p.x_in) + (long)m0 * p.ldx + p.Z, xb);
    rxo = make_rsrc(reinterpret_cast<DT*>(p.x_out) + (long)m0 * p.ldx + p.Z, xb);
    rw = make_rsrc(p.WaT, (uint32_t)((long)A * 4 * H * (long)sizeof(DT)));
    rb = make_rsrc(p.bg, (uint32_t)(16 * H));
    rht = make_rsrc(p.h_trace ? p.h_trace + (long)m0 * H : nullptr, p.h_trace ? hb : 0u);
    rct = make_rsrc(p.c_trace ? p.c_trace + (long)m0 * H : nullptr, p.c_trace ? hb : 0u);
  }

  // biases of units u0 .. u0+3 (gate order i, f, g, o)
  __device__ __forceinline__ void bias(int u0, bool ok, float4 (&b)[4]) const {
#pragma unroll
    for (int t = 0; t < 4; ++t) b[t] = as_float4(bload16(rb, ok ? (uint32_t)(u0 + t) * 16u : kOffNone));
  }

  // four 16-byte pieces of DT: units u0 .. u0+3 x 4 gates from WaT row a
  __device__ __forceinline__ void gather(uint32_t off, float4 (&w)[4]) const {
    if constexpr (sizeof(DT) == 4) {
#pragma unroll
      for (int t = 0; t < 4; ++t) w[t] = as_float4(bload16(rw, off == kOffNone ? kOffNone : off + 16u * t));
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 v = bload16(rw, off == kOffNone ? kOffNone : off + 16u * h);
        w[2 * h] = make_float4(bf16_bits_to_f32(v.x & 0xffffu), bf16_bits_to_f32(v.x >> 16),
                               bf16_bits_to_f32(v.y & 0xffffu), bf16_bits_to_f32(v.y >> 16));
        w[2 * h + 1] = make_float4(bf16_bits_to_f32(v.z & 0xffffu), bf16_bits_to_f32(v.z >> 16),
                                   bf16_bits_to_f32(v.w & 0xffffu), bf16_bits_to_f32(v.w >> 16));
      }
    }
  }

  __device__ __forceinline__ Gate4In load(int ml, int u0, int a, bool ok, const float4 (&b)[4]) const {
    Gate4In in;
    in.live = nll || a >= 0;
    const bool gok = ok && a >= 0 && a < A;
    float4 w[4];
    gather(gok ? ((uint32_t)a * 4u * H + 4u * u0) * (uint32_t)sizeof(DT) : kOffNone, w);
#pragma unroll
    for (int t = 0; t < 4; ++t)
      in.add[t] = make_float4(b[t].x + w[t].x, b[t].y + w[t].y, b[t].z + w[t].z, b[t].w + w[t].w);
    in.c = as_float4(bload16(rc, ok ? ((uint32_t)ml * H + u0) * 4u : kOffNone));
    const uint32_t ox = ok && !in.live ? (uint32_t)ml * ldxb + (uint32_t)u0 * (uint32_t)sizeof(DT) : kOffNone;
    if constexpr (sizeof(DT) == 4) {
      in.hprev = as_float4(bload16(rxi, ox));
    } else {
      const uint2 v = bload8(rxi, ox);
      in.hprev = make_float4(bf16_bits_to_f32(v.x & 0xffffu), bf16_bits_to_f32(v.x >> 16),
                             bf16_bits_to_f32(v.y & 0xffffu), bf16_bits_to_f32(v.y >> 16));
    }
    return in;
  }

  // g[t]: GEMM part of the gates (i, f, g, o) of unit u0 + t.  FUSED: the bf16
  // cell over one common denominator (lstm_cell_fused), which clamps its inputs
  // (a NaN becomes a number); else separate sigmoids and tanhs, as GateIO has.
  template <bool FUSED>
  __device__ __forceinline__ void commit(int ml, int u0, bool ok, const Gate4In& in, const float4 (&g)[4]) const {
    float cv[4], hv[4];
    const float cin[4] = {in.c.x, in.c.y, in.c.z, in.c.w};
    const float hin[4] = {in.hprev.x, in.hprev.y, in.hprev.z, in.hprev.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      float cn, hn;
      if constexpr (sizeof(DT) == 4 || !FUSED) {
        cn = fsigmoid(g[t].y + in.add[t].y) * cin[t] +
             fsigmoid(g[t].x + in.add[t].x) * ftanh_cell<DT>(g[t].z + in.add[t].z);
        hn = fsigmoid(g[t].w + in.add[t].w) * ftanh_cell<DT>(cn);
      } else {
        lstm_cell_fused(g[t].x + in.add[t].x, g[t].y + in.add[t].y, g[t].z + in.add[t].z, g[t].w + in.add[t].w,
                        cin[t], cn, hn);
      }
      cv[t] = in.live ? cn : cin[t];
      hv[t] = in.live ? hn : hin[t];
    }
    const uint32_t ec = ((uint32_t)ml * H + u0) * 4u;
    const uint32_t ex = (uint32_t)ml * ldxb + (uint32_t)u0 * (uint32_t)sizeof(DT);
    const float4 c4 = make_float4(cv[0], cv[1], cv[2], cv[3]);
    bstore16(rc, ok && in.live ? ec : kOffNone, as_uint4(c4));
    float4 h4;
    if constexpr (sizeof(DT) == 4) {
      h4 = make_float4(hv[0], hv[1], hv[2], hv[3]);
      bstore16(rxo, ok ? ex : kOffNone, as_uint4(h4));
    } else {
      // h is stored rounded (a frozen row's h_t is already a bf16 value)
      const uint2 hb = make_uint2(pack2_bf16(hv[0], hv[1]), pack2_bf16(hv[2], hv[3]));
      bstore8(rxo, ok ? ex : kOffNone, hb);
      h4 = make_float4(bf16_bits_to_f32(hb.x & 0xffffu), bf16_bits_to_f32(hb.x >> 16),
                       bf16_bits_to_f32(hb.y & 0xffffu), bf16_bits_to_f32(hb.y >> 16));
    }
    if (trace) {
      bstore16(rht, ok ? ec : kOffNone, as_uint4(h4));
      bstore16(rct, ok ? ec : kOffNone, as_uint4(c4));
    }
  }
};

// Gate kernel on the register-staged core.  The GEMM tile is staged through
// LDS as E[row][feature] (fp32) and the epilogue then runs with thread t on
// the four-unit group t % GPR of rows t / GPR, t / GPR + RSTEP, ...
template <class C>
__global__ void __launch_bounds__(C::NT) k_gates(const GatesArgs p) {
  using DT = typename C::DT;
  constexpr int NBW = C::NBW, MBW = C::MBW;
  constexpr int GPR = C::BN / 16;          // groups of four units per tile row
  constexpr int RSTEP = C::NT / GPR;       // rows per pass of the block
  constexpr int ELD = C::BN + 4;           // staged row stride (floats)
  constexpr int IPT = (C::BM + RSTEP - 1) / RSTEP;
  constexpr int E_BYTES = C::BM * ELD * 4;
  constexpr int LDS = C::LDS_BYTES > E_BYTES ? C::LDS_BYTES : E_BYTES;
  static_assert(C::NT % GPR == 0, "whole groups per block");
  __shared__ __attribute__((aligned(16))) char lds_raw[LDS];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int n0 = nt * C::BN, m0 = mt * C::BM;
  const int grp = threadIdx.x % GPR, r0 = threadIdx.x / GPR;
  const int u0 = n0 / 4 + 4 * grp;
  // actions of this thread's epilogue rows, fetched ahead of the GEMM
  int act[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int r = r0 + k * RSTEP, m = m0 + r;
    act[k] = (r < C::BM && m < p.M) ? p.act[m] : -1;
  }
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wg), p.ldk, p.ldk, n0, C::BN, 4 * p.H);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x_in), p.ldx, p.ldx, m0, C::BM, p.M);
  f32x4 acc[NBW][MBW];
  C::run(acc, w, x, (int)p.ldk, reinterpret_cast<DT*>(lds_raw));

  float* E = reinterpret_cast<float*>(lds_raw);
  const Gate4IO<DT> io(p, m0, C::BM);
  const bool uok = u0 < p.H;  // H % 16 == 0: the whole group is inside
  float4 b[4];
  io.bias(u0, uok, b);
  // the epilogue's loads go out before the staging barrier, so that their
  // latency passes under the staging
  Gate4In in[IPT];
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int r = r0 + k * RSTEP;
    in[k] = io.load(r, u0, act[k], uok && r < C::BM && m0 + r < p.M, b);
  }
  if (C::kw() == 0) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
    const int wn = C::wn(), wmi = C::wm();
#pragma unroll
    for (int j = 0; j < MBW; ++j)
#pragma unroll
      for (int i = 0; i < NBW; ++i)
        *reinterpret_cast<f32x4*>(E + ((wmi * MBW + j) * 16 + r16) * ELD + (wn * NBW + i) * 16 + 4 * g) = acc[i][j];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < IPT; ++k) {
    const int r = r0 + k * RSTEP;
    if (r >= C::BM) continue;
    float4 gsum[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) gsum[t] = *reinterpret_cast<const float4*>(E + r * ELD + 16 * grp + 4 * t);
    io.template commit<true>(r, u0, uok && m0 + r < p.M, in[k], gsum);
  }
}

// Gate kernel with the epilogue straight from the MFMA accumulators (four
// 16-row blocks per wave, no split K): the weight tile is loaded with the
// gate permutation of GemmD::run, so lane (g, r16) holds, in acc[q][j][v],
// gate q of unit n0/4 + 16 wn + 4 g + v for row (wm MBW + j) 16 + r16 of the
// tile.  Each lane then runs the LSTM cell of four consecutive units of its
// MBW rows, with the next row's loads in flight under the current row's
// cell; no LDS staging, no barrier after the GEMM.  FEW: the sums (runs of
// p.runs slices) and the cell of k_gates_rd.
template <class C, bool FEW>
__global__ void __launch_bounds__(C::NT) k_gates_direct(const GatesArgs p) {
  using DT = typename C::DT;
  constexpr int MBW = C::MBW;
  static_assert(C::NBW == 4 && C::KSPLIT == 1, "four gate blocks per wave");
  __shared__ __attribute__((aligned(16))) char lds_raw[C::LDS_BYTES];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int n0 = nt * C::BN, m0 = mt * C::BM;
  const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  const int wn = C::wn(), wmi = C::wm();
  const int u0 = n0 / 4 + 16 * wn + 4 * g;  // this lane's four units
  // the lane's rows and their actions, fetched ahead of the GEMM
  int act[MBW];
#pragma unroll
  for (int j = 0; j < MBW; ++j) {
    const int m = m0 + (wmi * MBW + j) * 16 + r16;
    act[j] = m < p.M ? p.act[m] : -1;
  }
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wg), p.ldk, p.ldk, n0, C::BN, 4 * p.H);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x_in), p.ldx, p.ldx, m0, C::BM, p.M);
  f32x4 acc[4][MBW];
  C::template run<SrcX<DT>, true, FEW ? KSum::Runs : KSum::Chain>(acc, w, x, (int)p.ldk,
                                                                 reinterpret_cast<DT*>(lds_raw), NoWork{}, p.runs);

  const Gate4IO<DT> io(p, m0, C::BM);
  const bool uok = u0 < p.H;  // H % 16 == 0: the four units are inside together
  float4 b[4];
  io.bias(u0, uok, b);
  auto row_of = [&](int j) { return (wmi * MBW + j) * 16 + r16; };
  auto ok_of = [&](int j) { return uok && m0 + row_of(j) < p.M; };
  Gate4In cur = io.load(row_of(0), u0, act[0], ok_of(0), b);
#pragma unroll
  for (int j = 0; j < MBW; ++j) {
    Gate4In nxt;
    if (j + 1 < MBW) nxt = io.load(row_of(j + 1), u0, act[j + 1], ok_of(j + 1), b);
    float4 gs[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) gs[t] = make_float4(acc[0][j][t], acc[1][j][t], acc[2][j][t], acc[3][j][t]);
    io.template commit<!FEW>(row_of(j), u0, ok_of(j), cur, gs);
    if (j + 1 < MBW) cur = nxt;
  }
}

// Gates on the register-direct core: tiles of BN/4 hidden units x BM rows.
// Each of the first threads owns one (unit, row) of the epilogue and issues
// its loads before the GEMM.
template <class R>
__global__ void __launch_bounds__(R::MAXT) k_gates_rd(const GatesArgs p) {
  using DT = typename R::DT;
  extern __shared__ __attribute__((aligned(16))) float lds_dyn[];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int n0 = nt * R::BN, m0 = mt * R::BM;
  constexpr int UPT = R::BN / 4;  // hidden units per tile
  static_assert(UPT * R::BM <= 256, "one epilogue element per thread of the first four waves");
  const int t = threadIdx.x;
  const int ul = t % UPT, ml = t / UPT;
  const int m = m0 + ml, u = n0 / 4 + ul;
  const bool mine = t < UPT * R::BM;
  const bool ok = mine && m < p.M && u < p.H;
  const GateIO<DT> io(p, m0, R::BM);
  GateIn in{};
  if (mine) in = io.load(ml, u, ok ? p.act[m] : -1, ok);
  const SrcX<DT> w(reinterpret_cast<const DT*>(p.Wg), p.ldk, p.ldk, n0, R::BN, 4 * p.H);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x_in), p.ldx, p.ldx, m0, R::BM, p.M);
  R::run(lds_dyn, w, x, (int)p.ldk);
  if (mine) {
    const float4 g4 = *reinterpret_cast<const float4*>(R::E(lds_dyn) + ml * R::ELD + 4 * ul);
    io.commit(ml, u, ok, in, g4.x, g4.y, g4.z, g4.w);
  }
}

// ===========================================================================
// small element-wise kernels
// ===========================================================================
// X_0 = [q(z0) | q(h0) | 0], zero padding columns of X_1, z_out[0] = z0,
// c = c0, done state, traces of step 0.
template <typename DT>
__global__ void k_rollout_init(int B, int Z, int H, int ldx, const float* __restrict__ z0,
                               const float* __restrict__ h0, const float* __restrict__ c0,
                               const uint8_t* __restrict__ done_io, float* __restrict__ z_out,
                               DT* __restrict__ X0, DT* __restrict__ X1, float* __restrict__ c,
                               int32_t* __restrict__ done_state, float* __restrict__ h_trace,
                               float* __restrict__ c_trace, unsigned* __restrict__ sync,
                               unsigned preset_err) {
  const long stride = (long)gridDim.x * blockDim.x;
  const long i0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long i = i0; i < kSyncWords; i += stride) sync[i] = i == kSyncErr ? preset_err : 0u;
  for (long i = i0; i < (long)B * ldx; i += stride) {
    const long b = i / ldx;
    const int col = (int)(i % ldx);
    float v = 0.f;
    if (col < Z) v = z0[b * Z + col];
    else if (col < Z + H) v = h0 ? h0[b * H + col - Z] : 0.f;
    DType<DT>::store(X0, i, v);
    if (col >= Z + H) DType<DT>::store(X1, i, 0.f);
  }
  for (long i = i0; i < (long)B * Z; i += stride) z_out[i] = z0[i];
  for (long i = i0; i < (long)B * H; i += stride) {
    const float cv = c0 ? c0[i] : 0.f;
    c[i] = cv;
    if (h_trace) {
      h_trace[i] = DType<DT>::round(h0 ? h0[i] : 0.f);
      c_trace[i] = cv;
    }
  }
  for (long i = i0; i < B; i += stride) done_state[i] = done_io ? (done_io[i] != 0) : 0;
}

template <typename DT>
__global__ void k_rollout_finish(int B, int Z, int H, int ldx, const DT* __restrict__ XT,
                                 const float* __restrict__ c, const int32_t* __restrict__ done_state,
                                 float* __restrict__ h_T, float* __restrict__ c_T,
                                 uint8_t* __restrict__ done_io) {
  const long stride = (long)gridDim.x * blockDim.x;
  const long i0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long i = i0; i < (long)B * H; i += stride) {
    if (h_T) h_T[i] = DType<DT>::load(XT, (i / H) * ldx + Z + i % H);
    if (c_T) c_T[i] = c[i];
  }
  if (done_io)
    for (long i = i0; i < B; i += stride) done_io[i] = (uint8_t)done_state[i];
}

// Padding of variable-length rollouts: z_out[t+1, b, :] = 0 for t >= lengths[b].
__global__ void k_rollout_pad(int T, int B, int Z, const int32_t* __restrict__ lengths,
                              float* __restrict__ z_out) {
  const long stride = (long)gridDim.x * blockDim.x;
  const long n = (long)T * B * Z;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const long tb = i / Z;
    const int t = (int)(tb / B), b = (int)(tb % B);
    if (t >= lengths[b]) z_out[(long)B * Z + i] = 0.f;
  }
}

// X_t[:, 0:Z] = q(z_t) for t = 0..T, padding columns zero, h_0 = c_0 = 0.
template <typename DT>
__global__ void k_nll_init(int T, int B, int Z, int H, int ldx, const float* __restrict__ z,
                           DT* __restrict__ X, float* __restrict__ c, unsigned* __restrict__ sync,
                           unsigned preset_err) {
  const long stride = (long)gridDim.x * blockDim.x;
  const long i0 = (long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long i = i0; i < kSyncWords; i += stride) sync[i] = i == kSyncErr ? preset_err : 0u;
  const int ncol = ldx - H;  // z columns, then padding columns
  for (long i = i0; i < (long)(T + 1) * B * ncol; i += stride) {
    const long r = i / ncol;
    const int cc = (int)(i % ncol);
    if (cc < Z) DType<DT>::store(X, r * ldx + cc, z[r * Z + cc]);
    else DType<DT>::store(X, r * ldx + H + cc, 0.f);
  }
  for (long i = i0; i < (long)B * H; i += stride) {
    DType<DT>::store(X, (i / H) * ldx + Z + i % H, 0.f);
    c[i] = 0.f;
  }
}

// Per (t, b): sum the dim-tile partials, reward SE and done BCE from the head
// logits, padding mask; one partial sum per block for the means.
__global__ void __launch_bounds__(256)
    k_nll_reduce(int T, int B, int ntd, const float* __restrict__ part,
                 const float* __restrict__ head, const float* __restrict__ rewards,
                 const uint8_t* __restrict__ dones, const int32_t* __restrict__ lengths,
                 float* __restrict__ loglik, float* __restrict__ reward_se,
                 float* __restrict__ done_bce, float* __restrict__ wgsum) {
  __shared__ float s[4][256];
  const long M = (long)T * B;
  const long m = (long)blockIdx.x * 256 + threadIdx.x;
  float ll = 0.f, se = 0.f, bce = 0.f, cnt = 0.f;
  if (m < M) {
    const int t = (int)(m / B), b = (int)(m % B);
    int len = lengths ? lengths[b] : T;
    len = len < 0 ? 0 : (len > T ? T : len);
    if (t < len) {
      for (int k = 0; k < ntd; ++k) ll += part[m * ntd + k];
      const float rr = head[2 * m], rd = head[2 * m + 1];
      const float dr = rr - rewards[m];
      se = dr * dr;
      bce = fmaxf(rd, 0.f) + log1pf(expf(-fabsf(rd))) - (dones[m] ? rd : 0.f);
      cnt = 1.f;
    }
    loglik[m] = ll;
    reward_se[m] = se;
    done_bce[m] = bce;
  }
  s[0][threadIdx.x] = ll;
  s[1][threadIdx.x] = se;
  s[2][threadIdx.x] = bce;
  s[3][threadIdx.x] = cnt;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 4; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x < 4) wgsum[(long)blockIdx.x * 4 + threadIdx.x] = s[threadIdx.x][0];
}

__global__ void __launch_bounds__(256)
    k_nll_means(int nwg, int Z, const float* __restrict__ wgsum, float* __restrict__ means) {
  __shared__ double s[4][256];
  double acc[4] = {0, 0, 0, 0};
  for (int i = threadIdx.x; i < nwg; i += 256)
    for (int k = 0; k < 4; ++k) acc[k] += wgsum[(long)i * 4 + k];
  for (int k = 0; k < 4; ++k) s[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 4; ++k) s[k][threadIdx.x] += s[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double n = s[3][0];
    means[0] = n > 0 ? (float)(-s[0][0] / (n * Z)) : 0.f;
    means[1] = n > 0 ? (float)(s[1][0] / n) : 0.f;
    means[2] = n > 0 ? (float)(s[2][0] / n) : 0.f;
  }
}

// ===========================================================================
// host-side launch logic
// ===========================================================================
namespace {

// Gate tiles by dtype.
template <typename DT> struct Cfgs;
template <> struct Cfgs<float> {
  using Gates64x32 = Gemm<float, 2, 1, 2, 2, 1, 32, 4>;
  using Gates64x64 = GemmD<float, 4, 1, 1, 4, 4>;
  using Gates128x64 = GemmD<float, 4, 2, 2, 2, 2>;
};
template <> struct Cfgs<bf16_t> {
  using Gates64x32 = GemmD<bf16_t, 4, 1, 1, 2, 4>;
  using Gates64x64 = GemmD<bf16_t, 4, 1, 1, 4, 4>;
  using Gates128x64 = GemmD<bf16_t, 4, 2, 2, 2, 2>;
  using Gates128 = GemmD<bf16_t, 4, 2, 2, 4, 2>;      // 128 x 128 on eight waves
  using Gates256 = GemmD<bf16_t, 4, 8, 4, 2, 2>;      // 256 x 256 on eight waves
  using Gates256w16 = GemmD<bf16_t, 4, 4, 4, 4, 2>;   // ... on sixteen
};

}  // namespace

// Tiles of a gate launch with tile C, and of one with the register-direct
// tile R.
template <class C>
long gate_tiles(const GatesArgs& a) {
  return (long)((4 * a.H + C::BN - 1) / C::BN) * ((a.M + C::BM - 1) / C::BM);
}

// the epilogue from the accumulators where the core has four 16-row blocks
// per wave, else through the staged tile
template <class C, typename DT, bool FEW = false>
hipError_t launch_gates_cfg(const char* name, GatesArgs a, hipStream_t s) {
  a.map = tile_map((4 * a.H + C::BN - 1) / C::BN, (a.M + C::BM - 1) / C::BM,
                   (size_t)4 * a.H * a.ldk * sizeof(DT));
  if constexpr (IsGemmD<C>::value && C::NBW == 4)
    return launch(name, k_gates_direct<C, FEW>, dim3(grid_of(a.map)), dim3(C::NT), 0, s, a);
  else
    return launch(name, k_gates<C>, dim3(grid_of(a.map)), dim3(C::NT), 0, s, a);
}

// Register-direct gate launch with tile R on nw waves (rd_fit).
template <class R, typename DT>
hipError_t launch_gates_rd(GatesArgs a, int nw, hipStream_t s) {
  const size_t lds = R::lds_bytes(nw);
  hipError_t e = allow_lds(k_gates_rd<R>, lds);
  if (e != hipSuccess) return e;
  a.map = tile_map((4 * a.H + R::BN - 1) / R::BN, (a.M + R::BM - 1) / R::BM,
                   (size_t)4 * a.H * a.ldk * sizeof(DT));
  return launch(R::BM == 16 ? "gates/rd16" : "gates/rd32", k_gates_rd<R>, dim3(grid_of(a.map)), dim3(64 * nw), lds, s, a);
}

// Gate tile of a call.  A launch takes about fixed + per * n, n the number of
// tiles that the busiest CU gets: a large tile moves fewer bytes per MFMA
// (smaller `per` for its area), a small one spreads a call with few rows over
// more CUs and rounds its last tile up by less.  The constants are
// microseconds fitted to launches at H 1024, Z 64 (bf16) and H 512, Z 64
// (fp32); both terms scale with K alike, so their comparison holds at other
// sizes too (checked at H 256 and 368).  Measured launches, us:
//   bf16, rows            256    512   1024   2000   3000   4096   6000  16384
//   64 x 64               7.8    9.9   18.0   33.8   49.1   64.0
//   128 x 64             10.1   10.5   13.3   26.0   35.0   43.5   69.2  184.8
//   128 x 128, 8 waves   12.7   12.9   14.5   21.8   31.4   45.4   63.8  164.0
//   256 x 256, 8 waves   31.9   32.1   32.9   37.1   35.9   39.4   68.8  152.2
//   256 x 256, 16 waves                       36.1          40.3   66.1  148.1
// (64 x 32 register-staged tiles and 32 x 32 register-direct ones, which
// these sizes ran on before: 23.4, 15.0, 26.5, 48.1 at 256 to 2000 rows.)
// The register-direct tiles, which hide the whole K loop in one round trip,
// are the fastest while every CU gets at most one (16 rows 5.9, 64 rows 7.2)
// and fall off steeply beyond (128 rows 12.7 against 7.4 for 64 x 32).
// In bf16 the sums and the cell do not follow the tile: calls of at most
// kFewRows rows, where K fits the register-direct tiles, have theirs on every
// tile, larger calls the chain and the fused cell.
constexpr int kFewRows = 256;
template <typename DT>
hipError_t launch_gates(GatesArgs a, hipStream_t s) {
  using RD16 = GemmRD<DT, 2, 1, 4, 640>;
  using RD32 = GemmRD<DT, 2, 2, 4, 640>;
  constexpr bool bf = sizeof(DT) == 2;
  const bool few = a.M <= kFewRows && rd_fit<RD32>((int)a.ldk);
  if (!bf || few) {
    const int n16 = rd_fit<RD16>((int)a.ldk), n32 = rd_fit<RD32>((int)a.ldk);
    if (n16 && gate_tiles<RD16>(a) <= kCUs) return launch_gates_rd<RD16, DT>(a, n16, s);
    if (n32 && gate_tiles<RD32>(a) <= kCUs) return launch_gates_rd<RD32, DT>(a, n32, s);
  }
  using Cf = Cfgs<DT>;
  auto cost = [](long tiles, float fixed, float per) { return fixed + per * (float)((tiles + kCUs - 1) / kCUs); };
  const float c64x32 = cost(gate_tiles<typename Cf::Gates64x32>(a), bf ? 4.9f : 7.0f, bf ? 2.4f : 5.2f);
  const float c64x64 = cost(gate_tiles<typename Cf::Gates64x64>(a), bf ? 3.8f : 4.0f, bf ? 3.9f : 10.3f);
  const float c128x64 = cost(gate_tiles<typename Cf::Gates128x64>(a), bf ? 4.5f : 6.0f, bf ? 5.6f : 18.0f);
  const float small = std::min({c64x32, c64x64, c128x64});
  if constexpr (bf) {
    if (few) {
      a.runs = rd_run<RD32>((int)a.ldk, rd_fit<RD32>((int)a.ldk));
      if (c128x64 <= small) return launch_gates_cfg<typename Cf::Gates128x64, DT, true>("gates/128x64", a, s);
      if (c64x64 <= small) return launch_gates_cfg<typename Cf::Gates64x64, DT, true>("gates/64x64", a, s);
      return launch_gates_cfg<typename Cf::Gates64x32, DT, true>("gates/64x32", a, s);
    }
    const float c128 = cost(gate_tiles<typename Cf::Gates128>(a), 2.5f, 10.2f);
    const long t256 = gate_tiles<typename Cf::Gates256>(a);
    const float c256 = cost(t256, 0.0f, 38.0f);
    if (c256 <= c128 && c256 <= small)  // sixteen waves from the second tile per CU on
      return t256 > kCUs ? launch_gates_cfg<typename Cf::Gates256w16, DT>("gates/256x256/16", a, s)
                         : launch_gates_cfg<typename Cf::Gates256, DT>("gates/256x256/8", a, s);
    if (c128 <= small) return launch_gates_cfg<typename Cf::Gates128, DT>("gates/128x128", a, s);
  }
  if (c128x64 <= small) return launch_gates_cfg<typename Cf::Gates128x64, DT>("gates/128x64", a, s);
  if (c64x64 <= small) return launch_gates_cfg<typename Cf::Gates64x64, DT>("gates/64x64", a, s);
  return launch_gates_cfg<typename Cf::Gates64x32, DT>("gates/64x32", a, s);
}

namespace {

// ---------------------------------------------------------------------------
// WM_FLAG_CHECK: device-side precondition checks.  Each thread counts the
// violations in its grid-stride share and adds a nonzero count to the
// status word sync[kSyncViol]; k_check_zero first clears both status words
// (the workspace's bytes are the caller's until the call's init kernel).
// ---------------------------------------------------------------------------
__global__ void k_check_zero(unsigned* __restrict__ sync) {
  if (threadIdx.x == 0) {
    sync[kSyncErr] = 0u;
    sync[kSyncViol] = 0u;
  }
}

// bytes other than 0 and 1 (the masks)
__global__ void k_check_bytes01(const uint8_t* __restrict__ p, long n, unsigned* __restrict__ sync) {
  const long stride = (long)gridDim.x * blockDim.x;
  unsigned bad = 0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) bad += p[i] > 1u;
  if (bad) atomicAdd(sync + kSyncViol, bad);
}

// steps inside their sequence (t < lengths[b]): an action outside
// [0, A) u {-1, -2}, or a done byte other than 0 and 1
__global__ void k_check_nll(int T, int B, int A, const int32_t* __restrict__ actions,
                            const uint8_t* __restrict__ dones, const int32_t* __restrict__ lengths,
                            unsigned* __restrict__ sync) {
  const long stride = (long)gridDim.x * blockDim.x;
  unsigned bad = 0;
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < (long)T * B; i += stride) {
    const int t = (int)(i / B), b = (int)(i % B);
    if (lengths && t >= lengths[b]) continue;
    const int32_t a = actions[i];
    bad += (a >= A || a < -2) + (dones[i] > 1u);
  }
  if (bad) atomicAdd(sync + kSyncViol, bad);
}

unsigned elem_grid(long n) {
  long g = (n + 255) / 256;
  if (g < 1) g = 1;
  if (g > 4096) g = 4096;
  return (unsigned)g;
}

// After the last step: the final state and done flags, and the padding of
// variable-length rollouts.
template <typename DT>
hipError_t rollout_tail(const Layout& L, const RolloutBufs& R, const DT* XT, hipStream_t s) {
  const long BH = (long)R.B * L.H;
  hipError_t e = launch("finish", k_rollout_finish<DT>, dim3(elem_grid(BH)), dim3(256), 0, s, R.B, L.Z, L.H,
                        L.ldx, XT, R.c, R.done_state, R.h_T, R.c_T, R.done_io);
  if (e != hipSuccess || !R.lengths) return e;
  return launch("finish", k_rollout_pad, dim3(elem_grid((long)R.T * R.B * L.Z)), dim3(256), 0, s, R.T, R.B,
                L.Z, R.lengths, R.z_out);
}

template <typename DT>
hipError_t rollout_impl(const Packed& P, const RolloutBufs& R, hipStream_t s) {
  const Layout& L = P.L;
  const char* base = reinterpret_cast<const char*>(P.base);
  const int B = R.B, T = R.T, Z = L.Z, H = L.H;
  DT* X = reinterpret_cast<DT*>(R.x);
  const long BX = (long)B * L.ldx, BH = (long)B * H, BZ = (long)B * Z;
  const bool trace = (R.flags & WM_FLAG_TRACE) != 0;
  hipError_t e = launch("init", k_rollout_init<DT>, dim3(elem_grid(BX)), dim3(256), 0, s, B, Z, H,
                        L.ldx, R.z0, R.h0, R.c0, R.done_io, R.z_out, X, X + BX, R.c, R.done_state,
                        trace ? R.h_trace : nullptr, trace ? R.c_trace : nullptr, R.sync,
                        R.preset_err);
  if (e != hipSuccess) return e;
  if (T > 0) {
    // one persistent launch for every step when the batch and dims allow it
    e = launch_rollout_persist(P, R, s);
    if (e == hipSuccess) return rollout_tail<DT>(L, R, X + (long)(T & 1) * BX, s);
    if (e != hipErrorNotSupported) return e;
  }

  CtrlArgs ca{};
  ca.Wc = base + L.off_Wc;
  ca.bc = reinterpret_cast<const float*>(base + L.off_bc);
  ca.ldk = L.ldk;
  ca.Z = Z; ca.H = H; ca.A = L.A; ca.Nc = L.Nc; ca.M = B;
  ca.ldx = L.ldx;
  ca.mask = R.mask;
  ca.k0 = R.k0; ca.k1 = R.k1; ca.traj0 = R.traj0;
  ca.done_state = R.done_state;
  ca.use_done = (R.flags & WM_FLAG_DONE) != 0;
  ca.lengths = R.lengths;
  ca.lg_ws = R.lg;
  ca.N = L.N;
  ca.Lc = L.Lc;

  GatesArgs ga{};
  ga.Wg = base + L.off_Wg;
  ga.WaT = base + L.off_WaT;
  ga.bg = reinterpret_cast<const float*>(base + L.off_bg);
  ga.ldk = L.ldk;
  ga.ldx = L.ldx;
  ga.H = H; ga.A = L.A; ga.Z = Z; ga.M = B;
  ga.nll_mode = 0;
  ga.c = R.c;

  MdnArgs ma{};
  ma.Wm = base + L.off_Wm;
  ma.bm = reinterpret_cast<const float*>(base + L.off_bm);
  ma.ldh = L.ldh;
  ma.ldx = L.ldx;
  ma.H = H; ma.Z = Z; ma.K = L.K; ma.Nm = L.Nm; ma.M = B;
  ma.k0 = R.k0; ma.k1 = R.k1; ma.traj0 = R.traj0; ma.tau = R.tau;
  ma.sig = (R.flags & WM_FLAG_SIGMA_TAU) ? sqrtf(R.tau) : 1.0f;
  ma.nll_mode = 0;
  const int mdn_tiles = Z / 8;
  // The controller's h part from the mixture launches (step 0's from h0).  Step
  // t's waits in the z and h columns of the buffer of X_t+1, whose last reader
  // was the gate launch of step t - 1 and whose next writer is that of step t.
  const bool hpart = ctrl_h_wanted(L, B);
  auto lh_of = [&](int t) { return reinterpret_cast<float*>(X + (long)((t + 1) & 1) * BX); };
  if (hpart) {
    ma.zt = Z / 4;
    ma.Wc = ca.Wc;
    ma.ldk = L.ldk;
    ma.Nc = L.Nc;
    ma.ldl = ca.ldlh = L.ldx;
    if (R.h0) {
      ma.x = X;
      ma.lh = lh_of(0);
      if ((e = launch_ctrl_h(ma, L.Q, s)) != hipSuccess) return e;
    }
  }

  for (int t = 0; t <= T; ++t) {
    const uint32_t step = R.step0 + (uint32_t)t;
    DT* Xt = X + (long)(t & 1) * BX;
    DT* Xn = X + (long)((t + 1) & 1) * BX;
    ca.x = Xt;
    ca.step = step;
    ca.t = t;
    ca.mode = t < T ? 1 : 2;
    // step t's [B, A] slice of a per-step mask (the tail step draws no action)
    ca.mask = (R.flags & WM_FLAG_STEP_MASK) ? R.mask + (long)(t < T ? t : T - 1) * B * L.A : R.mask;
    ca.act_t = t < T ? R.actions + (long)t * B : nullptr;
    ca.rew_t = t < T ? R.rewards + (long)t * B : nullptr;
    ca.done_t = t < T ? R.dones + (long)t * B : nullptr;
    ca.act_prev = t > 0 ? R.actions + (long)(t - 1) * B : nullptr;
    ca.rew_prev = t > 0 ? R.rewards + (long)(t - 1) * B : nullptr;
    ca.done_prev = t > 0 ? R.dones + (long)(t - 1) * B : nullptr;
    ca.lh = hpart && (t > 0 || R.h0) ? lh_of(t) : nullptr;
    e = hpart ? launch_ctrl_z(ca, s) : launch_ctrl<SrcX<DT>>(ca, s);
    if (e != hipSuccess) return e;
    if (t == T) break;

    ga.x_in = Xt;
    ga.x_out = Xn;
    ga.act = R.actions + (long)t * B;
    ga.h_trace = trace ? R.h_trace + (long)(t + 1) * BH : nullptr;
    ga.c_trace = trace ? R.c_trace + (long)(t + 1) * BH : nullptr;
    e = launch_gates<DT>(ga, s);
    if (e != hipSuccess) return e;

    ma.x = Xn;
    if (hpart) ma.lh = lh_of(t + 1);
    ma.act = R.actions + (long)t * B;
    ma.z_prev = R.z_out + (long)t * BZ;
    ma.z_next = R.z_out + (long)(t + 1) * BZ;
    ma.step = step;
    e = launch_mdn<DT>(ma, L.Q, mdn_tiles, s);
    if (e != hipSuccess) return e;
  }
  return rollout_tail<DT>(L, R, X + (long)(T & 1) * BX, s);
}

// Which fp32 recurrences run one launch per step on split products
// (wm_recur.hip).  Splitting the operands costs three launches, 6 to 15 us of a
// call (25 at H 2048), so it takes steps to pay for it.
// Against one fp32 gate launch per step, us a step, gates and split, and the T
// from which a whole pass is the shorter (-: never), Z 16 to 64:
//   B            16              150             600            1500             4096
//   H 128    4.8,  4.6  26   5.0,  4.8  47   7.3,  6.6  11   8.1,  8.8  -   13.2, 13.1  -
//   H 256    5.9,  5.1   9   8.5,  5.8   3  11.2,  9.9   6  17.2, 16.1  7   34.5, 32.3  4
//   H 512    6.9,  6.0  13    14,   10   5    25,   20   2    45,   37  1    105,   94  1
//   H 1024    19,    8   2    27,   19   2    61,   45   1   125,  107  1    320,  280  1
//   H 2048    34,   17   2    67,   52   3   194,  168   2   413,  407  6   1073,  998  7
//   H 4096    82,   70  16   209,  345   -   655, 1340   -  1546, 3339  -   4089, 9136  -
// Where a step is short on both sides (small H and few rows) its gain is small.
// At H 4096 the weights' planes (411 MB) no longer fit the 256 MB last-level
// cache; the line is drawn at half of it.
// Of the batches that the persistent kernel serves, those whose rows per XCD
// (above 32) make its fp32 MFMAs the longer part.  Whole likelihood passes, T 32,
// Z 64, K 1, persistent and per step, us:
//   B             128        200        256        384        512
//   H 256     144, 197   197, 210   203, 206   326, 262   337, 254
//   H 512     211, 254   310, 344   319, 309   587, 443   531, 471
bool recur_serves(const Layout& L, int B, int T) {
  if (L.dt != 0) return false;
  if (persist_plan(L, B, true)) return B > 256 && T >= 8;
  if (recur_weight_bytes(L) > ((size_t)128 << 20) || (L.H < 192 && B > 1024)) return false;
  return T >= (L.H >= 768 ? 4 : (long)B * L.H <= 32768 ? 16 : 8);
}

// The planes a call brings in its workspace, and no call that does not need
// them: the size follows from the call's dims, B and T alone (not from the
// device or a switch), and does not shrink as B or T grows, so that the
// workspace of a larger call serves a smaller one.
size_t recur_plane_bytes(const Layout& L, int B, int T) {
  if (L.H < 192) B = std::min(B, 1024);
  return recur_serves(L, B, T) ? recur_fwd_bytes(L, B, T) : 0;
}

// heads = false: the recurrence only (X_1 .. X_T), for the training gradient
template <typename DT>
hipError_t nll_impl(const Packed& P, const NllBufs& N, hipStream_t s, bool heads = true) {
  const Layout& L = P.L;
  const char* base = reinterpret_cast<const char*>(P.base);
  const int B = N.B, T = N.T, Z = L.Z, H = L.H;
  const long BX = (long)B * L.ldx, BZ = (long)B * Z, M = (long)T * B;
  DT* X = reinterpret_cast<DT*>(N.x);
  hipError_t e = launch("nll_init", k_nll_init<DT>, dim3(elem_grid((long)(T + 1) * B * (L.ldx - H))),
                        dim3(256), 0, s, T, B, Z, H, L.ldx, N.z, X, N.c, N.sync, N.preset_err);
  if (e != hipSuccess) return e;

  GatesArgs ga{};
  ga.Wg = base + L.off_Wg;
  ga.WaT = base + L.off_WaT;
  ga.bg = reinterpret_cast<const float*>(base + L.off_bg);
  ga.ldk = L.ldk;
  ga.ldx = L.ldx;
  ga.H = H; ga.A = L.A; ga.Z = Z; ga.M = B;
  ga.nll_mode = 1;
  ga.c = N.c;
  // the recurrence: one persistent launch for small batches, else one launch
  // per step, in fp32 on split products (recur_serves).  The training
  // gradient's (heads = false) keeps to the fp32 products: Adam's first step
  // divides by |g| + 1e-8, and where a gradient is that small another rounding
  // of the sums moves the parameter by up to the whole step.  While the
  // persistent kernels' phases are being timed they serve all they can.
  if (heads && N.planes && recur_serves(L, B, T) && !(phases_timed() && persist_usable(L, B, true)))
    e = launch_recur_fwd(P, N, s);
  else
    e = launch_nll_persist(P, N, s);
  if (e != hipSuccess && e != hipErrorNotSupported) return e;
  for (int t = 0; e == hipErrorNotSupported && t < T; ++t) {
    ga.x_in = X + (long)t * BX;
    ga.x_out = X + (long)(t + 1) * BX;
    ga.act = N.actions + (long)t * B;
    const hipError_t eg = launch_gates<DT>(ga, s);
    if (eg != hipSuccess) return eg;
  }
  if (!heads) return hipSuccess;

  const int ntd = Z / 8;
  MdnArgs ma{};
  ma.Wm = base + L.off_Wm;
  ma.bm = reinterpret_cast<const float*>(base + L.off_bm);
  ma.ldh = L.ldh;
  ma.ldx = L.ldx;
  ma.H = H; ma.Z = Z; ma.K = L.K; ma.Nm = L.Nm; ma.M = (int)M;
  ma.x = X + BX;  // rows of X_1 .. X_T
  ma.z_tgt = N.z + BZ;
  ma.part = N.part;
  ma.head = N.head;
  ma.ntd = ntd;
  ma.nll_mode = 1;
  e = launch_mdn<DT>(ma, L.Q, ntd + 1, s);
  if (e != hipSuccess) return e;

  const int nwg = (int)((M + 255) / 256);
  e = launch("nll_reduce", k_nll_reduce, dim3(nwg), dim3(256), 0, s, T, B, ntd, N.part, N.head,
             N.rewards, N.dones, N.lengths, N.loglik, N.reward_se, N.done_bce, N.wgsum);
  if (e != hipSuccess || !N.means) return e;
  return launch("nll_means", k_nll_means, dim3(1), dim3(256), 0, s, nwg, Z, N.wgsum, N.means);
}

}  // namespace

size_t rollout_workspace(const Layout& L, int B, char* ws, RolloutBufs* R) {
  size_t o = 0;
  const size_t os = o;
  o = wm_align256(o + (size_t)kSyncWords * 4);  // barrier and status words
  const size_t ox = o;
  o = wm_align256(o + (size_t)2 * B * L.ldx * L.esz);  // X_t, X_t+1
  const size_t oc = o;
  o = wm_align256(o + (size_t)B * L.H * 4);  // c
  const size_t od = o;
  o = wm_align256(o + (size_t)B * 4);  // done state
  const size_t pb = persist_partial_bytes(L, B);
  const size_t op = o;
  o = wm_align256(o + pb);  // persistent-kernel controller partials
  // logits of a two-level controller too wide for the staged tiles
  const bool wide2 = L.N > 0 && (L.Nc / 16 + 3) / 4 > 5;
  const size_t og = o;
  if (wide2) o = wm_align256(o + (size_t)B * L.Nc * 4);
  if (ws && R) {
    R->lg = wide2 ? reinterpret_cast<float*>(ws + og) : nullptr;
    R->x = ws + ox;
    R->c = reinterpret_cast<float*>(ws + oc);
    R->done_state = reinterpret_cast<int32_t*>(ws + od);
    R->sync = reinterpret_cast<unsigned*>(ws + os);
    R->P = pb ? reinterpret_cast<float*>(ws + op) : nullptr;
  }
  return o;
}

size_t nll_workspace(const Layout& L, int B, int T, char* ws, NllBufs* N, bool with_planes) {
  const size_t M = (size_t)T * B;
  size_t o = 0;
  const size_t os = o;
  o = wm_align256(o + (size_t)kSyncWords * 4);  // barrier and status words
  const size_t ox = o;
  o = wm_align256(o + (size_t)(T + 1) * B * L.ldx * L.esz);  // X_0 .. X_T
  const size_t oc = o;
  o = wm_align256(o + (size_t)B * L.H * 4);  // c
  const size_t op = o;
  o = wm_align256(o + M * (L.Z / 8) * 4);  // dim-tile partials
  const size_t oh = o;
  o = wm_align256(o + M * 2 * 4);  // reward / done logits
  const size_t og = o;
  o = wm_align256(o + ((M + 255) / 256) * 4 * 4);  // block sums
  const size_t opl = o;
  const size_t pb = with_planes ? recur_plane_bytes(L, B, T) : 0;
  o = wm_align256(o + pb);  // operand planes of the split recurrence
  if (ws && N) {
    N->sync = reinterpret_cast<unsigned*>(ws + os);
    N->x = ws + ox;
    N->c = reinterpret_cast<float*>(ws + oc);
    N->part = reinterpret_cast<float*>(ws + op);
    N->head = reinterpret_cast<float*>(ws + oh);
    N->wgsum = reinterpret_cast<float*>(ws + og);
    N->planes = pb ? ws + opl : nullptr;
  }
  return o;
}

hipError_t launch_check_zero(unsigned* sync, hipStream_t s) {
  return launch("check", k_check_zero, dim3(1), dim3(64), 0, s, sync);
}

hipError_t launch_check_bytes01(const uint8_t* p, long n, unsigned* sync, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  return launch("check", k_check_bytes01, dim3(elem_grid(n)), dim3(256), 0, s, p, n, sync);
}

hipError_t launch_check_nll(int T, int B, int A, const int32_t* actions, const uint8_t* dones,
                            const int32_t* lengths, unsigned* sync, hipStream_t s) {
  if ((long)T * B <= 0) return hipSuccess;
  return launch("check", k_check_nll, dim3(elem_grid((long)T * B)), dim3(256), 0, s, T, B, A, actions,
                dones, lengths, sync);
}

hipError_t launch_pack(const Packed& P, void* packed, const float* W_g, const float* b_g,
                       const float* W_m, const float* b_m, const float* w_r, const float* b_r,
                       const float* w_d, const float* b_d, const float* W_c, const float* b_c,
                       hipStream_t s) {
  char* out = reinterpret_cast<char*>(packed);
  if (P.L.dt == 0)  // two more sections: the transposed copies
    return launch("pack", k_pack<float>, dim3(1024, 9), dim3(256), 0, s, P.L, out, W_g, b_g, W_m, b_m, w_r,
                  b_r, w_d, b_d, W_c, b_c);
  return launch("pack", k_pack<bf16_t>, dim3(1024, 7), dim3(256), 0, s, P.L, out, W_g, b_g, W_m, b_m, w_r, b_r,
                w_d, b_d, W_c, b_c);
}

hipError_t launch_rollout(const Packed& P, const RolloutBufs& R, hipStream_t s) {
  return P.L.dt == 0 ? rollout_impl<float>(P, R, s) : rollout_impl<bf16_t>(P, R, s);
}

hipError_t launch_nll_recurrence(const Packed& P, const NllBufs& N, hipStream_t s) {
  return nll_impl<float>(P, N, s, false);
}

hipError_t launch_nll(const Packed& P, const NllBufs& N, hipStream_t s) {
  return P.L.dt == 0 ? nll_impl<float>(P, N, s) : nll_impl<bf16_t>(P, N, s);
}

}  // namespace wm
