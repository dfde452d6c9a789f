// The mixture head of the per-step path (wm_kernels.hip runs it once per dream
// step, or once over all rows of the likelihood pass).
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

static constexpr float kHalfLn2Pi = 0.91893853320467274178f;

// ===========================================================================
// k_mdn: mixture head on h_{t+1}.  Each wave owns one group of four latent
// dims (Q output blocks), so each lane holds all features of one dim.
// Rollout epilogue: component pick + Box-Muller + z commit.
// NLL epilogue: per-dim log-likelihood, summed over the tile's dims; the
// extra last tile column computes the reward / done logits.
// ===========================================================================
// z_{t+1,j} of row m (mixture_noise / mixture_pick with the call's step,
// temperature and trajectory index).
__device__ __forceinline__ MdnNoise mdn_noise(const MdnArgs& p, const Rng& rng, int m, int j, int K) {
  return mixture_noise(rng, K, p.step, p.traj0 + (uint32_t)m, j);
}

template <int Q>
__device__ __forceinline__ float mdn_pick(const MdnArgs& p, const MdnNoise& n,
                                          const float (&feat)[4 * Q], int K) {
  return mixture_pick<Q>(K, p.tau, n, feat, p.sig);
}

template <int Q>
__device__ __forceinline__ float mdn_draw(const MdnArgs& p, const Rng& rng, int m, int j,
                                          const float (&feat)[4 * Q], int K) {
  return mdn_pick<Q>(p, mdn_noise(p, rng, m, j, K), feat, K);
}

// log sum_k pi_k N(x; mu_k, sigma_k) of one latent dim (pi at tau = 1).
template <int Q>
__device__ __forceinline__ float mdn_loglik(float x, const float (&feat)[4 * Q], int K) {
  float mx = -INFINITY;
#pragma unroll
  for (int f = 0; f < 4 * Q; ++f)
    if (f < K) mx = fmaxf(mx, feat[f]);
  float se = 0.f;
#pragma unroll
  for (int f = 0; f < 4 * Q; ++f)
    if (f < K) se += expf(feat[f] - mx);
  const float lse_pi = mx + logf(se);
  float terms[4 * Q];
  float tmax = -INFINITY;
#pragma unroll
  for (int f = 0; f < 4 * Q; ++f) {
    terms[f] = -INFINITY;
    if (f < K) {
      float mu = 0.f, ls = 0.f;
#pragma unroll
      for (int f2 = 0; f2 < 4 * Q; ++f2) {
        if (f2 == K + f) mu = feat[f2];
        if (f2 == 2 * K + f) ls = feat[f2];
      }
      const float d = (x - mu) * expf(-ls);
      terms[f] = (feat[f] - lse_pi) - 0.5f * d * d - ls - kHalfLn2Pi;
      tmax = fmaxf(tmax, terms[f]);
    }
  }
  float st = 0.f;
#pragma unroll
  for (int f = 0; f < 4 * Q; ++f)
    if (f < K) st += expf(terms[f] - tmax);
  return tmax + logf(st);
}

// z_{t+1,j} of row m goes to the fp32 output and, rounded, to X_{t+1}.
template <typename DT>
__device__ __forceinline__ void mdn_commit(const MdnArgs& p, int m, int j, float z) {
  p.z_next[(long)m * p.Z + j] = z;
  DType<DT>::store(reinterpret_cast<DT*>(p.x), (long)m * p.ldx + j, z);
}

// KC: the number of mixture components (the call's K), a compile-time
// constant so that the feature selections of the epilogue fold away
// ORD: the order of the sum over K (KSum)
// kMdnWaves: two work-groups per CU where their LDS fits twice, also with the
// rarely taken second product of a split tile (GemmD)
template <class C> constexpr int kMdnWaves = 1;
template <int Q> constexpr int kMdnWaves<GemmD<float, Q, 4, 2, 2, 2, true>> = Q <= 5 ? 2 : 1;
template <class C, int KC, KSum ORD>
__global__ void __launch_bounds__(C::NT, kMdnWaves<C>) k_mdn(const MdnArgs p) {
  using DT = typename C::DT;
  constexpr int K = KC;
  constexpr int Q = C::NBW, MBW = C::MBW, WAVES_N = C::WAVES_N, WAVES_M = C::WAVES_M;
  static_assert(WAVES_N == 2, "the NLL epilogue sums two dim groups per work-group");
  __shared__ __attribute__((aligned(16))) char lds_raw[C::LDS_BYTES];
  // NLL partial sums of the second dim group; reuses the GEMM's LDS, which
  // is free once run() has returned
  float(*red)[MBW * 16] = reinterpret_cast<float(*)[MBW * 16]>(lds_raw);
  static_assert(WAVES_M * MBW * 16 * 4 <= C::LDS_BYTES, "partial sums fit the GEMM's LDS");
  int ntile, mt;
  if (!tile_of(p.map, ntile, mt)) return;
  const int n0 = ntile * C::BN, m0 = mt * C::BM;
  const int lane = threadIdx.x & 63;
  const int wn = C::wn(), wmi = C::wm();
  const int g = lane >> 4;
  const int Z = p.Z;
  const int J = ntile * WAVES_N + wn;  // dim group of this wave
  const int j = 4 * J + g;             // latent dim of this lane
  const bool head_tile = p.nll_mode && ntile == p.ntd;
  const bool ctl = sizeof(DT) == 4 && p.lh && 2 * ntile >= p.zt;  // a tile of the controller's h part
  // rollout: the actions of this lane's rows and their previous latents
  // (kept by frozen rows), fetched ahead of the GEMM
  int actp[MBW];
  float zpv[MBW];
  if (!p.nll_mode) {
    const long mval = max(0, min(C::BM, p.M - m0));
    const rsrc_t ra = uniform_rsrc(p.act + m0, (uint32_t)(mval * 4));
    const rsrc_t rz = uniform_rsrc(p.z_prev + (long)m0 * Z, (uint32_t)(mval * Z * 4));
#pragma unroll
    for (int jj = 0; jj < MBW; ++jj) {
      const int ml = (wmi * MBW + jj) * 16 + (lane & 15);
      const bool ok = !ctl && m0 + ml < p.M && j < Z;  // (a call for the h part alone has neither)
      actp[jj] = (int)bload4(ra, ok ? (uint32_t)ml * 4u : kOffNone);
      zpv[jj] = __uint_as_float(bload4(rz, ok ? (uint32_t)(ml * Z + j) * 4u : kOffNone));
    }
  }
  const int nc0 = ctl ? n0 - p.zt / 2 * C::BN : 0;  // its first row of W_c
  const SrcX<DT> w(ctl ? reinterpret_cast<const DT*>(p.Wc) + Z : reinterpret_cast<const DT*>(p.Wm),
                   ctl ? p.ldk : p.ldh, ctl ? p.ldk - Z : p.ldh, ctl ? nc0 : n0, C::BN, ctl ? p.Nc : p.Nm);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x) + p.Z, p.ldx, p.ldx - p.Z, m0, C::BM, p.M);
  const Rng rng{p.k0, p.k1};
  // The four lanes of a row (lane groups g, dims 4J + g) need the same
  // stream-2 block.  With two row blocks per lane, lane group g draws the
  // block and both Box-Muller pairs for row block g % 2 only, and every lane
  // reads its deviates from the drawing lanes (shuffles, all lanes active),
  // instead of each lane drawing both blocks.  On the direct core these
  // draws run while the GEMM's first chunks load: they do not depend on the
  // product.  (Drawing the component noise there too, for every row, frozen
  // or not, made the mixture kernel slower.)
  constexpr bool kPre = IsGemmD<C>::value && MBW == 2;
  float eps[MBW];
  auto draw_eps = [&]() {
    if constexpr (MBW == 2) {
      const float4 e = gauss_group(rng, p.step, p.traj0 + (uint32_t)(m0 + (wmi * MBW + (g & 1)) * 16 + (lane & 15)), J);
#pragma unroll
      for (int jj = 0; jj < MBW; ++jj) {
        const int src = jj * 16 + (lane & 15);
        const float v0 = __shfl(e.x, src), v1 = __shfl(e.y, src), v2 = __shfl(e.z, src), v3 = __shfl(e.w, src);
        eps[jj] = g == 0 ? v0 : (g == 1 ? v1 : (g == 2 ? v2 : v3));
      }
    }
  };
  auto pre = [&]() {
    if (!p.nll_mode && !ctl) draw_eps();
  };
  f32x4 acc[Q][MBW];
  auto none = []() {};
  if constexpr (!IsGemmD<C>::value)
    C::run(acc, w, x, (int)p.ldh, reinterpret_cast<DT*>(lds_raw));
  else if constexpr (kPre)
    C::template run<SrcX<DT>, false, ORD>(acc, w, x, (int)p.ldh, reinterpret_cast<DT*>(lds_raw), pre, p.runs);
  else
    C::template run<SrcX<DT>, false, ORD>(acc, w, x, (int)p.ldh, reinterpret_cast<DT*>(lds_raw), none, p.runs);
  const bool owner = C::kw() == 0;  // holds the summed tile

  if (ctl) {
    if (!owner) return;  // no barrier below
#pragma unroll
    for (int jj = 0; jj < MBW; ++jj) {
      const int m = m0 + (wmi * MBW + jj) * 16 + (lane & 15);
      if (m >= p.M) continue;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int n = nc0 + (wn * Q + q) * 16 + 4 * g;
        if (n < p.Nc) *reinterpret_cast<f32x4*>(p.lh + (long)m * p.ldl + n) = acc[q][jj];
      }
    }
    return;
  }
  if (head_tile) {
    // Rows 0 and 1 of the block are the reward and done logits.
    if (owner && wn == 0 && g == 0) {
#pragma unroll
      for (int jj = 0; jj < MBW; ++jj) {
        const int m = m0 + (wmi * MBW + jj) * 16 + (lane & 15);
        if (m < p.M) {
          p.head[2 * (long)m] = acc[0][jj][0] + p.bm[n0];
          p.head[2 * (long)m + 1] = acc[0][jj][1] + p.bm[n0 + 1];
        }
      }
    }
    return;
  }

  // features f = 4q + v of dim j: acc[q][.][v] + bias
  float bias[4 * Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const float4 b4 = *reinterpret_cast<const float4*>(p.bm + J * 16 * Q + 16 * q + 4 * g);
    bias[4 * q] = b4.x; bias[4 * q + 1] = b4.y; bias[4 * q + 2] = b4.z; bias[4 * q + 3] = b4.w;
  }

  if (!p.nll_mode) {
    if (!owner) return;  // no barrier below
    if constexpr (!kPre) draw_eps();
#pragma unroll
    for (int jj = 0; jj < MBW; ++jj) {
      const int m = m0 + (wmi * MBW + jj) * 16 + (lane & 15);
      if (m >= p.M || j >= Z) continue;
      if (actp[jj] < 0) {
        mdn_commit<DT>(p, m, j, zpv[jj]);
        continue;
      }
      float feat[4 * Q];
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) feat[4 * q + v] = acc[q][jj][v] + bias[4 * q + v];
      if constexpr (MBW == 2) {
        MdnNoise nz;
        component_noise(nz, rng, K, p.step, p.traj0 + (uint32_t)m, j);
        nz.eps = eps[jj];
        mdn_commit<DT>(p, m, j, mdn_pick<Q>(p, nz, feat, K));
      } else {
        mdn_commit<DT>(p, m, j, mdn_draw<Q>(p, rng, m, j, feat, K));
      }
    }
  } else {
#pragma unroll
    for (int jj = 0; jj < MBW; ++jj) {
      const int m = m0 + (wmi * MBW + jj) * 16 + (lane & 15);
      float ll = 0.f;
      if (owner && m < p.M && j < Z) {
        float feat[4 * Q];
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
          for (int v = 0; v < 4; ++v) feat[4 * q + v] = acc[q][jj][v] + bias[4 * q + v];
        ll = mdn_loglik<Q>(p.z_tgt[(long)m * Z + j], feat, K);
      }
      // sum over the four dims of the group (lane groups), then the two waves
      ll += __shfl_xor(ll, 16);
      ll += __shfl_xor(ll, 32);
      if (owner && wn == 1 && g == 0) red[wmi][jj * 16 + (lane & 15)] = ll;
      __syncthreads();
      if (owner && wn == 0 && g == 0 && m < p.M)
        p.part[(long)m * p.ntd + ntile] = ll + red[wmi][jj * 16 + (lane & 15)];
      __syncthreads();
    }
  }
}

// Rollout mixture head on the register-direct core: one group of four
// latent dims (16Q feature rows) x BM rows per tile.  Each of the first
// threads owns one (dim, row) and draws its noise before the GEMM.
template <class R>
__global__ void __launch_bounds__(R::MAXT) k_mdn_rd(const MdnArgs p) {
  using DT = typename R::DT;
  constexpr int Q = R::NBW;
  extern __shared__ __attribute__((aligned(16))) float lds_dyn[];
  int J, mt;
  if (!tile_of(p.map, J, mt)) return;
  const int n0 = J * R::BN, m0 = mt * R::BM;
  const int t = threadIdx.x;
  const int d = t & 3, ml = t >> 2;
  const int m = m0 + ml, j = 4 * J + d;
  const bool ctl = sizeof(DT) == 4 && p.lh && J >= p.zt;  // a tile of the controller's h part
  const int nc0 = (J - p.zt) * R::BN;
  const bool mine = !ctl && t < 4 * R::BM && m < p.M && j < p.Z;
  const Rng rng{p.k0, p.k1};
  bool live = false;
  float zprev = 0.f;
  MdnNoise noise{};
  if (mine) {
    live = p.act[m] >= 0;
    if (live) noise = mdn_noise(p, rng, m, j, p.K);
    else zprev = p.z_prev[(long)m * p.Z + j];
  }
  const SrcX<DT> w(ctl ? reinterpret_cast<const DT*>(p.Wc) + p.Z : reinterpret_cast<const DT*>(p.Wm),
                   ctl ? p.ldk : p.ldh, ctl ? p.ldk - p.Z : p.ldh, ctl ? nc0 : n0, R::BN, ctl ? p.Nc : p.Nm);
  const SrcX<DT> x(reinterpret_cast<const DT*>(p.x) + p.Z, p.ldx, p.ldx - p.Z, m0, R::BM, p.M);
  R::run(lds_dyn, w, x, (int)p.ldh);
  if (ctl) {
    for (int e = t; e < R::BM * R::BN / 4; e += (int)blockDim.x) {
      const int r = e / (R::BN / 4), n = 4 * (e % (R::BN / 4));
      if (m0 + r < p.M && nc0 + n < p.Nc)
        *reinterpret_cast<float4*>(p.lh + (long)(m0 + r) * p.ldl + nc0 + n) =
            *reinterpret_cast<const float4*>(R::E(lds_dyn) + r * R::ELD + n);
    }
    return;
  }
  if (!mine) return;
  if (!live) {
    mdn_commit<DT>(p, m, j, zprev);
    return;
  }
  const float* E = R::E(lds_dyn);
  float feat[4 * Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * q + 4 * d + v;
      feat[4 * q + v] = E[ml * R::ELD + r] + p.bm[n0 + r];
    }
  mdn_commit<DT>(p, m, j, mdn_pick<Q>(p, noise, feat, p.K));
}

namespace {

// Mixture tiles by dtype.
template <typename DT> struct Cfgs;
template <> struct Cfgs<float> {
  template <int Q> using Mdn16 = Gemm<float, Q, 1, 2, 1, 2, 32, 4>;  // 32Q x 16, K split 2
  template <int Q> using Mdn32 = GemmD<float, Q, 1, 2, 2, 2>;
  template <int Q> using Mdn128 = GemmD<float, Q, 4, 2, 2, 2, true>;  // split products
};
template <> struct Cfgs<bf16_t> {
  template <int Q> using Mdn32 = GemmD<bf16_t, Q, 1, 2, 2, 2>;
  template <int Q> using Mdn64 = GemmD<bf16_t, Q, 2, 2, 2, 2>;
  template <int Q> using Mdn128 = GemmD<bf16_t, Q, 2, 2, 4, 2>;  // eight waves
};

// name: of the launch, or null: "mdn" and its tile
template <class C, typename DT, int KC, KSum ORD = KSum::Chain>
hipError_t launch_mdn_cfg(const char* name, MdnArgs a, int ntiles, hipStream_t s) {
  a.map = tile_map(ntiles, (a.M + C::BM - 1) / C::BM, (size_t)a.Nm * a.ldh * sizeof(DT));
  constexpr const char* tile = C::BM == 16 ? "mdn/16" : C::BM == 32 ? "mdn/32" : C::BM == 64 ? "mdn/64" : "mdn/128";
  return launch(name ? name : tile, k_mdn<C, KC, ORD>, dim3(grid_of(a.map)), dim3(C::NT), 0, s, a);
}

// Mixture tile of a call, chosen as the gate tiles are (launch_gates): the
// least fixed + per * n, n the tiles of the busiest CU (with one tile per CU
// nothing overlaps its start and end: a figure of its own).  Measured launches at
// K 8 (Q 6), H 1024 (bf16), us:
//   rows, Z            256,64  1024,64  2000,64  4096,64  6000,128  16384,128
//   192 x 32             10.1     10.3     15.0     25.4      75.0      199.6
//   192 x 64             13.1     13.1     14.0     18.4      50.9      131.0
//   192 x 128, 8 waves                     17.3     18.9      45.4      109.0
//   192 x 256, 8 waves   25.4     25.4     25.9     26.9      54.8      110.4
//   192 x 16, K split 2  12.7     16.1     30.6     56.6
// (the last two were what calls above and up to 2048 rows ran on before).
// The tiles of eight waves need whole DMA instructions per wave: an even Q.
// Register-direct tiles (one dim group x 16 rows) serve rollouts while every
// CU gets at most one (9.9 us at 256 rows, Z 64; 17.5 at 512).
struct MdnCost {
  float c16, c32, c64, c128;  // the tiles of that many rows; INFINITY: none
  float best() const { return std::min(std::min(c16, c32), std::min(c64, c128)); }
};
MdnCost mdn_cost(bool bf16, int Q, int M, int ntiles) {
  auto cost = [&](int bm, float one, float fixed, float per) {
    const long n = ((long)ntiles * ((M + bm - 1) / bm) + kCUs - 1) / kCUs;
    return n == 1 ? one : fixed + per * (float)n;
  };
  if (!bf16)
    return MdnCost{cost(16, 17.0f, 3.0f, 10.6f), cost(32, 18.7f, 3.5f, 14.2f), INFINITY, cost(128, 40.0f, 5.0f, 28.0f)};
  return MdnCost{INFINITY, cost(32, 10.2f, 2.5f, 6.1f), cost(64, 13.8f, 2.2f, 8.1f),
                 Q % 2 == 0 ? cost(128, 18.5f, 2.6f, 13.3f) : INFINITY};
}

// In bf16 the sums over K do not follow the tile but the call (KSum): rollouts
// of at most kRunRows rows, where K fits the register-direct tiles, have the
// runs of those; other calls of at most kPairRows rows the even and odd slices
// apart; larger ones a chain.  (128-row tiles are left to the chain: below
// 2048 rows the 64-row ones are as fast.)
constexpr int kRunRows = 1024, kPairRows = 2048;

template <typename DT, int Q, int KC>
hipError_t launch_mdn_q(const char* name, const MdnArgs& a, int ntiles, hipStream_t s) {
  using R = GemmRD<DT, Q, 1, 4, 640>;
  constexpr bool bf = sizeof(DT) == 2;
  const int nw = a.nll_mode ? 0 : rd_fit<R>((int)a.ldh);
  const bool few = bf && nw && a.M <= kRunRows;
  MdnArgs b = a;
  if (nw && (few || !bf)) {
    const int nt = (a.lh ? a.zt + (a.Nc + R::BN - 1) / R::BN : a.Z / 4);  // one dim group per tile
    const long tiles = (long)nt * ((a.M + R::BM - 1) / R::BM);
    if (tiles <= kCUs) {
      const size_t lds = R::lds_bytes(nw);
      hipError_t e = allow_lds(k_mdn_rd<R>, lds);
      if (e != hipSuccess) return e;
      b.map = tile_map(nt, (a.M + R::BM - 1) / R::BM, (size_t)a.Nm * a.ldh * sizeof(DT));
      return launch(name ? name : "mdn/rd", k_mdn_rd<R>, dim3(grid_of(b.map)), dim3(64 * nw), lds, s, b);
    }
    b.runs = rd_run<R>((int)a.ldh, nw);
  }
  using Cf = Cfgs<DT>;
  if (a.lh) ntiles = a.zt / 2 + (a.Nc + 32 * Q - 1) / (32 * Q);
  const MdnCost c = mdn_cost(bf, Q, a.M, ntiles);
  if constexpr (bf) {
    using T32 = typename Cf::template Mdn32<Q>;
    using T64 = typename Cf::template Mdn64<Q>;
    if (few)
      return c.c64 <= c.c32 ? launch_mdn_cfg<T64, DT, KC, KSum::Runs>(name, b, ntiles, s)
                            : launch_mdn_cfg<T32, DT, KC, KSum::Runs>(name, b, ntiles, s);
    if (a.M <= kPairRows)
      return c.c64 <= c.c32 ? launch_mdn_cfg<T64, DT, KC, KSum::Pairs>(name, b, ntiles, s)
                            : launch_mdn_cfg<T32, DT, KC, KSum::Pairs>(name, b, ntiles, s);
  }
  if constexpr (Q % 2 == 0 || sizeof(DT) == 4) {
    if (c.c128 <= c.best()) return launch_mdn_cfg<typename Cf::template Mdn128<Q>, DT, KC>(name, a, ntiles, s);
  }
  if constexpr (bf) {
    if (c.c64 <= c.c32) return launch_mdn_cfg<typename Cf::template Mdn64<Q>, DT, KC>(name, a, ntiles, s);
  } else {
    if (c.c16 <= c.c32) return launch_mdn_cfg<typename Cf::template Mdn16<Q>, DT, KC>(name, a, ntiles, s);
  }
  return launch_mdn_cfg<typename Cf::template Mdn32<Q>, DT, KC>(name, a, ntiles, s);
}

// one instantiation per component count K (which fixes Q = ceil(3K / 4))
template <typename DT>
hipError_t launch_mdn_k(const char* name, const MdnArgs& a, int Q, int ntiles, hipStream_t s) {
  if (a.K < 1 || a.K > 8 || Q != (3 * a.K + 3) / 4) return hipErrorInvalidValue;
  switch (a.K) {
    case 1: return launch_mdn_q<DT, 1, 1>(name, a, ntiles, s);
    case 2: return launch_mdn_q<DT, 2, 2>(name, a, ntiles, s);
    case 3: return launch_mdn_q<DT, 3, 3>(name, a, ntiles, s);
    case 4: return launch_mdn_q<DT, 3, 4>(name, a, ntiles, s);
    case 5: return launch_mdn_q<DT, 4, 5>(name, a, ntiles, s);
    case 6: return launch_mdn_q<DT, 5, 6>(name, a, ntiles, s);
    case 7: return launch_mdn_q<DT, 6, 7>(name, a, ntiles, s);
    default: return launch_mdn_q<DT, 6, 8>(name, a, ntiles, s);
  }
}

}  // namespace

template <typename DT>
hipError_t launch_mdn(const MdnArgs& a, int Q, int ntiles, hipStream_t s) {
  return launch_mdn_k<DT>(nullptr, a, Q, ntiles, s);
}

// The comparison is of times at H 512, where mdn_cost's fp32 figures were
// taken; all of them grow with H alike.  What the controller saves, in these
// units: about 6 us (10 from H 1024 on) up to 80 logits, 0.08 us a logit beyond.
// Whole rollout steps, whole product and h part beside the mixture, us:
//   rows                   64           300          1000          2000          4000
//   H 128, A 32          16,  15                                 20,  18   (8000) 34,  36
//   H 256, A 32          20,  18       24,  21       28,  25     35,  35       50,  53
//   H 368, A 50          24,  19       29,  24       40,  34     59,  53       82,  76
//   H 512, A 64          28,  23       43,  37       54,  54     82,  85      130, 139
//   H 512, A 300         53,  29       67,  43       78,  61    104,  92
//   H 1024, A 64         77,  57       93,  73      136, 139    225, 223      374, 428
//   H 1024, A 600       259,  73      272,  90      316, 156
//   H 2048, A 64        125,  84      188, 147      355, 340
//   H 2048, A 400       336,  95      396, 158      569, 350
bool ctrl_h_wanted(const Layout& L, int B) {
  if (L.dt == 1 || L.Z + L.ldh > L.ldk || L.Nc > L.Kx) return false;
  if (L.N > 0 && L.Nc / 16 > 20) return false;
  const float with = mdn_cost(L.dt == 1, L.Q, B, L.Z / 8 + (L.Nc + 32 * L.Q - 1) / (32 * L.Q)).best();
  return with <= mdn_cost(L.dt == 1, L.Q, B, L.Z / 8).best() + std::max(L.H >= 1024 ? 10.0f : 6.0f, 0.08f * (float)L.Nc);
}

hipError_t launch_ctrl_h(MdnArgs a, int Q, hipStream_t s) {
  a.zt = 0;
  return launch_mdn_k<float>("lh", a, Q, 0, s);
}

template hipError_t launch_mdn<float>(const MdnArgs&, int, int, hipStream_t);
template hipError_t launch_mdn<bf16_t>(const MdnArgs&, int, int, hipStream_t);

}  // namespace wm
