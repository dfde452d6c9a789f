// The world-model training step's gradient.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "wm_device.h"
#include "wm_gemm.h"
#include "wm_kernels.h"
#include "wm_profile.h"

namespace wm {

static constexpr float kHalfLn2Pi = 0.91893853320467274178f;

// ===========================================================================
// World-model training step: the gradient of the summed NLL means with
// respect to the gate, mixture, reward and done weights (fp32), by
// backpropagation through time after the forward NLL pass.
//
//   forward   X (z_t | h_t) from the NLL pass; where the persistent kernel
//             runs it, the gate activations and c_{t+1} of every step come
//             with it; otherwise the pre-activations of every step in one
//             GEMM and a scan that adds bias and one-hot column, applies the
//             gates and records c_t
//   heads     mixture/reward/done outputs of every h_{t+1} in one GEMM; an
//             element-wise kernel turns them into d loss / d output (dM)
//   back      dh_heads = dM W_m; per step (backwards) the LSTM backward gives
//             dG_t and dc_t, and dh_t = dG_t W_h for the step before (small
//             batches: both in one launch, k_grad_step)
//   weights   dW_g^T = X^T dG and dW_m = dM^T H over all T B rows, with the
//             bias gradients summed in the same pass (k_gemm_tn reads X, dG,
//             dM and H as stored, K outer), the one-hot columns by a
//             deterministic reduction, then the canonical layout
// The forward and per-step products are C[m][n] = sum_k A[m][k] B[n][k] on
// the direct-to-LDS core (both operands K-contiguous: the packing kernel
// also writes W_h^T and W_m^T for them).
// ===========================================================================
namespace {

using GradGemm = GemmD<float, 4, 2, 2, 2, 2>;   // 128 x 64 tiles: the products over all rows
using GradGemmS = GemmD<float, 2, 2, 2, 2, 2>;  // 64 x 64 tiles: the per-step product dG_t . W_h

// out[m][n] = sum_{k < Kpad} A[m][k] B[n][k] for m < M, n < N (Kpad a
// multiple of 32; columns of A and B up to Kpad must be readable, zero
// beyond the data)
// Split K: work-group row y takes columns [y Kpad, (y + 1) Kpad) and writes
// out + y oslice (the caller sums the slices).
template <class C>
__global__ void __launch_bounds__(C::NT) k_gemm_nt(const float* A, long lda, int M, const float* Bm, long ldb,
                                                   int N, int Kpad, float* out, long ldo, long oslice,
                                                   TileMap map) {
  __shared__ __attribute__((aligned(16))) char lds[C::LDS_BYTES];
  int nt, mt;
  if (!tile_of(map, nt, mt)) return;
  A += (long)blockIdx.y * Kpad;
  Bm += (long)blockIdx.y * Kpad;
  out += (long)blockIdx.y * oslice;
  const int n0 = nt * C::BN, m0 = mt * C::BM;
  const SrcX<float> w(Bm, ldb, Kpad, n0, C::BN, N);
  const SrcX<float> x(A, lda, Kpad, m0, C::BM, M);
  f32x4 acc[C::NBW][C::MBW];
  C::run(acc, w, x, Kpad, reinterpret_cast<float*>(lds));
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wn = C::wn(), wmi = C::wm();
#pragma unroll
  for (int j = 0; j < C::MBW; ++j) {
    const int m = m0 + (wmi * C::MBW + j) * 16 + r16;
    if (m >= M) continue;
#pragma unroll
    for (int i = 0; i < C::NBW; ++i) {
      const int n = n0 + (wn * C::NBW + i) * 16 + 4 * g;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (n + v < N) out[(long)m * ldo + n + v] = acc[i][j][v];
    }
  }
}

// N = sum_b min(max(len_b, 0), T) (all B T without lengths)
__global__ void k_len_sum(const int32_t* lengths, int B, int T, float* nout) {
  __shared__ long part[256];
  long s = 0;
  for (int b = threadIdx.x; b < B; b += 256) s += lengths ? min(max(lengths[b], 0), T) : T;
  part[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    long t = 0;
    for (int i = 0; i < 256; ++i) t += part[i];
    nout[0] = (float)t;
  }
}

__device__ __forceinline__ float sig_(float x) { return 1.0f / (1.0f + expf(-x)); }

// forward scan of one (row b, unit u): pre-activations G (packed gate
// order, row r = t B + b, column 4u + q) plus bias and the action's column
// -> activations i, f, tanh g, o in place; c_t into Cs [T+1, B, H]
__global__ void __launch_bounds__(256) k_grad_fwd_scan(float* G, const float* bg, const float* WaT,
                                                       const int32_t* actions, float* Cs, int B, int T, int H,
                                                       int A) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)B * H) return;
  const int b = (int)(idx / H), u = (int)(idx % H);
  const float4 bias = reinterpret_cast<const float4*>(bg)[u];
  float c = 0.f;
  Cs[(long)b * H + u] = 0.f;
  for (int t = 0; t < T; ++t) {
    const long r = (long)t * B + b;
    float4 g = reinterpret_cast<float4*>(G + r * 4 * H)[u];
    const int a = actions[r];
    float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
    if (a >= 0 && a < A) w = reinterpret_cast<const float4*>(WaT + (long)a * 4 * H)[u];
    const float i = sig_(g.x + bias.x + w.x), f = sig_(g.y + bias.y + w.y);
    const float gg = tanhf(g.z + bias.z + w.z), o = sig_(g.w + bias.w + w.w);
    c = f * c + i * gg;
    reinterpret_cast<float4*>(G + r * 4 * H)[u] = make_float4(i, f, gg, o);
    Cs[((long)(t + 1) * B + b) * H + u] = c;
  }
}

// d loss / d head output of one row r = t B + b: for each latent dim j the
// mixture features of packed rows 16 Q J + 16 q + 4 g + v (j = 4J + g,
// feature 4q + v); thread j = Z takes the reward/done block and the padding
// columns.  M holds the head's GEMM outputs and is overwritten with dM.
// lrow [T B, Z+1] receives each (row, dim)'s share of the loss: -loglik_j /
// (N Z), and (se + bce) / N in column Z (0 on padded steps).
template <int KC>
__global__ void __launch_bounds__(256) k_grad_heads(float* M, long ldm, const float* bm, const float* z,
                                                    const float* rewards, const uint8_t* dones,
                                                    const int32_t* lengths, const float* nsum, int B, int T,
                                                    int Z, int Nm, int NmP, float* lrow) {
  constexpr int K = KC, Q = (3 * K + 3) / 4;
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)T * B * (Z + 1)) return;
  const long r = idx / (Z + 1);
  const int j = (int)(idx % (Z + 1));
  const int t = (int)(r / B), b = (int)(r % B);
  const float N = nsum[0];
  const bool valid = t < (lengths ? min(max(lengths[b], 0), T) : T) && N > 0.f;
  float* row = M + r * ldm;
  if (j == Z) {
    const int hr = Nm - 16;
    const float rr = row[hr] + bm[hr], rd = row[hr + 1] + bm[hr + 1];
    const float dr = rr - rewards[r], dd = (float)dones[r];
    // softplus(rd) - d rd, stable for either sign of rd
    const float bce = fmaxf(rd, 0.f) + log1pf(expf(-fabsf(rd))) - dd * rd;
    lrow[r * (Z + 1) + Z] = valid ? (dr * dr + bce) / N : 0.f;
    row[hr] = valid ? 2.0f * dr / N : 0.f;
    row[hr + 1] = valid ? (sig_(rd) - dd) / N : 0.f;
    for (int c = hr + 2; c < Nm; ++c) row[c] = 0.f;
    for (int c = Nm; c < NmP; ++c) row[c] = 0.f;
    return;
  }
  const int J = j >> 2, g = j & 3;
  float f[4 * Q];
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 16 * Q * J + 16 * q + 4 * g + v;
      f[4 * q + v] = row[c] + bm[c];
    }
  const float x = z[(long)(t + 1) * B * Z + (long)b * Z + j];  // target z_{t+1, j}
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < K; ++k) mx = fmaxf(mx, f[k]);
  float se = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) se += expf(f[k] - mx);
  const float lse_pi = mx + logf(se);
  float joint[K], uu[K], sg[K];
  float jm = -INFINITY;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float mu = f[K + k], ls = f[2 * K + k];
    sg[k] = expf(ls);
    uu[k] = (x - mu) / sg[k];
    joint[k] = (f[k] - lse_pi) - 0.5f * uu[k] * uu[k] - ls - kHalfLn2Pi;
    jm = fmaxf(jm, joint[k]);
  }
  float sj = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) sj += expf(joint[k] - jm);
  const float ll = jm + logf(sj);
  const float s = valid ? -1.0f / (N * (float)Z) : 0.f;  // d loss / d loglik_j
  lrow[r * (Z + 1) + j] = s * ll;
  float d[4 * Q];
#pragma unroll
  for (int k = 0; k < 4 * Q; ++k) d[k] = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float gam = expf(joint[k] - ll), pi = expf(f[k] - lse_pi);
    d[k] = s * (gam - pi);
    d[K + k] = s * gam * uu[k] / sg[k];
    d[2 * K + k] = s * gam * (uu[k] * uu[k] - 1.0f);
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
#pragma unroll
    for (int v = 0; v < 4; ++v) row[16 * Q * J + 16 * q + 4 * g + v] = d[4 * q + v];
}

// LSTM backward of step t for (row b, unit u): with dh = d loss / d h_{t+1}
// (heads + the later steps) and dc = d loss / d c_{t+1} from the later steps,
// writes dG_t (pre-activation gradients, packed gate order) and the new dc
// (dhr: S slices [S, B, H] of the later step's dG . W_h, summed in order)
__global__ void __launch_bounds__(256) k_grad_lstm_back(const float* G, const float* Cs, const float* dhh,
                                                        const float* dhr, int S, float* dc, float* dG, int B,
                                                        int H, int t, int last) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)B * H) return;
  const int b = (int)(idx / H), u = (int)(idx % H);
  const long r = (long)t * B + b;
  const float4 a = reinterpret_cast<const float4*>(G + r * 4 * H)[u];  // i, f, g, o
  const float c1 = Cs[((long)(t + 1) * B + b) * H + u], c0 = Cs[((long)t * B + b) * H + u];
  float dh = dhh[r * H + u];
  if (!last) {
    float sum = 0.f;
    for (int k = 0; k < S; ++k) sum += dhr[(long)k * B * H + (long)b * H + u];
    dh += sum;
  }
  const float dcn = last ? 0.f : dc[(long)b * H + u];
  const float th = tanhf(c1);
  const float d_o = dh * th;
  const float dcc = dcn + dh * a.w * (1.0f - th * th);
  const float d_i = dcc * a.z, d_f = dcc * c0, d_g = dcc * a.x;
  dc[(long)b * H + u] = dcc * a.y;
  reinterpret_cast<float4*>(dG + r * 4 * H)[u] =
      make_float4(d_i * a.x * (1.0f - a.x), d_f * a.y * (1.0f - a.y), d_g * (1.0f - a.z * a.z),
                  d_o * a.w * (1.0f - a.w));
}

// The same with the product that feeds it, in one launch per step:
//   dh = dhh_t + sum over eight slices of (dG_{t+1} . W_h over H / 2 columns)
// for 16 units x 16 rows per work-group, a wave per slice.  Operands come from
// the L2 straight into registers, kStepD K slices of 16 ahead of the products;
// the slices meet in LDS and are summed in order, so that the results are to
// the bit those of the product in eight launched slices and k_grad_lstm_back.
// Both are chains of latencies while the tiles fit the CUs: at B 100, H 256
// the launch takes 7.0 us and a step 4.1 us less than with two launches.
constexpr int kStepS = 8, kStepD = 4;
struct StepArgs {
  const float* Wh;      // W_h^T [H, 4H]
  const float* dGn;     // [B, 4H] of step t + 1, or null: t is the last
  const float* G;       // [B, 4H] activations of step t
  const float *c0, *c1; // [B, H] c_t, c_{t+1}
  const float* dhh;     // [B, H]
  float* dc;            // [B, H], in place
  float* dG;            // [B, 4H]
  int B, H;
  TileMap map;
};
__global__ void __launch_bounds__(64 * kStepS) k_grad_step(const StepArgs p) {
  __shared__ __attribute__((aligned(16))) f32x4 red[kStepS][64];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int H = p.H, H4 = 4 * H, n0 = 16 * nt, m0 = 16 * mt;
  // wave 0 takes the epilogue: units u0 .. u0 + 3 of row m per lane, their
  // inputs loaded ahead of the product
  const int u0 = n0 + 4 * g, m = m0 + r16;
  const bool ok = wave == 0 && m < p.B;
  const long e = ok ? (long)m * H + u0 : 0;
  float4 act[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) act[t] = reinterpret_cast<const float4*>(p.G)[e + t];  // i, f, g, o
  const float4 c0 = *reinterpret_cast<const float4*>(p.c0 + e), c1 = *reinterpret_cast<const float4*>(p.c1 + e);
  const float4 dh = *reinterpret_cast<const float4*>(p.dhh + e);
  const float4 dc = p.dGn ? *reinterpret_cast<const float4*>(p.dc + e) : make_float4(0.f, 0.f, 0.f, 0.f);
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  if (p.dGn) {
    const SrcX<float> w(p.Wh, H4, H4, n0, 16, H), x(p.dGn, H4, H4, m0, 16, p.B);
    const int Ks = H4 / kStepS, k0 = wave * Ks + 4 * g, k1 = (wave + 1) * Ks, n = Ks / 16;
    const uint32_t wr = w.row(r16), xr = x.row(r16);
    uint4 a[kStepD], b[kStepD];
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    auto load = [&](int d, int s) {  // zeros past the slice
      a[d] = w.load(wr, k0 + 16 * s, k1);
      b[d] = x.load(xr, k0 + 16 * s, k1);
    };
#pragma unroll
    for (int d = 0; d < kStepD; ++d) load(d, d);
    __builtin_amdgcn_sched_barrier(0);
    for (int s = kStepD; s < n; s += kStepD) {
#pragma unroll
      for (int d = 0; d < kStepD; ++d) {
        Mfma<float>::step(acc, a[d], b[d]);
        load(d, s + d);
        // keeps each stage's products ahead of the next one's loads
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < kStepD; ++d) Mfma<float>::step(acc, a[d], b[d]);
    red[wave][lane] = acc;
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int k = 0; k < kStepS; ++k) sum += red[k][lane];
    }
  }
  if (!ok) return;
  const float c0v[4] = {c0.x, c0.y, c0.z, c0.w}, c1v[4] = {c1.x, c1.y, c1.z, c1.w};
  const float dhv[4] = {dh.x, dh.y, dh.z, dh.w}, dcv[4] = {dc.x, dc.y, dc.z, dc.w};
  float dcn[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float4 q = act[t];
    const float dht = p.dGn ? dhv[t] + sum[t] : dhv[t];
    const float th = tanhf(c1v[t]);
    const float d_o = dht * th;
    const float dcc = dcv[t] + dht * q.w * (1.0f - th * th);
    const float d_i = dcc * q.z, d_f = dcc * c0v[t], d_g = dcc * q.x;
    dcn[t] = dcc * q.y;
    reinterpret_cast<float4*>(p.dG)[e + t] =
        make_float4(d_i * q.x * (1.0f - q.x), d_f * q.y * (1.0f - q.y), d_g * (1.0f - q.z * q.z),
                    d_o * q.w * (1.0f - q.w));
  }
  *reinterpret_cast<float4*>(p.dc + e) = make_float4(dcn[0], dcn[1], dcn[2], dcn[3]);
}

// add(part[k n]) for k = 0 .. S - 1 in order, eight loads in flight (the sums
// over slices are bound by reading them, and have too few threads to hide the
// latency of one load after the other: the four sums of a training step at
// 65536 rows, H 512 took 102 us so, 49 us now)
template <class F>
__device__ __forceinline__ void each_slice(const float* part, long n, int S, F&& add) {
  int k = 0;
  for (; k + 8 <= S; k += 8) {
    float v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = part[(long)(k + q) * n];
#pragma unroll
    for (int q = 0; q < 8; ++q) add(v[q]);
  }
  for (; k < S; ++k) add(part[(long)k * n]);
}

// one-hot columns: dWa[a][j] = sum over rows r with action a of dG[r][j].
// Block (256-column tile, row chunk, group of 64 actions): each thread owns
// one column and accumulates the chunk's rows in row order into an LDS slot
// per action; partial [chunk][a][j], summed over the chunks in order.
// Bound by reading dG once per launch.  The rows of the group are listed
// first, so that kActRows of them are in flight while the ones before are
// added; two blocks per CU (the slots' LDS) leave latency nothing else to hide
// behind.  102 us (5.2 TB/s) at 65536 rows, H 512, A 64; four rows in flight
// behind a test of each row's action took 244.
constexpr int kActGroup = 64, kActRows = 16;
__global__ void __launch_bounds__(256) k_grad_actions(const float* dG, const int32_t* actions, long R, int H4,
                                                      int A, int nchunk, float* part) {
  __shared__ float acc[kActGroup][256];
  __shared__ uint32_t list[256 + 2 * kActRows];  // (row << 8 | action) of the group's rows
  __shared__ int count[4];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int j = blockIdx.x * 256 + tid, ch = blockIdx.y, a0 = blockIdx.z * kActGroup;
  const long r0 = R * ch / nchunk, r1 = R * (ch + 1) / nchunk;
  for (int a = 0; a < kActGroup; ++a) acc[a][tid] = 0.f;
  for (long rb = r0; rb < r1; rb += 256) {
    const long r = rb + tid;
    const int av = r < r1 ? actions[r] : -1;
    const bool in = av >= a0 && av < A && av < a0 + kActGroup;
    const uint64_t bal = __ballot(in);
    __syncthreads();  // the list of the rows before has been read
    if ((tid & 63) == 0) count[wave] = __popcll(bal);
    __syncthreads();
    int at = 0, n = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if (w < wave) at += count[w];
      n += count[w];
    }
    if (in) list[at + __popcll(bal & ((1ull << (tid & 63)) - 1))] = (uint32_t)tid << 8 | (uint32_t)(av - a0);
    // past the end: a row beyond the resource, which reads as zeros
    if (tid < 2 * kActRows) list[n + tid] = 256u << 8;
    __syncthreads();
    // (columns past H4 read other rows' values and are not written out)
    const rsrc_t rg = uniform_rsrc(dG + rb * H4, (uint32_t)(min((long)256, r1 - rb) * H4 * 4));
    uint32_t ea[kActRows], eb[kActRows];
    float va[kActRows], vb[kActRows];
    auto load = [&](int k, uint32_t (&e)[kActRows], float (&v)[kActRows]) {
#pragma unroll
      for (int q = 0; q < kActRows; ++q) e[q] = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[k + q]);
#pragma unroll
      for (int q = 0; q < kActRows; ++q)
        v[q] = __uint_as_float(bload4(rg, 4u * ((e[q] >> 8) * (uint32_t)H4 + (uint32_t)j)));
    };
    auto add = [&](const uint32_t (&e)[kActRows], const float (&v)[kActRows]) {
#pragma unroll
      for (int q = 0; q < kActRows; ++q) acc[e[q] & 0xffu][tid] += v[q];
    };
    // pairs of batches; the one past the end is the padding (k + 2 kActRows
    // stays within the list: k < n)
    load(0, ea, va);
    for (int k = 0; k < n; k += 2 * kActRows) {
      load(k + kActRows, eb, vb);
      add(ea, va);
      if (k + kActRows >= n) break;
      load(k + 2 * kActRows, ea, va);
      add(eb, vb);
    }
  }
  if (j >= H4) return;
  const int na = min(kActGroup, A - a0);
  for (int a = 0; a < na; ++a) part[((long)ch * A + a0 + a) * H4 + j] = acc[a][tid];
}
__global__ void __launch_bounds__(256) k_grad_actions_sum(const float* part, long n, int nchunk, float* out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  each_slice(part + i, n, nchunk, [&](float v) { s += v; });
  out[i] = s;
}

// Fixed-order sum of n floats: block b sums its contiguous piece (each
// thread a strided share, then a tree over the block) into part[b]; one
// block then sums part[0 .. nb) the same way.
constexpr int kFlatBlocks = 512;
__global__ void __launch_bounds__(256) k_flat_sum(const float* x, long n, float* part) {
  __shared__ float red[256];
  const long per = (n + gridDim.x - 1) / gridDim.x;
  const long i0 = (long)blockIdx.x * per, i1 = min(n, i0 + per);
  float acc = 0.f;
  for (long i = i0 + threadIdx.x; i < i1; i += 256) acc += x[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// packed-order gradients -> canonical layout
struct UnpackArgs {
  int Z, H, A, K, Q, Nm, ldk;
  const float *dWgT, *dWa, *dbg, *dWm, *dbm;  // [ldk, 4H], [A, 4H], [4H], [NmP, H], [NmP]
  float *W_g, *b_g, *W_m, *b_m, *w_r, *b_r, *w_d, *b_d;
};
__global__ void __launch_bounds__(256) k_grad_unpack(const UnpackArgs p) {
  const int Z = p.Z, H = p.H, A = p.A, K = p.K, Q = p.Q;
  const long ng = (long)4 * H * (Z + A + H), nm = (long)3 * Z * K * H;
  const long total = ng + 4 * H + nm + 3 * Z * K + 2 * H + 2;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    long e = i;
    if (e < ng) {  // W_g: canonical row q H + u <- packed row 4u + q
      const int cr = (int)(e / (Z + A + H)), c = (int)(e % (Z + A + H));
      const int pr = 4 * (cr % H) + cr / H;
      float v;
      if (c < Z) v = p.dWgT[(long)c * 4 * H + pr];
      else if (c < Z + A) v = p.dWa[(long)(c - Z) * 4 * H + pr];
      else v = p.dWgT[(long)(Z + c - Z - A) * 4 * H + pr];
      p.W_g[e] = v;
      continue;
    }
    e -= ng;
    if (e < 4 * H) {
      p.b_g[e] = p.dbg[4 * (e % H) + e / H];
      continue;
    }
    e -= 4 * H;
    auto prow = [&](long cr) {  // canonical mixture row p ZK + j K + k -> packed row
      const int pp = (int)(cr / ((long)Z * K)), rem = (int)(cr % ((long)Z * K));
      const int j = rem / K, k = rem % K, f = pp * K + k;
      return 16 * Q * (j >> 2) + 16 * (f >> 2) + 4 * (j & 3) + (f & 3);
    };
    if (e < nm) {
      const long cr = e / H;
      p.W_m[e] = p.dWm[(long)prow(cr) * H + e % H];
      continue;
    }
    e -= nm;
    if (e < 3 * Z * K) {
      p.b_m[e] = p.dbm[prow(e)];
      continue;
    }
    e -= 3 * Z * K;
    if (e < H) { p.w_r[e] = p.dWm[(long)(p.Nm - 16) * H + e]; continue; }
    e -= H;
    if (e < H) { p.w_d[e] = p.dWm[(long)(p.Nm - 15) * H + e]; continue; }
    e -= H;
    if (e == 0) p.b_r[0] = p.dbm[p.Nm - 16];
    else p.b_d[0] = p.dbm[p.Nm - 15];
  }
}

// K slices of an M x N x Kpad product: doubled (up to kGradMaxSplit) while
// the tiles number under 512 and the 32-column chunks divide evenly
constexpr int kGradMaxSplit = 8;
template <class C = GradGemm>
int split_of(int M, int N, int Kpad, long target = 512) {
  const long tiles = (long)((N + C::BN - 1) / C::BN) * ((M + C::BM - 1) / C::BM);
  const int chunks = Kpad / 32;
  int S = 1;
  while (S < kGradMaxSplit && tiles * S < target && chunks % (2 * S) == 0 && chunks / (2 * S) >= 4) S *= 2;
  return S;
}

// the per-step product: its tile shape and K slices
using BpttGemm = GradGemmS;
int bptt_split(int B, int H) { return split_of<BpttGemm>(B, H, 4 * H, 256); }

// out (ldo) = A . B^T in S K-slices; S > 1 writes slice y to out + y oslice
template <class C = GradGemm>
hipError_t gemm_nt_slices(const char* name, const float* A, long lda, int M, const float* Bm, long ldb, int N,
                          int Kpad, int S, float* out, long ldo, long oslice, hipStream_t s) {
  const int Ks = Kpad / S;
  const TileMap map = tile_map((N + C::BN - 1) / C::BN, (M + C::BM - 1) / C::BM, (size_t)N * Ks * 4);
  return launch(name, k_gemm_nt<C>, dim3(grid_of(map), (unsigned)S), dim3(C::NT), 0, s, A, lda, M, Bm, ldb, N,
                Ks, out, ldo, oslice, map);
}

// x[0 .. n) = 0
__global__ void __launch_bounds__(256) k_zero(float* x, long n) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) x[i] = 0.f;
}

// ===========================================================================
// k_gemm_tn: out[m][n] = sum over rows k of A[k][m] B[k][n], both operands
// row-major with the reduction over their rows (the weight-gradient products
// over the T B rows read their activation and gradient matrices as stored,
// no transposed copies).  K slice s covers rows [s Ks, (s+1) Ks) and writes
// its own partial [M, N] (summed in fp64 afterwards).  128 x 64 tiles, four
// waves of 64 x 32; chunks of 16 rows reach LDS by LDS-DMA in a ring of four
// stages.  A fragment read takes rows 4g + j, j < 4, of a chunk (one MFMA
// each): the 16-byte pieces of staged row k are XOR-permuted by ((k/4) mod 4)
// * 4, so that the four lane groups g read four distinct 64-byte bank
// windows.  SUMA / SUMB: the work-groups of the first tile column / row also
// sum A's / B's columns over their rows (an extra MFMA block against ones)
// into colsum partials [S, M] / [S, N].  Work-group -> tile: XCD x takes
// the x-th eighth of all tiles, slice by slice, each slice's m fastest, so
// that a slice's rows are shared in one L2, or a few when slices are fewer
// than XCDs (whole slices per XCD before: 4500 rows left five XCDs idle, and
// the two products took 390 us, 320 with this alone).
// ===========================================================================
constexpr int kTnBM = 128, kTnBN = 64, kTnBK = 16, kTnStages = 4;
constexpr int kTnStageBytes = (kTnBM + kTnBN) * kTnBK * 4;  // 12 KB: A rows, then B rows

struct TnArgs {
  const float* A;
  const float* Bm;
  long lda, ldb, K;
  int Ks, S, M, N, ntm, ntn;
  float* part;  // [S, M, N] partials (ldp = N)
  float* csA;   // [S, M] or null
  float* csB;   // [S, N] or null
};

__global__ void __launch_bounds__(256) k_gemm_tn(const TnArgs p) {
  __shared__ __attribute__((aligned(1024))) char lds[kTnStages * kTnStageBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const int per = p.ntm * p.ntn, total = p.S * per, share = (total + 7) / 8;
  const int r = blockIdx.x >> 3, tile = (blockIdx.x & 7) * share + r;
  if (r >= share || tile >= total) return;
  const int sl = tile / per, nt = (tile % per) / p.ntm, mt = (tile % per) % p.ntm;
  const int m0 = mt * kTnBM, n0 = nt * kTnBN;
  const long k0 = (long)sl * p.Ks;
  const long k1 = min(p.K, k0 + (long)p.Ks);
  const int nk = (int)((k1 - k0 + kTnBK - 1) / kTnBK);
  // the slice's rows only: rows past k1 (and the tail of the last row) read zero
  const u32x4 ra = rsrc_words(p.A + k0 * p.lda, (uint32_t)((k1 - k0) * p.lda * 4));
  const u32x4 rb = rsrc_words(p.Bm + k0 * p.ldb, (uint32_t)((k1 - k0) * p.ldb * 4));
  const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)lds);
  // this wave's three DMA instructions per chunk: q < 8 stage A rows 2q, 2q+1
  // (32 pieces each), q >= 8 B rows 4(q-8) .. +3 (16 pieces each)
  bool isa[3];
  uint32_t off[3];
#pragma unroll
  for (int t = 0; t < 3; ++t) {
    const int q = wave * 3 + t;
    isa[t] = q < 8;
    if (isa[t]) {
      const int row = 2 * q + (lane >> 5), pc = (lane & 31) ^ (((row >> 2) & 3) << 2);
      off[t] = (uint32_t)(row * p.lda + m0) * 4u + 16u * (uint32_t)pc;
    } else {
      const int row = 4 * (q - 8) + (lane >> 4), pc = (lane & 15) ^ (((row >> 2) & 3) << 2);
      off[t] = (uint32_t)(row * p.ldb + n0) * 4u + 16u * (uint32_t)pc;
    }
  }
  const uint32_t stepa = (uint32_t)(kTnBK * p.lda) * 4u, stepb = (uint32_t)(kTnBK * p.ldb) * 4u;
  auto issue = [&](int kc) {
    const uint32_t base = lds0 + (uint32_t)(kc % kTnStages) * kTnStageBytes + (uint32_t)wave * 3u * 1024u;
#pragma unroll
    for (int t = 0; t < 3; ++t)
      dma16(isa[t] ? ra : rb, off[t] + (uint32_t)kc * (isa[t] ? stepa : stepb), base + 1024u * t);
  };
#pragma unroll
  for (int c = 0; c < kTnStages - 1; ++c)
    if (c < nk) issue(c);

  const int wm = wave >> 1, wn = wave & 1;
  const bool suma = p.csA && nt == 0 && wn == 0;  // wave-uniform
  const bool sumb = p.csB && mt == 0 && wm == 0;
  f32x4 acc[4][2], cs[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    acc[i][0] = acc[i][1] = cs[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // lane byte offsets inside a stage: A element (4g + j, (wm 4 + i) 16 + r16),
  // B element (4g + j, (wn 2 + jb) 16 + r16)
  uint32_t oa[4], ob[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) oa[i] = (uint32_t)(4 * g * 512 + (((wm * 4 + i) ^ g) & 7) * 64 + r16 * 4);
#pragma unroll
  for (int jb = 0; jb < 2; ++jb) ob[jb] = (uint32_t)(kTnBM * kTnBK * 4 + 4 * g * 256 + (((wn * 2 + jb) ^ g) & 3) * 64 + r16 * 4);
  for (int kc = 0; kc < nk; ++kc) {
    const int young = min(kTnStages - 2, nk - 1 - kc);
    if (young >= 2) vm_wait<6>();
    else if (young == 1) vm_wait<3>();
    else vm_wait<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    if (kc + kTnStages - 1 < nk) issue(kc + kTnStages - 1);
    const char* buf = lds + (kc % kTnStages) * kTnStageBytes;
    // all fragments of the chunk first, the column sums last: with their
    // branches between the rows each row's reads were waited for on their own
    // (65536 rows, H 512: both products 2463 us, 2142 so; 4500 rows, H 256:
    // 320 and 223)
    float fa[4][4], fb[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[j][i] = *reinterpret_cast<const float*>(buf + oa[i] + j * 512);
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) fb[j][jb] = *reinterpret_cast<const float*>(buf + ob[jb] + j * 256);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
          acc[i][jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[j][i], fb[j][jb], acc[i][jb], 0, 0, 0);
    if (suma) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) cs[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[j][i], 1.0f, cs[i], 0, 0, 0);
    }
    if (sumb) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) cs[jb] = __builtin_amdgcn_mfma_f32_16x16x4f32(1.0f, fb[j][jb], cs[jb], 0, 0, 0);
    }
  }
  // lane (g, r16) holds C[4g + v][r16]: rows m, columns n
  float* part = p.part + (long)sl * p.M * p.N;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      const int n = n0 + (wn * 2 + jb) * 16 + r16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + (wm * 4 + i) * 16 + 4 * g + v;
        if (m < p.M && n < p.N) part[(long)m * p.N + n] = acc[i][jb][v];
      }
    }
  if (suma && r16 == 0) {  // every column of C holds A's column sums
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + (wm * 4 + i) * 16 + 4 * g + v;
        if (m < p.M) p.csA[(long)sl * p.M + m] = cs[i][v];
      }
  }
  if (sumb && g == 0) {  // every row of C holds B's column sums
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      const int n = n0 + (wn * 2 + jb) * 16 + r16;
      if (n < p.N) p.csB[(long)sl * p.N + n] = cs[jb][0];
    }
  }
}

// The weight-gradient products reduce over all T B rows.  A K slice
// accumulates its products in fp32, one MFMA after another, so its rounding
// error grows with the slice's length; the slices are therefore kept to at
// most kMaxSliceK rows and summed in fp64 (relative error of the product
// then ~ 1e-5 of the terms' magnitude at T B = 65536).
constexpr int kMaxSliceK = 2048;
int split_long(int M, int N, int Kpad) {
  int S = split_of(M, N, Kpad);
  while (Kpad / S > kMaxSliceK && (Kpad / 32) % (2 * S) == 0) S *= 2;
  return S;
}

// out[m][n] = sum_s part[s][m][n] in slice order, accumulated in fp64
__global__ void __launch_bounds__(256) k_sum_slices(const float* part, int S, int M, int N, float* out, long ldo) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= (long)M * N) return;
  const long mn = (long)M * N;
  double acc = 0.0;
  each_slice(part + i, mn, S, [&](float v) { acc += (double)v; });
  out[(i / N) * ldo + i % N] = (float)acc;
}

// out (ldo) = A . B^T, split over K through `part` ([S, M, N]) when that
// fills the chip better, or (long_k) to bound the fp32 accumulation chains
hipError_t gemm_nt(const float* A, long lda, int M, const float* Bm, long ldb, int N, int Kpad, float* out,
                   long ldo, float* part, hipStream_t s, bool long_k = false) {
  const int S = part ? (long_k ? split_long(M, N, Kpad) : split_of(M, N, Kpad)) : 1;
  if (S == 1) return gemm_nt_slices("grad_gemm", A, lda, M, Bm, ldb, N, Kpad, 1, out, ldo, 0, s);
  const hipError_t e = gemm_nt_slices("grad_gemm", A, lda, M, Bm, ldb, N, Kpad, S, part, N, (long)M * N, s);
  if (e != hipSuccess) return e;
  return launch("grad_sum", k_sum_slices, dim3((unsigned)(((long)M * N + 255) / 256)), dim3(256), 0, s, part, S, M,
                N, out, ldo);
}

// K slices of a product over K rows (kMaxSliceK rows each)
inline int tn_slices(long K) { return (int)((K + kMaxSliceK - 1) / kMaxSliceK); }

// out (ldo) = A^T B over the K rows of both (A [K, lda] with M used columns,
// B [K, ldb] with N), through the slice partials `part` ([S, M, N]) summed in
// fp64; with csA (csB) also the column sums of A (B) into colsum ([M] or [N],
// slice partials in cpart [S, M or N]).
hipError_t gemm_tn(const float* A, long lda, int M, const float* Bm, long ldb, int N, long K, float* part,
                   float* out, long ldo, bool sum_a, bool sum_b, float* cpart, float* colsum, hipStream_t s) {
  if (sum_a && sum_b) return hipErrorInvalidValue;  // one colsum register set per wave
  TnArgs a{};
  a.A = A; a.Bm = Bm; a.lda = lda; a.ldb = ldb; a.K = K;
  a.Ks = kMaxSliceK;
  a.S = tn_slices(K);
  a.M = M; a.N = N;
  a.ntm = (M + kTnBM - 1) / kTnBM;
  a.ntn = (N + kTnBN - 1) / kTnBN;
  a.part = part;
  a.csA = sum_a ? cpart : nullptr;
  a.csB = sum_b ? cpart : nullptr;
  const long nwg = 8 * (((long)a.S * a.ntm * a.ntn + 7) / 8);
  hipError_t e = launch("grad_gemm_tn", k_gemm_tn, dim3((unsigned)nwg), dim3(256), 0, s, a);
  if (e != hipSuccess) return e;
  e = launch("grad_sum", k_sum_slices, dim3((unsigned)(((long)M * N + 255) / 256)), dim3(256), 0, s,
             (const float*)part, a.S, M, N, out, ldo);
  if (e != hipSuccess || !(sum_a || sum_b)) return e;
  const int nc = sum_a ? M : N;
  return launch("grad_sum", k_sum_slices, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, (const float*)cpart,
                a.S, 1, nc, colsum, (long)nc);
}

template <int KC>
hipError_t launch_heads_k(float* M, long ldm, const float* bm, const float* z, const float* rewards,
                          const uint8_t* dones, const int32_t* lengths, const float* nsum, int B, int T, int Z,
                          int Nm, int NmP, float* lrow, hipStream_t s) {
  const long n = (long)T * B * (Z + 1);
  return launch("grad_heads", k_grad_heads<KC>, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, M, ldm,
                bm, z, rewards, dones, lengths, nsum, B, T, Z, Nm, NmP, lrow);
}

}  // namespace

// row chunks of the one-hot column reduction: about 512 work-groups
static int act_chunks(const Layout& L) {
  const int tiles = (4 * L.H + 255) / 256 * ((L.A + kActGroup - 1) / kActGroup);
  return std::min(64, std::max(1, 512 / tiles));
}

size_t grad_workspace(const Layout& L, int B, int T, char* ws, GradWs* G) {
  const long TB = (long)T * B;
  const int H = L.H, H4 = 4 * H, NmP = (L.Nm + 31) / 32 * 32;
  size_t o = 0;
  auto take = [&](size_t bytes) { const size_t at = o; o = wm_align256(o + bytes); return at; };
  const size_t oG = take((size_t)TB * H4 * 4), oC = take((size_t)(T + 1) * B * H * 4);
  const size_t oM = take((size_t)TB * NmP * 4), odG = take((size_t)TB * H4 * 4);
  const size_t odhh = take((size_t)TB * H * 4), odh = take((size_t)B * H * 4), odc = take((size_t)B * H * 4);
  const size_t odWgT = take((size_t)L.ldk * H4 * 4), odWa = take((size_t)L.A * H4 * 4);
  const size_t odWm = take((size_t)NmP * H * 4), odbg = take((size_t)H4 * 4), odbm = take((size_t)NmP * 4);
  const size_t opart = take((size_t)std::max(kFlatBlocks, tn_slices(TB)) * std::max(H4, NmP) * 4);
  const size_t oapart = take((size_t)act_chunks(L) * L.A * H4 * 4);
  // split-K partials: the largest of the products that split, and the
  // per-step slices of dG_t . W_h (always)
  auto split_need = [](int M, int N, int Kpad, bool long_k = false) {
    const int S = long_k ? split_long(M, N, Kpad) : split_of(M, N, Kpad);
    return S > 1 ? (size_t)S * M * N : (size_t)0;
  };
  const size_t nsplit = std::max({(size_t)bptt_split(B, H) * B * H, split_need((int)TB, H4, L.ldk),
                                  split_need((int)TB, L.Nm, L.ldh), split_need((int)TB, H, NmP),
                                  (size_t)tn_slices(TB) * L.ldk * H4, (size_t)tn_slices(TB) * NmP * H});
  const size_t osplit = take(nsplit * 4);
  const size_t on = take(16);
  const size_t ofwd = take((size_t)TB * (L.Z + 1) * 4);  // loss terms [TB, Z+1]
  if (ws && G) {
    auto f = [&](size_t at) { return reinterpret_cast<float*>(ws + at); };
    G->G = f(oG); G->Cs = f(oC); G->M = f(oM); G->dG = f(odG); G->dhh = f(odhh); G->dh = f(odh);
    G->dc = f(odc);
    G->dWgT = f(odWgT); G->dWa = f(odWa); G->dWm = f(odWm); G->dbg = f(odbg); G->dbm = f(odbm);
    G->part = f(opart); G->apart = f(oapart); G->split = f(osplit); G->nsum = f(on); G->fwd = f(ofwd);
  }
  return o;
}

hipError_t launch_nll_grad(const Packed& P, NllBufs N, const GradWs& G, const GradOut& out, hipStream_t s) {
  const Layout& L = P.L;
  const int B = N.B, T = N.T, Z = L.Z, H = L.H, A = L.A, H4 = 4 * H;
  const long TB = (long)T * B;
  const int NmP = (L.Nm + 31) / 32 * 32;
  const char* base = reinterpret_cast<const char*>(P.base);
  const float* Wg = reinterpret_cast<const float*>(base + L.off_Wg);
  const float* WaT = reinterpret_cast<const float*>(base + L.off_WaT);
  const float* bg = reinterpret_cast<const float*>(base + L.off_bg);
  const float* Wm = reinterpret_cast<const float*>(base + L.off_Wm);
  const float* bm = reinterpret_cast<const float*>(base + L.off_bm);
  const float* WhT = reinterpret_cast<const float*>(base + L.off_WhT);  // [H, 4H]
  const float* WmT = reinterpret_cast<const float*>(base + L.off_WmT);  // [H, NmP]
  const float* X = reinterpret_cast<const float*>(N.x);
  const float* Hn = X + (long)B * L.ldx + Z;  // h_1 .. h_T: rows of X_1 .. X_T from column Z
  hipError_t e;
#define WM_TRY(x) do { e = (x); if (e != hipSuccess) return e; } while (0)
  // forward recurrence: X (z_t | h_t) for every step. Where the persistent
  // kernel serves it, it also leaves the gate activations and c_{t+1} of
  // every step; otherwise they are recomputed from X (pre-activations of
  // every step in one GEMM, then a scan that applies the gates and records
  // c_t).
  const bool traced = persist_usable(L, B, true);
  N.g_trace = traced ? G.G : nullptr;
  N.c_trace = traced ? G.Cs : nullptr;
  WM_TRY(launch_nll_recurrence(P, N, s));
  WM_TRY(launch("grad_len", k_len_sum, dim3(1), dim3(256), 0, s, N.lengths, B, T, G.nsum));
  if (traced) {
    WM_TRY(launch("grad_zero", k_zero, dim3((unsigned)(((long)B * H + 255) / 256)), dim3(256), 0, s, G.Cs,
                  (long)B * H));  // c_0
  } else {
    WM_TRY(gemm_nt(X, L.ldx, (int)TB, Wg, L.ldk, H4, L.ldk, G.G, H4, G.split, s));
    WM_TRY(launch("grad_scan", k_grad_fwd_scan, dim3((unsigned)(((long)B * H + 255) / 256)), dim3(256), 0, s,
                  G.G, bg, WaT, N.actions, G.Cs, B, T, H, A));
  }
  // head outputs of every h_{t+1}, then d loss / d output in place
  WM_TRY(gemm_nt(Hn, L.ldx, (int)TB, Wm, L.ldh, L.Nm, L.ldh, G.M, NmP, G.split, s));
  switch (L.K) {
#define WM_HK(k)                                                                                       \
  case k:                                                                                              \
    WM_TRY(launch_heads_k<k>(G.M, NmP, bm, N.z, N.rewards, N.dones, N.lengths, G.nsum, B, T, Z, L.Nm, \
                             NmP, G.fwd, s));                                                          \
    break;
    WM_HK(1) WM_HK(2) WM_HK(3) WM_HK(4) WM_HK(5) WM_HK(6) WM_HK(7) WM_HK(8)
#undef WM_HK
    default: return hipErrorInvalidValue;
  }
  if (out.loss) {  // the loss: a fixed-order sum of its (row, dim) terms
    WM_TRY(launch("grad_loss", k_flat_sum, dim3(kFlatBlocks), dim3(256), 0, s, (const float*)G.fwd,
                  TB * (Z + 1), G.part));
    WM_TRY(launch("grad_loss", k_flat_sum, dim3(1), dim3(256), 0, s, (const float*)G.part, (long)kFlatBlocks,
                  out.loss));
  }
  // d loss / d h_{t+1} through the heads: dM [TB, NmP] . W_m (the packed
  // W_m^T [H, NmP], zero columns past Nm)
  WM_TRY(gemm_nt(G.M, NmP, (int)TB, WmT, NmP, H, NmP, G.dhh, H, G.split, s));
  // back through time (the packed W_h^T [H, 4H])
  const unsigned eg = (unsigned)(((long)B * H + 255) / 256);
  const int Sb = bptt_split(B, H);  // K slices of dG_t . W_h
  const long BH = (long)B * H;
  // One launch per step while its 16 x 16 tiles fit the CUs, else the product
  // on 64 x 64 tiles and the cell apart.  Whole training steps, T 40, two
  // launches and one, us: B 100, 200, 256 at H 256 1139, 1218, 1284 and 977,
  // 1053, 1091; B 40, 100 at H 512 1582, 1647 and 1500, 1516; B 60 at H 1024
  // 3877 and 3802; beyond, B 200 at H 512 (416 tiles) 1883 and 2021.  (Tiles of
  // 32 x 32 were slower throughout: 26.9 us a step at B = H = 512, where the
  // two launches take 22.)
  const bool fused = Sb == kStepS && (long)(H / 16) * ((B + 15) / 16) <= kCUs;
  for (int t = T - 1; t >= 0; --t) {
    if (fused) {
      StepArgs a{};
      a.Wh = WhT;
      a.dGn = t == T - 1 ? nullptr : G.dG + (long)(t + 1) * BH * 4;
      a.G = G.G + (long)t * BH * 4;
      a.c0 = G.Cs + (long)t * BH;
      a.c1 = G.Cs + (long)(t + 1) * BH;
      a.dhh = G.dhh + (long)t * BH;
      a.dc = G.dc;
      a.dG = G.dG + (long)t * BH * 4;
      a.B = B; a.H = H;
      a.map = tile_map(H / 16, (B + 15) / 16, (size_t)H * H4 * 4);
      WM_TRY(launch("grad_step", k_grad_step, dim3(grid_of(a.map)), dim3(64 * kStepS), 0, s, a));
      continue;
    }
    WM_TRY(launch("grad_lstm", k_grad_lstm_back, dim3(eg), dim3(256), 0, s, G.G, G.Cs, G.dhh, G.split, Sb, G.dc,
                  G.dG, B, H, t, t == T - 1 ? 1 : 0));
    if (t > 0)
      WM_TRY(gemm_nt_slices<BpttGemm>("grad_gemm_bptt", G.dG + (long)t * B * H4, H4, B, WhT, H4, H, H4, Sb, G.split, H,
                            (long)B * H, s));
  }
  // dW_g^T [ldk, 4H] = X^T . dG over all rows, read as stored; the bias
  // gradient (dG's column sums) from the same pass
  WM_TRY(gemm_tn(X, L.ldx, L.ldk, G.dG, H4, H4, TB, G.split, G.dWgT, H4, false, true, G.part, G.dbg, s));
  const int nch = act_chunks(L);
  WM_TRY(launch("grad_actions", k_grad_actions,
                dim3((unsigned)((H4 + 255) / 256), (unsigned)nch, (unsigned)((A + kActGroup - 1) / kActGroup)),
                dim3(256), 0, s, G.dG, N.actions, TB, H4, A, nch, G.apart));
  WM_TRY(launch("grad_actions", k_grad_actions_sum, dim3((unsigned)(((long)A * H4 + 255) / 256)), dim3(256), 0,
                s, G.apart, (long)A * H4, nch, G.dWa));
  // dW_m [NmP, H] = dM^T . H over all rows, and the head bias gradient
  // (dM's column sums)
  WM_TRY(gemm_tn(G.M, NmP, NmP, Hn, L.ldx, H, TB, G.split, G.dWm, H, true, false, G.part, G.dbm, s));
  // canonical layout
  const UnpackArgs u{Z, H, A, L.K, L.Q, L.Nm, L.ldk, G.dWgT, G.dWa, G.dbg, G.dWm, G.dbm,
                     out.W_g, out.b_g, out.W_m, out.b_m, out.w_r, out.b_r, out.w_d, out.b_d};
  WM_TRY(launch("grad_unpack", k_grad_unpack, dim3(1024), dim3(256), 0, s, u));
#undef WM_TRY
  return hipSuccess;
}

}  // namespace wm
