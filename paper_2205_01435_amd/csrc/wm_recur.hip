// The LSTM recurrence of the fp32 likelihood pass, one launch per step, on the
// bf16 matrix unit from three-term splits (split3).  A step is a product of its
// activations with weights that stay the same for the whole call, bound by the
// bytes a CU pulls from the L2: every operand is therefore split once, where it
// is written, and stored as "planes": for 16 rows and 32 columns K, the three bf16 terms as
// three 1 KB pieces, each laid out as one MFMA fragment (lane 16 g + r holds
// columns 8 g .. 8 g + 7 of row r in 16 bytes), so that a wave's load of a
// fragment is one contiguous 1 KB and needs neither LDS nor conversion.
//   piece p of row block R, slice s of a matrix of S slices: at
//   ((R S + s) 3 + p) 1024 bytes.
// A work-group of four waves owns one output tile; the waves take interleaved
// K slices, loads running ahead of the products in registers, and their
// partial tiles meet in LDS in a fixed order.  The epilogue applies the LSTM
// cell and writes the next step's planes beside the fp32 results.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "wm_device.h"
#include "wm_gemm.h"
#include "wm_kernels.h"
#include "wm_profile.h"
#include "wm_split.h"

namespace wm {
namespace {

constexpr int kPiece = 1024;       // bytes of one plane piece
constexpr int kFrag = 3 * kPiece;  // ... of the three terms

inline int slices(int cols) { return (cols + 31) / 32; }
inline int blocks(int rows) { return (rows + 15) / 16; }

struct Terms {  // eight values as three 16-byte plane entries
  uint4 p[3];
};
__device__ __forceinline__ Terms terms8(const float (&x)[8]) {
  const Split3 s = split3(x);
  return Terms{{__builtin_bit_cast(uint4, s.h), __builtin_bit_cast(uint4, s.m), __builtin_bit_cast(uint4, s.l)}};
}
__device__ __forceinline__ void store_terms(char* at, const Terms& t) {
#pragma unroll
  for (int p = 0; p < 3; ++p) *reinterpret_cast<uint4*>(at + p * kPiece) = t.p[p];
}

// ---------------------------------------------------------------------------
// planes of the call's constants
// ---------------------------------------------------------------------------
// The gate weights, rows permuted so that row block 4 w + i holds gate i of
// units 16 w .. 16 w + 15 (packed row 4 u + i), columns z (nz slices, zero
// past Z) then h (nh slices, zero past H).
__global__ void __launch_bounds__(256) k_planes_gates(const float* Wg, long ldk, int Z, int H, int nz, int nh,
                                                      char* out) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  const int nks = nz + nh;
  if (idx >= (long)(H / 4) * nks * 64) return;
  const int lane = (int)(idx & 63), s = (int)((idx >> 6) % nks), R = (int)((idx >> 6) / nks);
  const int unit = 16 * (R >> 2) + (lane & 15);
  const float* row = Wg + (long)(4 * unit + (R & 3)) * ldk;
  const bool hs = s >= nz;
  const int c0 = 32 * (hs ? s - nz : s) + 8 * (lane >> 4), lim = hs ? H : Z;
  float x[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) x[v] = c0 + v < lim ? row[(hs ? Z : 0) + c0 + v] : 0.f;
  store_terms(out + ((long)R * nks + s) * kFrag + lane * 16, terms8(x));
}

// A row-major matrix of R16 row blocks (rows past `rows` zero) and S slices
// (columns past `cols` zero).
__global__ void __launch_bounds__(256) k_planes_rows(const float* A, long lda, int rows, int cols, int R16, int S,
                                                     long rstride, long pstride, char* out) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  if (idx >= (long)R16 * S * 64) return;
  A += (long)blockIdx.y * rstride;
  out += (long)blockIdx.y * pstride;
  const int lane = (int)(idx & 63), s = (int)((idx >> 6) % S), R = (int)((idx >> 6) / S);
  const int r = 16 * R + (lane & 15), c0 = 32 * s + 8 * (lane >> 4);
  float x[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) x[v] = r < rows && c0 + v < cols ? A[(long)r * lda + c0 + v] : 0.f;
  store_terms(out + ((long)R * S + s) * kFrag + lane * 16, terms8(x));
}

__global__ void __launch_bounds__(256) k_planes_zero(uint4* p, long n) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// ---------------------------------------------------------------------------
// the product: acc[i][j] += sum over this wave's slices of A block i . B block j
// ---------------------------------------------------------------------------
// One operand's planes of a tile: row blocks R0 .. (those at or past `rb`
// read as zero) of a matrix of S slices.
struct PlaneSrc {
  rsrc_t r;
  uint32_t stride;  // bytes between row blocks
  int left;         // row blocks inside the matrix
  __device__ PlaneSrc(const char* base, int S, int R0, int rb) {
    stride = (uint32_t)S * kFrag;
    left = max(0, rb - R0);
    r = uniform_rsrc(base + (long)R0 * stride, (uint32_t)min(left, 8) * stride);
  }
  // term p of row block i, slice s (uniform), 16 bytes at lane offset lo
  // (kOffNone: zeros)
  __device__ __forceinline__ bf16x8 load(int i, int s, int p, uint32_t lo) const {
    return __builtin_bit_cast(bf16x8, bload16(r, (uint32_t)i * stride + (uint32_t)(s * kFrag + p * kPiece) + lo));
  }
};

template <int NB, int MB>
struct Stage {
  Split3 a[NB], b[MB];
  __device__ __forceinline__ void load(const PlaneSrc& A, int sa, const PlaneSrc& B, int sb, uint32_t lo) {
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      a[i].h = A.load(i, sa, 0, lo);
      a[i].m = A.load(i, sa, 1, lo);
      a[i].l = A.load(i, sa, 2, lo);
    }
#pragma unroll
    for (int j = 0; j < MB; ++j) {
      b[j].h = B.load(j, sb, 0, lo);
      b[j].m = B.load(j, sb, 1, lo);
      b[j].l = B.load(j, sb, 2, lo);
    }
  }
  __device__ __forceinline__ void mul(f32x4 (&acc)[MB][NB]) const {
#pragma unroll
    for (int j = 0; j < MB; ++j) mfma_split(acc[j], a, b[j]);
  }
};

// Slices wave, wave + 4, ... of S, D stages in flight: start() issues the
// first D, run() multiplies and keeps the loads ahead.  load(stage, s) fills a
// stage with slice s (zeros past the last one, without a branch: the compiler
// would wait for every load in flight at it).  A load that only reads zeros
// still takes its 16 cycles of address work, so the last D stages load nothing.
template <int NB, int MB, int D>
struct PlaneProduct {
  Stage<NB, MB> st[D];
  template <class F>
  __device__ __forceinline__ void start(int wave, F load) {
#pragma unroll
    for (int d = 0; d < D; ++d) load(st[d], wave + 4 * d);
    __builtin_amdgcn_sched_barrier(0);
  }
  template <class F>
  __device__ __forceinline__ void run(f32x4 (&acc)[MB][NB], int S, int wave, F load) {
    for (int s = wave + 4 * D; s < S; s += 4 * D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        st[d].mul(acc);
        load(st[d], s + 4 * d);
        // the products of a stage may not drift below the loads of the next:
        // they would then wait for all stages at once
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < D; ++d) st[d].mul(acc);
  }
};

// ---------------------------------------------------------------------------
// forward step: 16 units (64 gate rows) x 16 MB rows per work-group
// ---------------------------------------------------------------------------
struct FwdArgs {
  const char *Wp, *zp, *hp;  // planes: gate weights, z_t, h_t
  char* hp_out;              // h_{t+1}
  const float *bg, *WaT;
  const int32_t* act;        // [B]
  float* c;                  // [B, H], in place
  float* x_out;              // X_{t+1}: fp32 h at columns Z .. of rows of ldx
  const float *Wg, *x_in;    // row-major: packed gate rows of ldk, X_t = [z_t | h_t] of ldx
  long ldk;
  int B, H, A, Z, nz, nh;
  long ldx;
  TileMap map;
};

// The sums of one 16 x 16 tile (units 16 nt .. x rows 16 R ..) over all of K
// from the row-major operands on the fp32 unit, by one wave, where the split
// sums came out as NaN: infinities and values that round to one in bf16 do not
// survive the split (split3).  Rare, so one fragment at a time.
__device__ __forceinline__ void fwd_fp32(const FwdArgs& p, f32x4 (&s)[4], int nt, int R) {
  const int lane = threadIdx.x & 63, g = lane >> 4, r16 = lane & 15;
  const int m = 16 * R + r16, kx = p.Z + p.H;  // a multiple of 4: a piece of four columns is whole
  const float* x = p.x_in + (long)min(m, p.B - 1) * p.ldx;
  f32x4 c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < kx; k0 += Mfma<float>::KSLICE) {
    const int k = k0 + 4 * g;
    const bool in = k < kx;
    uint4 b = *reinterpret_cast<const uint4*>(x + (in ? k : 0));
    if (!in || m >= p.B) b = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      uint4 a = *reinterpret_cast<const uint4*>(p.Wg + (long)(4 * (16 * nt + r16) + i) * p.ldk + (in ? k : 0));
      if (!in) a = make_uint4(0u, 0u, 0u, 0u);
      Mfma<float>::step(c[i], a, b);
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = nan_to(s[i], c[i]);
}

template <int MB>
__global__ void __launch_bounds__(256, 1) k_recur_fwd(const FwdArgs p) {
  __shared__ __attribute__((aligned(16))) f32x4 red[4][MB][4][64];
  int nt, mt;
  if (!tile_of(p.map, nt, mt)) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, r16 = lane & 15;
  const uint32_t lo = (uint32_t)lane * 16u;
  const int nks = p.nz + p.nh, rbs = (p.B + 15) >> 4;
  const int H = p.H, m = 16 * (mt * MB + wave) + r16, u0 = 16 * nt + 4 * g;
  const bool ok = wave < MB && m < p.B;
  // the epilogue's inputs, ahead of the product
  const rsrc_t rb = uniform_rsrc(p.bg, (uint32_t)(16 * H));
  const rsrc_t rw = uniform_rsrc(p.WaT, (uint32_t)((long)p.A * 16 * H));
  const int a = ok ? p.act[m] : -1;
  float4 bias[4], wa[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) bias[t] = as_float4(bload16(rb, ok ? (uint32_t)(u0 + t) * 16u : kOffNone));
  const float4 c4 = ok ? *reinterpret_cast<const float4*>(p.c + (long)m * H + u0) : make_float4(0.f, 0.f, 0.f, 0.f);

  f32x4 acc[MB][4];
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    // the z slices, then the h slices
    const PlaneSrc W(p.Wp, nks, 4 * nt, H / 4);
    const PlaneSrc xz(p.zp, p.nz, mt * MB, rbs), xh(p.hp, p.nh, mt * MB, rbs);
    auto load = [&](Stage<4, MB>& st, int sl) {
      const bool z = sl < p.nz;
      PlaneSrc x = xh;
      if (z) x = xz;
      st.load(W, sl, x, z ? sl : sl - p.nz, sl < nks ? lo : kOffNone);
    };
    PlaneProduct<4, MB, 2> pp;
    pp.start(wave, load);
    // the one-hot columns, once the actions are in
#pragma unroll
    for (int t = 0; t < 4; ++t)
      wa[t] = as_float4(bload16(rw, a >= 0 && a < p.A ? ((uint32_t)a * 4u * H + 4u * (u0 + t)) * 4u : kOffNone));
    pp.run(acc, nks, wave, load);
  }
#pragma unroll
  for (int j = 0; j < MB; ++j)
#pragma unroll
    for (int i = 0; i < 4; ++i) red[wave][j][i][lane] = acc[j][i];
  __syncthreads();
  if (wave >= MB) return;
  // gate i of unit u0 + t of row m is element t of block i
  f32x4 s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    s[i] = (red[0][wave][i][lane] + red[1][wave][i][lane]) + (red[2][wave][i][lane] + red[3][wave][i][lane]);
  const float cin[4] = {c4.x, c4.y, c4.z, c4.w};
  float cv[4], hv[4];
  auto cell = [&]() {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const float gi = fsigmoid(s[0][t] + (bias[t].x + wa[t].x)), gf = fsigmoid(s[1][t] + (bias[t].y + wa[t].y));
      const float gg = ftanh(s[2][t] + (bias[t].z + wa[t].z)), go = fsigmoid(s[3][t] + (bias[t].w + wa[t].w));
      cv[t] = gf * cin[t] + gi * gg;
      hv[t] = go * ftanh(cv[t]);
    }
  };
  cell();
  // a NaN in a sum reaches h, and only a NaN does
  if (__ballot(any_nan(f32x4{hv[0], hv[1], hv[2], hv[3]}))) {
    fwd_fp32(p, s, nt, mt * MB + wave);
    cell();
  }
  if (!ok) return;
  *reinterpret_cast<float4*>(p.c + (long)m * H + u0) = make_float4(cv[0], cv[1], cv[2], cv[3]);
  *reinterpret_cast<float4*>(p.x_out + (long)m * p.ldx + p.Z + u0) = make_float4(hv[0], hv[1], hv[2], hv[3]);
  const float x8[8] = {hv[0], hv[1], hv[2], hv[3], 0.f, 0.f, 0.f, 0.f};
  const Terms t8 = terms8(x8);
  char* at = p.hp_out + ((long)(m >> 4) * p.nh + (u0 >> 5)) * kFrag + (((u0 & 31) >> 3) * 16 + r16) * 16 + (u0 & 7) * 2;
#pragma unroll
  for (int q = 0; q < 3; ++q) *reinterpret_cast<uint2*>(at + q * kPiece) = make_uint2(t8.p[q].x, t8.p[q].y);
}

template <int MB>
hipError_t launch_fwd(FwdArgs a, hipStream_t s) {
  // Weights too large for the L2s even in eighths are still split eight ways:
  // an XCD that walked all of them would read them once per row tile (B 1000,
  // H 1024: 135 us a step so, 74 with an eighth each; fp32 gate launches 86)
  const size_t wbytes = (size_t)(a.H / 4) * (a.nz + a.nh) * kFrag;
  a.map = tile_map(a.H / 16, (a.B + 16 * MB - 1) / (16 * MB), std::min(wbytes, 8 * kL2Budget));
  return launch("nll_step", k_recur_fwd<MB>, dim3(grid_of(a.map)), dim3(256), 0, s, a);
}

}  // namespace

// The z planes of this many steps at a time: few enough that a long pass does
// not hold planes by its length (6 bytes per value, rows in sixteens), enough
// that their launch is lost in the steps.
constexpr int kPlaneSteps = 256;

size_t recur_weight_bytes(const Layout& L) { return (size_t)(L.H / 4) * (slices(L.Z) + slices(L.H)) * kFrag; }

size_t recur_fwd_bytes(const Layout& L, int B, int T) {
  const int nz = slices(L.Z), nh = slices(L.H);
  return wm_align256(recur_weight_bytes(L)) + wm_align256((size_t)std::min(T, kPlaneSteps) * blocks(B) * nz * kFrag) +
         wm_align256((size_t)2 * blocks(B) * nh * kFrag);
}

hipError_t launch_recur_fwd(const Packed& P, const NllBufs& N, hipStream_t s) {
  const Layout& L = P.L;
  const char* base = reinterpret_cast<const char*>(P.base);
  const int B = N.B, T = N.T, Z = L.Z, H = L.H, nz = slices(Z), nh = slices(H), rbs = blocks(B);
  char* Wp = reinterpret_cast<char*>(N.planes);
  char* zp = Wp + wm_align256((size_t)(H / 4) * (nz + nh) * kFrag);
  char* hp = zp + wm_align256((size_t)std::min(T, kPlaneSteps) * rbs * nz * kFrag);
  const long hb = (long)rbs * nh * kFrag, zb = (long)rbs * nz * kFrag;
  auto grid = [](long n) { return (unsigned)((n + 255) / 256); };
  hipError_t e = launch("nll_planes", k_planes_gates, dim3(grid((long)(H / 4) * (nz + nh) * 64)), dim3(256), 0, s,
                        reinterpret_cast<const float*>(base + L.off_Wg), (long)L.ldk, Z, H, nz, nh, Wp);
  if (e != hipSuccess) return e;
  e = launch("nll_planes", k_planes_zero, dim3(grid(2 * hb / 16)), dim3(256), 0, s, reinterpret_cast<uint4*>(hp),
             2 * hb / 16);
  if (e != hipSuccess) return e;
  FwdArgs a{};
  a.Wp = Wp;
  a.bg = reinterpret_cast<const float*>(base + L.off_bg);
  a.WaT = reinterpret_cast<const float*>(base + L.off_WaT);
  a.c = N.c;
  a.B = B; a.H = H; a.A = L.A; a.Z = Z; a.nz = nz; a.nh = nh;
  a.ldx = L.ldx;
  a.Wg = reinterpret_cast<const float*>(base + L.off_Wg);
  a.ldk = L.ldk;
  const long BX = (long)B * L.ldx;
  for (int t = 0; t < T; ++t) {
    if (t % kPlaneSteps == 0) {
      e = launch("nll_planes", k_planes_rows, dim3(grid((long)rbs * nz * 64), (unsigned)std::min(T - t, kPlaneSteps)),
                 dim3(256), 0, s, N.z + (long)t * B * Z, (long)Z, B, Z, rbs, nz, (long)B * Z, zb, zp);
      if (e != hipSuccess) return e;
    }
    a.zp = zp + t % kPlaneSteps * zb;
    a.hp = hp + (t & 1) * hb;
    a.hp_out = hp + ((t + 1) & 1) * hb;
    a.act = N.actions + (long)t * B;
    a.x_in = reinterpret_cast<const float*>(N.x) + (long)t * BX;
    a.x_out = reinterpret_cast<float*>(N.x) + (long)(t + 1) * BX;
    // 32-row tiles once they number the CUs, 16-row ones below (launches at
    // B 512, H 512: 16, 32 and 64 rows 14.9, 11.8 and 12.1 us; B 100, H 256:
    // 5.1, 5.9 and 8.1; of these 2.4 are the launch itself)
    e = (long)(H / 16) * ((B + 31) / 32) >= kCUs ? launch_fwd<2>(a, s) : launch_fwd<1>(a, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace wm
