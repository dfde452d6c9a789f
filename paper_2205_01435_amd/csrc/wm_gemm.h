// GEMM cores of libwm and the host helpers that place their tiles: a
// register-staged pipeline (Gemm), a direct-to-LDS pipeline for larger row
// counts (GemmD) and a register-direct split-K core for few rows (GemmRD).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "wm_device.h"
#include "wm_split.h"

namespace wm {

// ===========================================================================
// GEMM core: a WG tile of BN weight rows x BM activation rows, both operands
// staged through two LDS buffers, with global loads issued STAGES chunks
// ahead into a ring of register stages so their latency overlaps the MFMAs.
// Waves are laid out WAVES_M x WAVES_N x KSPLIT; the KSPLIT waves of one
// (wm, wn) position take interleaved MFMA K slices of every chunk and are
// summed through LDS at the end, so that only waves with kw == 0 hold the
// result.
//   acc[i][j] = W[n0 + (wn*NBW + i)*16 .. +16, :] . X[m0 + (wm*MBW + j)*16 .. +16, :]^T
// over K = Kpad columns; both sources address the tile's rows only.
// ===========================================================================
template <typename DT_, int NBW_, int MBW_, int WAVES_N_, int WAVES_M_, int KSPLIT_, int BK_,
          int STAGES_>
struct Gemm {
  using DT = DT_;
  static constexpr int NBW = NBW_, MBW = MBW_, WAVES_N = WAVES_N_, WAVES_M = WAVES_M_;
  static constexpr int KSPLIT = KSPLIT_, BK = BK_, STAGES = STAGES_;
  static constexpr int VEC = DType<DT>::VEC;
  static constexpr int NWAVES = WAVES_N * WAVES_M * KSPLIT;
  static constexpr int NT = 64 * NWAVES;
  static constexpr int BN = 16 * NBW * WAVES_N;
  static constexpr int BM = 16 * MBW * WAVES_M;
  // LDS rows padded by 32 bytes: 16-byte fragment reads of 16 rows at a
  // 160-byte stride run conflict-free on gfx950 (144 bytes: two-way conflicts)
  static constexpr int LDL = BK + 2 * VEC;
  static constexpr int KV = BK / VEC;   // 16-byte vectors per row chunk
  static constexpr int WV = BN * KV;
  static constexpr int XV = BM * KV;
  static constexpr int WIT = (WV + NT - 1) / NT;
  static constexpr int XIT = (XV + NT - 1) / NT;
  static constexpr int BUF = (BN + BM) * LDL;  // elements per LDS buffer
  static constexpr int NSLICE = BK / Mfma<DT>::KSLICE;
  static constexpr int RED_BYTES = (KSPLIT - 1) * WAVES_N * WAVES_M * NBW * MBW * 64 * 16;
  static constexpr int PIPE_BYTES = 2 * BUF * (int)sizeof(DT);
  static constexpr int LDS_BYTES = PIPE_BYTES > RED_BYTES ? PIPE_BYTES : RED_BYTES;
  static_assert(BK % Mfma<DT>::KSLICE == 0, "BK must be a multiple of the MFMA K slice");
  static_assert(NSLICE % KSPLIT == 0, "K slices must split evenly over the K waves");

  __device__ static int kw() { return (threadIdx.x >> 6) % KSPLIT; }
  __device__ static int wn() { return ((threadIdx.x >> 6) / KSPLIT) % WAVES_N; }
  __device__ static int wm() { return (threadIdx.x >> 6) / (KSPLIT * WAVES_N); }

  template <class S>
  __device__ __forceinline__ static void gload(uint4 (&wr)[WIT], uint4 (&xr)[XIT],
                                               const SrcX<DT>& w, const S& x, int Kpad, int k0) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int it = 0; it < WIT; ++it) {
      const int v = tid + it * NT;
      if (WV % NT == 0 || v < WV) wr[it] = w.load(w.row(v / KV), k0 + (v % KV) * VEC, Kpad);
    }
#pragma unroll
    for (int it = 0; it < XIT; ++it) {
      const int v = tid + it * NT;
      if (XV % NT == 0 || v < XV) xr[it] = x.load(x.row(v / KV), k0 + (v % KV) * VEC, Kpad);
    }
  }

  __device__ __forceinline__ static void sstore(const uint4 (&wr)[WIT], const uint4 (&xr)[XIT],
                                                DT* buf) {
    const int tid = threadIdx.x;
    DT* Xl = buf + BN * LDL;
#pragma unroll
    for (int it = 0; it < WIT; ++it) {
      const int v = tid + it * NT;
      if (WV % NT == 0 || v < WV)
        *reinterpret_cast<uint4*>(buf + (v / KV) * LDL + (v % KV) * VEC) = wr[it];
    }
#pragma unroll
    for (int it = 0; it < XIT; ++it) {
      const int v = tid + it * NT;
      if (XV % NT == 0 || v < XV)
        *reinterpret_cast<uint4*>(Xl + (v / KV) * LDL + (v % KV) * VEC) = xr[it];
    }
  }

  __device__ __forceinline__ static void compute(f32x4 (&acc)[NBW][MBW], const DT* buf) {
    const int lane = threadIdx.x & 63;
    const int g = lane >> 4, r16 = lane & 15;
    const int wni = wn(), wmi = wm();
    const DT* Xl = buf + BN * LDL;
    for (int sl = kw(); sl < NSLICE; sl += KSPLIT) {
      const int ks = sl * Mfma<DT>::KSLICE;
      uint4 a[NBW], b[MBW];
#pragma unroll
      for (int i = 0; i < NBW; ++i)
        a[i] = *reinterpret_cast<const uint4*>(buf + ((wni * NBW + i) * 16 + r16) * LDL + ks + g * VEC);
#pragma unroll
      for (int j = 0; j < MBW; ++j)
        b[j] = *reinterpret_cast<const uint4*>(Xl + ((wmi * MBW + j) * 16 + r16) * LDL + ks + g * VEC);
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < MBW; ++j) Mfma<DT>::step(acc[i][j], a[i], b[j]);
    }
  }

  // w: weight rows n0 .. n0+BN-1; x: activation rows m0 .. m0+BM-1.
  template <class S>
  __device__ __forceinline__ static void run(f32x4 (&acc)[NBW][MBW], const SrcX<DT>& w, const S& x,
                                             int Kpad, DT* lds) {
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
      for (int j = 0; j < MBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    uint4 wr[STAGES][WIT], xr[STAGES][XIT];
    const int nk = (Kpad + BK - 1) / BK;
#pragma unroll
    for (int s = 0; s < STAGES; ++s)
      if (s < nk) gload(wr[s], xr[s], w, x, Kpad, s * BK);
    sstore(wr[0], xr[0], lds);
    __syncthreads();
    for (int kc0 = 0; kc0 < nk; kc0 += STAGES) {
#pragma unroll
      for (int s = 0; s < STAGES; ++s) {
        const int kc = kc0 + s;
        if (kc < nk) {
          compute(acc, lds + (kc & 1) * BUF);
          if (kc + 1 < nk) sstore(wr[(s + 1) % STAGES], xr[(s + 1) % STAGES], lds + ((kc + 1) & 1) * BUF);
          if (kc + STAGES < nk) gload(wr[s], xr[s], w, x, Kpad, (kc + STAGES) * BK);
          __syncthreads();
        }
      }
    }
    if constexpr (KSPLIT > 1) {
      // sum the K partials into the kw == 0 waves (LDS is free after the loop)
      f32x4* red = reinterpret_cast<f32x4*>(lds);
      const int lane = threadIdx.x & 63;
      const int pos = wm() * WAVES_N + wn();
      const int k = kw();
      if (k > 0) {
#pragma unroll
        for (int i = 0; i < NBW; ++i)
#pragma unroll
          for (int j = 0; j < MBW; ++j)
            red[((((k - 1) * WAVES_N * WAVES_M + pos) * NBW + i) * MBW + j) * 64 + lane] = acc[i][j];
      }
      __syncthreads();
      if (k == 0) {
        for (int kk = 1; kk < KSPLIT; ++kk)
#pragma unroll
          for (int i = 0; i < NBW; ++i)
#pragma unroll
            for (int j = 0; j < MBW; ++j)
              acc[i][j] += red[((((kk - 1) * WAVES_N * WAVES_M + pos) * NBW + i) * MBW + j) * 64 + lane];
      }
      __syncthreads();
    }
  }
};

// ===========================================================================
// GEMM core for large row counts: operands go from global memory straight
// into LDS (buffer loads with the LDS-DMA modifier, no staging registers and
// no LDS store instructions, which on gfx950 run at about a third of the
// LDS read rate), through a ring of STAGES buffers so that the loads of
// chunk k + STAGES - 1 fly while chunk k is multiplied.  A chunk is 128 bytes
// of K per row (64 bf16 or 32 fp32 values, two MFMA K slices); rows are
// stored unpadded with their 16-byte pieces permuted, piece c of row r at
// slot c ^ ((r >> 1) & 7), which keeps the 16-row fragment reads free of
// bank conflicts.  One LDS-DMA instruction fills 8 rows (1 KB): lane l
// loads piece (l & 7) ^ ((row >> 1) & 7) of row 8q + (l >> 3).
// Same interface as Gemm (without a K split); Kpad must be a multiple of
// the chunk.
// ===========================================================================
struct NoWork {
  __device__ __forceinline__ void operator()() const {}
};

// Order of a product's sum over K.  In bf16 it is part of a call's results: h
// is stored rounded, so another order of the fp32 sums now and then moves an
// element of h by 2^-9 of its size, and a dream that follows a near-tie the
// other way from there is another dream.  A call's tile is chosen for speed;
// the order follows the call's rows alone:
//   Chain  one chain of MFMA slices over all of K;
//   Runs   the order of the register-direct core (GemmRD): a chain per wave's
//          run of consecutive slices, the runs summed in order;
//   Pairs  that of two waves taking turns: the even slices, plus the odd ones.
enum class KSum { Chain, Runs, Pairs };

// SPLIT (fp32): the fragments are split into three bf16 terms as they leave
// LDS and multiplied on the bf16 matrix unit (split3).  The split costs 5.5
// VALU instructions per fragment value, so it pays with at least four 16-row
// blocks a side per wave: 65536 x 1040 x 512 on 128 x 128 tiles of four waves
// 446 us (156 TFLOP/s) against 671 us for the fp32 MFMA on its best tile,
// 539 us on 128 x 64.
template <typename DT_, int NBW_, int MBW_, int WAVES_N_, int WAVES_M_, int STAGES_, bool SPLIT_ = false>
struct GemmD {
  using DT = DT_;
  static constexpr int NBW = NBW_, MBW = MBW_, WAVES_N = WAVES_N_, WAVES_M = WAVES_M_;
  static constexpr int STAGES = STAGES_, KSPLIT = 1;
  static constexpr int VEC = DType<DT>::VEC;
  static constexpr int BK = 128 / (int)sizeof(DT);  // K per chunk
  static constexpr int NWAVES = WAVES_N * WAVES_M;
  static constexpr int NT = 64 * NWAVES;
  static constexpr int BN = 16 * NBW * WAVES_N;
  static constexpr int BM = 16 * MBW * WAVES_M;
  static constexpr int ROWS = BN + BM;
  static constexpr int STAGE_BYTES = ROWS * 128;
  static constexpr int LDS_BYTES = STAGES * STAGE_BYTES;
  static constexpr int NQ = ROWS / 8;        // DMA instructions per chunk
  static constexpr int QW = NQ / NWAVES;     // ... per wave
  static_assert(NQ % NWAVES == 0 && BN % 8 == 0, "whole DMA instructions per wave");
  static_assert(STAGES >= 2 && (STAGES - 2) * QW < 64, "vmcnt range");
  static_assert(2 * Mfma<DT>::KSLICE == BK, "two MFMA K slices per chunk");
  static_assert(!SPLIT_ || sizeof(DT) == 4, "the split serves fp32 operands");

  __device__ static int kw() { return 0; }
  __device__ static int wn() { return (threadIdx.x >> 6) % WAVES_N; }
  __device__ static int wm() { return (threadIdx.x >> 6) / WAVES_N; }

  // this wave's chunks are in LDS once at most `young` later chunks are in flight
  __device__ __forceinline__ static void wait_chunks(int young) {
    if constexpr (STAGES >= 4) {
      if (young >= 2) { vm_wait<2 * QW>(); return; }
    }
    if constexpr (STAGES >= 3) {
      if (young >= 1) { vm_wait<QW>(); return; }
    }
    vm_wait<0>();
  }

  // GPERM: tile row 64 w + 16 i + 4 g + v of the weights is packed row
  // 64 w + 16 g + 4 v + i, so that with four 16-row blocks per wave, block i
  // of a wave holds gate i of 16 consecutive hidden units and lane (g, r16)
  // gets all four gates of units 4 g .. 4 g + 3 (the packed rows interleave
  // the gates per unit: row 4 u + q)
  // pre(): caller work that does not depend on the product, run once the
  // first chunks' loads are issued, so that it fills their latency
  // ORD, runs: the order of the sum over K (KSum)
  template <class S, bool GPERM = false, KSum ORD = KSum::Chain, class Pre = NoWork>
  __device__ __forceinline__ static void run(f32x4 (&acc)[NBW][MBW], const SrcX<DT>& w, const S& x,
                                             int Kpad, DT* lds, Pre&& pre = Pre{}, int runs = 0) {
    static_assert(!S::kTwo, "the direct core reads one activation matrix");
    static_assert(!GPERM || NBW == 4, "the gate permutation needs four blocks per wave");
    static_assert(!SPLIT_ || ORD == KSum::Chain, "split products are summed in one chain");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, r16 = lane & 15;
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) char*)reinterpret_cast<char*>(lds));
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
      for (int j = 0; j < MBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // per-lane source offsets of this wave's DMA instructions (chunk 0); the
    // two buffer resources are selected per instruction rather than held in
    // one register quad each, which kept the scalar registers spilling
    const u32x4 rw = rsrc_words(w.base, w.bytes), rx = rsrc_words(x.base, x.bytes);
    bool isw[QW];
    uint32_t off[QW];
#pragma unroll
    for (int t = 0; t < QW; ++t) {
      const int q = wave * QW + t;  // uniform
      const int row = 8 * q + (lane >> 3);
      const int c = (lane & 7) ^ ((row >> 1) & 7);
      isw[t] = q < BN / 8;
      const int wr = GPERM ? (row & ~63) | (((row >> 2) & 3) << 4) | ((row & 3) << 2) | ((row >> 4) & 3) : row;
      off[t] = isw[t] ? w.row(wr) + 16u * c : x.row(row - BN) + 16u * c;
    }
    const int nk = Kpad / BK;
    auto issue = [&](int kc) {
      const uint32_t base = lds0 + (uint32_t)(kc % STAGES) * STAGE_BYTES + (uint32_t)wave * QW * 1024u;
#pragma unroll
      for (int t = 0; t < QW; ++t) dma16(isw[t] ? rw : rx, off[t] + 128u * (uint32_t)kc, base + 1024u * t);
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
      if (s < nk) issue(s);
    pre();

    constexpr bool kRuns = ORD == KSum::Runs, kPairs = ORD == KSum::Pairs, kTwo = kRuns || kPairs;
    f32x4 tot[kTwo ? NBW : 1][kTwo ? MBW : 1];  // the runs before this one; the odd slices
    int left = runs;                            // slices left in the run
    if constexpr (kTwo) {
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < MBW; ++j) tot[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    const int wni = wn(), wmi = wm();
    const int sw = (r16 >> 1) & 7;
    const uint32_t col0 = (uint32_t)((g ^ sw) << 4), col1 = (uint32_t)(((4 + g) ^ sw) << 4);
    for (int kc = 0; kc < nk; ++kc) {
      wait_chunks(min(STAGES - 2, nk - 1 - kc));
      __builtin_amdgcn_s_barrier();  // no fence: it would wait for every load in flight
      asm volatile("" : : : "memory");
      if (kc + STAGES - 1 < nk) issue(kc + STAGES - 1);
      const char* buf = reinterpret_cast<const char*>(lds) + (kc % STAGES) * STAGE_BYTES;
      if constexpr (SPLIT_) {
        Split3 a[NBW];
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          const char* r = buf + ((wni * NBW + i) * 16 + r16) * 128;
          a[i] = split3(*reinterpret_cast<const uint4*>(r + col0), *reinterpret_cast<const uint4*>(r + col1));
        }
#pragma unroll
        for (int j = 0; j < MBW; ++j) {
          const char* r = buf + (BN + (wmi * MBW + j) * 16 + r16) * 128;
          const Split3 b = split3(*reinterpret_cast<const uint4*>(r + col0), *reinterpret_cast<const uint4*>(r + col1));
          f32x4 c[NBW];
#pragma unroll
          for (int i = 0; i < NBW; ++i) c[i] = acc[i][j];
          mfma_split(c, a, b);
#pragma unroll
          for (int i = 0; i < NBW; ++i) acc[i][j] = c[i];
        }
      } else {
#pragma unroll
        for (int sl = 0; sl < 2; ++sl) {
          const uint32_t col = sl ? col1 : col0;
          uint4 a[NBW], b[MBW];
#pragma unroll
          for (int i = 0; i < NBW; ++i)
            a[i] = *reinterpret_cast<const uint4*>(buf + ((wni * NBW + i) * 16 + r16) * 128 + col);
#pragma unroll
          for (int j = 0; j < MBW; ++j)
            b[j] = *reinterpret_cast<const uint4*>(buf + (BN + (wmi * MBW + j) * 16 + r16) * 128 + col);
          if constexpr (kRuns) {
            if (left == 0) {
#pragma unroll
              for (int i = 0; i < NBW; ++i)
#pragma unroll
                for (int j = 0; j < MBW; ++j) {
                  tot[i][j] += acc[i][j];
                  acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
              left = runs;
            }
            --left;
          }
#pragma unroll
          for (int i = 0; i < NBW; ++i)
#pragma unroll
            for (int j = 0; j < MBW; ++j) {
              if constexpr (kPairs) Mfma<DT>::step(sl ? tot[i][j] : acc[i][j], a[i], b[j]);
              else Mfma<DT>::step(acc[i][j], a[i], b[j]);
            }
        }
      }
    }
    if constexpr (kTwo) {
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < MBW; ++j) acc[i][j] = tot[i][j] + acc[i][j];
    }
    __syncthreads();  // LDS free for the caller's epilogue
    if constexpr (SPLIT_) {
      // An infinity, or a value that rounds to one in bf16, leaves NaN in every
      // sum it enters (inf - inf in the split's remainder): those sums are
      // taken again on the fp32 unit, one 16-row block of weights at a time.
      bool bad = false;
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < MBW; ++j) bad |= any_nan(acc[i][j]);
      int* flag = reinterpret_cast<int*>(lds);
      const uint64_t bal = __ballot(bad);
      if (lane == 0) flag[wave] = bal != 0;
      __syncthreads();
      int any = 0;
#pragma unroll
      for (int v = 0; v < NWAVES; ++v) any |= flag[v];
      __syncthreads();
      if (!__builtin_amdgcn_readfirstlane(any)) return;
#pragma unroll
      for (int ib = 0; ib < NBW; ++ib) {
        f32x4 c[MBW];
#pragma unroll
        for (int j = 0; j < MBW; ++j) c[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kc = 0; kc < nk; ++kc) {
          issue(kc);
          vm_wait<0>();
          __syncthreads();
          const char* buf = reinterpret_cast<const char*>(lds) + (kc % STAGES) * STAGE_BYTES;
#pragma unroll
          for (int sl = 0; sl < 2; ++sl) {
            const uint32_t col = sl ? col1 : col0;
            const uint4 a = *reinterpret_cast<const uint4*>(buf + ((wni * NBW + ib) * 16 + r16) * 128 + col);
#pragma unroll
            for (int j = 0; j < MBW; ++j)
              Mfma<DT>::step(c[j], a, *reinterpret_cast<const uint4*>(buf + (BN + (wmi * MBW + j) * 16 + r16) * 128 + col));
          }
          __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < MBW; ++j) acc[ib][j] = nan_to(acc[ib][j], c[j]);
      }
    }
  }
};

template <class C> struct IsGemmD : std::false_type {};
template <typename DT, int NBW, int MBW, int WN, int WM, int ST, bool SP>
struct IsGemmD<GemmD<DT, NBW, MBW, WN, WM, ST, SP>> : std::true_type {};

// Work-group -> tile mapping.  Work-groups are dispatched round-robin over
// the eight XCDs, each with its own L2.  The XCDs form a gn x (8 / gn) grid
// over (weight-row tiles, activation-row tiles): XCD x owns a contiguous
// range of nper weight tiles, so that its slice of the weights stays in its
// L2 across calls, and a range of mper activation tiles, which it walks
// with the weight tile fastest, so that an activation tile it has fetched
// is reused by all of its weight tiles while still in L2.  The host picks
// gn (tile_map below).  Returns false for padding work-groups.
struct TileMap {
  int nt, mt;      // weight-row tiles, activation-row tiles
  int gn;          // XCD groups along the weight tiles (1, 2, 4 or 8)
  int nper, mper;  // tiles of each kind per XCD
};

__device__ __forceinline__ bool tile_of(const TileMap& t, int& n, int& m) {
  const int x = blockIdx.x & 7, r = blockIdx.x >> 3;
  const int nl = r % t.nper, ml = r / t.nper;
  n = (x % t.gn) * t.nper + nl;
  m = (x / t.gn) * t.mper + ml;
  return n < t.nt && m < t.mt;
}

// ===========================================================================
// Register-direct split-K GEMM for calls with few rows.  Every wave takes a
// contiguous run of at most SMAX MFMA K slices and loads all of its operand
// fragments for the whole tile straight from global memory into registers in
// one round trip (no LDS staging, no barrier inside the K loop), then runs
// its MFMAs.  The per-wave partial tiles meet in LDS and are summed in a
// fixed wave order, so results are deterministic; the sum lands in
// E[m][n] (tile rows m, features n, fp32) for an epilogue with any thread
// mapping.  The block has nwaves = blockDim.x / 64 waves, chosen by the host
// so that ceil(K slices / nwaves) <= SMAX.
// ===========================================================================
template <typename DT_, int NBW_, int MBW_, int SMAX_, int MAXT_>
struct GemmRD {
  using DT = DT_;
  static constexpr int NBW = NBW_, MBW = MBW_, SMAX = SMAX_;
  static constexpr int MAXT = MAXT_;  // largest block the kernels are compiled for
  static constexpr int KSLICE = Mfma<DT>::KSLICE, VEC = DType<DT>::VEC;
  static constexpr int BN = 16 * NBW, BM = 16 * MBW;
  static constexpr int TILE = BN * BM;  // floats per partial tile
  static constexpr int ELD = BN + 4;    // row stride of E (floats)

  static size_t lds_bytes(int nwaves) {
    return (size_t)nwaves * TILE * 4 + (size_t)BM * ELD * 4;
  }
  __device__ static float* E(float* lds) { return lds + (blockDim.x >> 6) * TILE; }

  // w: weight rows n0 .. n0+BN-1; x: activation rows m0 .. m0+BM-1;
  // pre(): caller work that does not depend on the product, run while the
  // operands are in flight
  template <class S, class Pre = NoWork>
  __device__ __forceinline__ static void run(float* lds, const SrcX<DT>& w, const S& x, int Kpad, Pre&& pre = Pre{}) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int g = lane >> 4, r16 = lane & 15;
    const int nsl = (Kpad + KSLICE - 1) / KSLICE;
    const int per = (nsl + nw - 1) / nw;
    const int s0 = wave * per;
    typename SrcX<DT>::Row wo[NBW];
    typename S::Row xo[MBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i) wo[i] = w.row(i * 16 + r16);
#pragma unroll
    for (int j = 0; j < MBW; ++j) xo[j] = x.row(j * 16 + r16);
    uint4 wf[NBW][SMAX], xf[MBW][SMAX];
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      const int sl = s0 + s;
      if (s < per && sl < nsl) {
        const int kl = sl * KSLICE + g * VEC;  // first column of this lane's vector
#pragma unroll
        for (int i = 0; i < NBW; ++i) wf[i][s] = w.load(wo[i], kl, Kpad);
#pragma unroll
        for (int j = 0; j < MBW; ++j) xf[j][s] = x.load(xo[j], kl, Kpad);
      } else {
#pragma unroll
        for (int i = 0; i < NBW; ++i) wf[i][s] = make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < MBW; ++j) xf[j][s] = make_uint4(0, 0, 0, 0);
      }
    }
    pre();
    f32x4 acc[NBW][MBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
      for (int j = 0; j < MBW; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      if (s < per && s0 + s < nsl) {
#pragma unroll
        for (int i = 0; i < NBW; ++i)
#pragma unroll
          for (int j = 0; j < MBW; ++j) Mfma<DT>::step(acc[i][j], wf[i][s], xf[j][s]);
      }
    }
    float* P = lds + wave * TILE;
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
      for (int j = 0; j < MBW; ++j)
        *reinterpret_cast<f32x4*>(P + ((i * MBW + j) * 64 + lane) * 4) = acc[i][j];
    __syncthreads();
    float* Et = E(lds);
    for (int e = threadIdx.x; e < TILE; e += blockDim.x) {
      float sum = 0.f;
      for (int w2 = 0; w2 < nw; ++w2) sum += lds[w2 * TILE + e];
      const int v = e & 3, l = (e >> 2) & 63, ij = e >> 8;
      const int j = ij % MBW, i = ij / MBW;
      Et[(j * 16 + (l & 15)) * ELD + i * 16 + 4 * (l >> 4) + v] = sum;
    }
    __syncthreads();
  }
};

// ===========================================================================
// host helpers
// ===========================================================================
constexpr int kCUs = 256;
constexpr size_t kRdLdsMax = 64 * 1024;  // LDS of a register-direct launch

inline int rd_waves(int Kpad, int kslice, int smax, int min_waves) {
  const int nsl = (Kpad + kslice - 1) / kslice;
  int nw = (nsl + smax - 1) / smax;
  return nw < min_waves ? min_waves : nw;
}

// Waves of a launch of the register-direct tile R over Kpad columns (at least
// four), or 0 where they do not fit its compiled block size or the LDS; and
// the slices of each wave's run.
template <class R>
int rd_fit(int Kpad) {
  const int nw = rd_waves(Kpad, R::KSLICE, R::SMAX, 4);
  return 64 * nw <= R::MAXT && R::lds_bytes(nw) <= kRdLdsMax ? nw : 0;
}
template <class R>
int rd_run(int Kpad, int nw) {
  return ((Kpad + R::KSLICE - 1) / R::KSLICE + nw - 1) / nw;
}

// Dynamic LDS above the default needs the kernel attribute raised once.
template <typename F>
hipError_t allow_lds(F* kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Weight bytes an XCD should keep in its L2 (4 MB) while activations stream.
constexpr size_t kL2Budget = 2560 * 1024;

// Picks gn for nt x mt tiles over `wbytes` of weights: the weights' per-XCD
// slice fits the L2 budget if possible, then the busiest XCD gets the fewest
// tiles, then the activations are re-read by the fewest XCD groups.
inline TileMap tile_map(int nt, int mt, size_t wbytes) {
  TileMap best{};
  bool best_fits = false;
  long best_tiles = 0;
  for (int gn = 1; gn <= 8; gn *= 2) {
    if (gn > 1 && gn > nt) break;
    TileMap t{nt, mt, gn, (nt + gn - 1) / gn, (mt + 8 / gn - 1) / (8 / gn)};
    const bool fits = wbytes / gn <= kL2Budget;
    const long tiles = (long)t.nper * t.mper;
    if (gn == 1 || (fits && !best_fits) || (fits == best_fits && tiles < best_tiles)) {
      best = t;
      best_fits = fits;
      best_tiles = tiles;
    }
  }
  return best;
}

inline unsigned grid_of(const TileMap& t) { return (unsigned)(8 * t.nper * t.mper); }

}  // namespace wm
