// Column DFTs of the long transforms, N = N1 x N2 = 2^15 .. 2^20.
//
// The decomposition is that of the paper's eq. (3), n = n1 + N1 n2 and
// k = k2 + N2 k1:
//   stage 1: Y[k2][n1] = sum_{n2} x[n1 + N1 n2] W_N2^{n2 k2}
//   stage 2: X[k2 + N2 k1] = sum_{n1} W_N1^{n1 k1} W_N^{n1 k2} Y[k2][n1].
// A workgroup runs TILE transforms side by side, adjacent n1 in stage 1 and
// adjacent k2 in stage 2, each of length L = R0 x R1 in two register passes
// with one LDS exchange between them (R0 values per lane, R1 lanes per
// column).  Every access moves whole 128-byte segments, the workspace whole
// 2 KiB blocks.
//
// What bounds it: each stage reads and writes every byte once, so the floor is
// two copies; a copy in the same access pattern takes 16.3 us per stage at
// 2^16 x 101 rows and 39-43 us at 2^16 x 256 on an MI355X, the stages take
// 17.4 + 18.3 and 44.8 + 41.3 us.  The arithmetic (VALU issue) of a stage is 30
// to 39% of its busy cycles (counted at 2^16 x 101 and 2^20 x 16) and overlaps
// with the rest as far as the resident workgroups (16 waves per CU, limited by
// 128 VGPRs and 34 or 68 KiB of LDS) are in different phases; at 2^20 x 16 the
// grid is two rounds of them, and the stages take 51 + 50 us.  Against three radix-4 or radix-8 passes per stage
// and a closing transpose through LDS (the shape before) the two-pass columns
// measure 36.1 against 45.7 us (2^16 x 101), 37.4 against 45.5 (2^15 x 200),
// 76 against 91 (2^17 x 101), 81 against 94 (2^18 x 51), 101.3 against 118
// (2^20 x 16), 28.8 against 37.9 (2^20 x 3) and
// 8.4 against 11.9 (2^16 x 1).
#pragma once

#include "kernels.hpp"

namespace stockfft {

// One column transform: pass 0 has lane t take a DFT_R0 over the elements
// t + R1 m, its output k then belongs to pass-1 butterfly k, leg t; pass 1
// has lane t take butterflies j = t + T b (b < BPT) and leaves output
// j + R0 q in slot b R1 + q.  The exchange is thus a transpose of the
// (k, t) plane of each column.
//
// SPLIT sends the real parts, then the imaginary parts through the LDS: half
// the space, twice the (4-byte) accesses and two more barriers.
//
// LDS layout: slot k KROW + t TILE + c for column c, one TILE-wide pad per k
// row, so that the accesses with lanes c fastest hit every bank once in both
// passes (no conflict counted in stage 2).  FLIP (stage 1) changes the lane
// order to t fastest for pass 1; there the column is rotated by spread(k)
// inside its 16, which gives the 32 lanes of a half wave 32 different slots
// modulo the banks.  The counters still show those reads taking twice their
// cycles, a third of stage 1's LDS cycles (64 of 192 per wave, split 128 of
// 384); the LDS is busy for an eighth of that stage's cycles.
template <int R0_, int R1_, int TILE_, bool SPLIT_, int WPE_>
struct Col {
  static constexpr int R0 = R0_, R1 = R1_, TILE = TILE_, WPE = WPE_;
  static constexpr bool SPLIT = SPLIT_;
  static constexpr int L = R0 * R1, E = R0, T = R1, BPT = R0 / R1;
  static constexpr int THREADS = TILE * T;
  static constexpr int KROW = TILE * (R1 + 1);
  static constexpr int SLOTS = R0 * KROW;
  static constexpr int LDS_BYTES = SLOTS * (SPLIT ? 4 : 8);
  static_assert(R0 % R1 == 0 && (TILE == 16 || TILE == 32) && THREADS % 64 == 0, "column shape");
  __device__ __forceinline__ static constexpr int spread(int k) {
    return SPLIT ? (64 / T) * (k >> 2) : (32 / T) * (k >> 1);
  }
  template <bool FLIP>
  __device__ __forceinline__ static int slot(int c, int k, int t) {
    if constexpr (FLIP) c = (c + spread(k)) & (TILE - 1);
    return k * KROW + t * TILE + c;
  }
};

__device__ __forceinline__ void col_poison(float& v) { v = __builtin_nanf(""); }
__device__ __forceinline__ void col_poison(c32& v) { v = lds_poison(); }

// Moves one 4- or 8-byte value per (lane, register) through the LDS:
// w[k] of (s, t) to r[b R1 + q] = value of (lane q, output j = t2 + T b) of
// column s2.
template <class C, bool FLIP, class V>
__device__ __forceinline__ void col_transpose(const V (&w)[C::R0], V (&r)[C::R0], V* lds, int s, int t,
                                              int s2, int t2) {
#pragma unroll
  for (int k = 0; k < C::R0; ++k) lds[C::template slot<FLIP>(s, k, t)] = w[k];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < C::BPT; ++b)
#pragma unroll
    for (int q = 0; q < C::R1; ++q) {
      V& slot = lds[C::template slot<FLIP>(s2, t2 + C::T * b, q)];
      r[b * C::R1 + q] = slot;
      if constexpr (kLdsPoison) col_poison(slot);
    }
}

template <class C, bool FLIP>
__device__ __forceinline__ void col_exchange(c32 (&a)[C::E], void* lds, int s, int t, int s2, int t2) {
  if constexpr (kLdsPoison) {  // debug builds: the whole buffer starts as NaNs
#pragma unroll 1
    for (int i = threadIdx.x; i < C::LDS_BYTES / 4; i += C::THREADS) col_poison(static_cast<float*>(lds)[i]);
    __syncthreads();
  }
  if constexpr (C::SPLIT) {
    float w[C::E], x[C::E], y[C::E];
#pragma unroll
    for (int k = 0; k < C::E; ++k) w[k] = a[k].x;
    col_transpose<C, FLIP>(w, x, static_cast<float*>(lds), s, t, s2, t2);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < C::E; ++k) w[k] = a[k].y;
    col_transpose<C, FLIP>(w, y, static_cast<float*>(lds), s, t, s2, t2);
#pragma unroll
    for (int k = 0; k < C::E; ++k) a[k] = c32{x[k], y[k]};
  } else {
    c32 r[C::E];
    col_transpose<C, FLIP>(a, r, static_cast<c32*>(lds), s, t, s2, t2);
#pragma unroll
    for (int k = 0; k < C::E; ++k) a[k] = r[k];
  }
}

template <class C, bool INV>
__device__ __forceinline__ void col_pass1(c32 (&a)[C::E]) {
#pragma unroll
  for (int b = 0; b < C::BPT; ++b) {
    c32 v[C::R1];
#pragma unroll
    for (int q = 0; q < C::R1; ++q) v[q] = a[b * C::R1 + q];
    Dft<C::R1, INV>::run(v);
#pragma unroll
    for (int q = 0; q < C::R1; ++q) a[b * C::R1 + q] = v[q];
  }
}

__device__ __forceinline__ c32 as_c32(u32x2 v) { return c32{__uint_as_float(v.x), __uint_as_float(v.y)}; }
__device__ __forceinline__ u32x2 as_u32x2(c32 v) { return u32x2{__float_as_uint(v.x), __float_as_uint(v.y)}; }

// Stage 1 of one tile: src and dst at the row's start (x, workspace).
// Workspace layout [k2 div KB][n1][k2 mod KB], KB the second stage's tile
// width: the task writes runs of KB values, the second stage reads its tile
// as one contiguous block.
// ptab: [k][t] = W_L^{k t}.
template <class C, int N1, int KB, bool INV, int LD>
__device__ __forceinline__ void col_stage1(const c32* src, c32* dst, const c32* ptab, void* lds, int tile) {
  const int tid = threadIdx.x;
  const int s = tid % C::TILE, t = tid / C::TILE;
  const Buf in(src);
  c32 a[C::E];
  const int vin = 8 * (tile * C::TILE + s + N1 * t);
#pragma unroll
  for (int m = 0; m < C::E; ++m) a[m] = as_c32(in.ld64<LD>(vin, 8 * N1 * C::R1 * m));
  const Buf pb(ptab);
  if constexpr (C::R0 <= 16) {  // registers to spare: the twiddles arrive with the data
    c32 p[C::R0];
#pragma unroll
    for (int k = 1; k < C::R0; ++k) p[k] = as_c32(pb.ld64(8 * t, 8 * C::T * k));
    Dft<C::R0, INV>::run(a);
#pragma unroll
    for (int k = 1; k < C::R0; ++k) a[k] = ctw<INV>(a[k], p[k]);
  } else {
    Dft<C::R0, INV>::run(a);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 1; k < C::R0; ++k) a[k] = ctw<INV>(a[k], as_c32(pb.ld64(8 * t, 8 * C::T * k)));
  }
  const int s2 = tid / C::T, t2 = tid % C::T;
  col_exchange<C, true>(a, lds, s, t, s2, t2);
  col_pass1<C, INV>(a);
  const Buf out(dst);
  const int vout = 8 * ((t2 / KB) * (N1 * KB) + (tile * C::TILE + s2) * KB + t2 % KB);
#pragma unroll
  for (int b = 0; b < C::BPT; ++b)
#pragma unroll
    for (int q = 0; q < C::R1; ++q) {
      const int c = C::T * b + C::R0 * q;
      out.st64<kDeviceScope>(as_u32x2(a[b * C::R1 + q]), vout, 8 * ((c / KB) * (N1 * KB) + c % KB));
    }
}

// Stage 2 of one tile of KB = TILE adjacent k2.  The stage twiddle of element
// n1 = t + R1 m is W_N^{n1 k2} = W_N^{t k2} W_{N / R1}^{m k2}: btab
// [tile][m][k2 mod TILE] holds the second factor, applied as the elements
// arrive; atab [tile][t][k2 mod TILE] the first, which is the same for every
// leg of the lane's DFT and so is applied to its outputs together with
// ptab [k][t] = W_L^{k t}.
template <class C, int N2, bool INV, int LD>
__device__ __forceinline__ void col_stage2(const c32* src, c32* dst, const c32* ptab, const c32* atab,
                                           const c32* btab, void* lds, int tile) {
  const int tid = threadIdx.x;
  const int s = tid % C::TILE, t = tid / C::TILE;
  const Buf in(src + (int64_t)tile * (C::L * C::TILE));
  c32 a[C::E];
#pragma unroll
  for (int m = 0; m < C::E; ++m) a[m] = as_c32(in.ld64<LD>(8 * tid, 8 * C::THREADS * m));
  {
    const Buf bb(btab + tile * (C::R0 * C::TILE));
    c32 w[C::R0];
#pragma unroll
    for (int m = 1; m < C::R0; ++m) w[m] = as_c32(bb.ld64(8 * s, 8 * C::TILE * m));
#pragma unroll
    for (int m = 1; m < C::R0; ++m) a[m] = ctw<INV>(a[m], w[m]);
  }
  Dft<C::R0, INV>::run(a);
  {
    const c32 w0 = as_c32(Buf(atab + tile * C::THREADS).ld64(8 * tid, 0));
    const Buf pb(ptab);
    a[0] = ctw<INV>(a[0], w0);
#pragma unroll
    for (int k = 1; k < C::R0; ++k) a[k] = ctw<INV>(a[k], cmul(w0, as_c32(pb.ld64(8 * t, 8 * C::T * k))));
  }
  col_exchange<C, false>(a, lds, s, t, s, t);
  col_pass1<C, INV>(a);
  const Buf out(dst);
  const int vout = 8 * (tile * C::TILE + s + N2 * t);
#pragma unroll
  for (int b = 0; b < C::BPT; ++b)
#pragma unroll
    for (int q = 0; q < C::R1; ++q)
      out.st64<kNT>(as_u32x2(a[b * C::R1 + q]), vout, 8 * N2 * (C::T * b + C::R0 * q));
}

// A split N = N1 x N2: C1 is the N2-point stage-1 shape, C2 the N1-point
// stage-2 shape.  Tables, one after another: P1, P2 (each shape's ptab), atab,
// btab (column_twiddles in twiddles.hpp builds them).
template <class C1_, class C2_>
struct Split {
  using C1 = C1_;
  using C2 = C2_;
  static constexpr int N1 = C2::L, N2 = C1::L;
  static constexpr int64_t N = (int64_t)N1 * N2;
  static constexpr int TILES1 = N1 / C1::TILE, TILES2 = N2 / C2::TILE;
  static constexpr int P1 = 0, P2 = P1 + C1::L, A = P2 + C2::L, B = A + N2 * C2::R1;
  static constexpr ColumnShape shape{C1::R0, C1::R1, C2::R0, C2::R1, C2::TILE};
};

template <class S, bool INV, int LD>
__global__ __launch_bounds__(S::C1::THREADS, S::C1::WPE) void k_columns_first(const c32* x, c32* y, const c32* tab) {
  __shared__ alignas(16) char lds[S::C1::LDS_BYTES];
  const int64_t row = blockIdx.x / S::TILES1;
  const int tile = (int)(blockIdx.x - row * S::TILES1);
  col_stage1<typename S::C1, S::N1, S::C2::TILE, INV, LD>(x + row * S::N, y + row * S::N, tab + S::P1, lds, tile);
}

template <class S, bool INV, int LD>
__global__ __launch_bounds__(S::C2::THREADS, S::C2::WPE) void k_columns_second(const c32* y, c32* out,
                                                                               const c32* tab) {
  __shared__ alignas(16) char lds[S::C2::LDS_BYTES];
  const int64_t row = blockIdx.x / S::TILES2;
  const int tile = (int)(blockIdx.x - row * S::TILES2);
  col_stage2<typename S::C2, S::N2, INV, LD>(y + row * S::N, out + row * S::N, tab + S::P2, tab + S::A, tab + S::B,
                                         lds, tile);
}

inline int64_t column_rows_per_launch(int tiles) {
  const int64_t per = max_groups_per_launch() / tiles;
  return per > 0 ? per : 1;
}

// Cache policy of the row and workspace loads: ordinary while input,
// workspace and output fit the 256 MiB Infinity Cache together, streaming
// beyond.  Both stages, us on an MI355X, ordinary / streaming: 2^16 x 101
// (159 MB) 36.1 / 39.3, 2^17 x 101 (318 MB) 76.1 / 75.6, 2^20 x 16 (403 MB)
// 103.7 / 102.9, 2^16 x 512 204 / 165, 2^20 x 32 235 / 190, 2^20 x 64 438 / 382.
inline bool columns_stream(int64_t batch, int64_t n) { return 3 * 8 * batch * n > (int64_t(256) << 20); }

// One workgroup per tile: a grid of exactly rows x tiles, no bounds to check.
template <class S, int LD>
hipError_t launch_columns_first_as(const c32* x, c32* y, const c32* tab, int64_t batch, bool inverse, hipStream_t s) {
  const int64_t per = column_rows_per_launch(S::TILES1);
  for (int64_t r0 = 0; r0 < batch; r0 += per) {
    const int64_t rows = batch - r0 < per ? batch - r0 : per;
    const dim3 grid((unsigned)(rows * S::TILES1)), block(S::C1::THREADS);
    if (inverse)
      k_columns_first<S, true, LD><<<grid, block, 0, s>>>(x + r0 * S::N, y + r0 * S::N, tab);
    else
      k_columns_first<S, false, LD><<<grid, block, 0, s>>>(x + r0 * S::N, y + r0 * S::N, tab);
  }
  return hipGetLastError();
}
template <class S, int LD>
hipError_t launch_columns_second_as(const c32* y, c32* out, const c32* tab, int64_t batch, bool inverse, hipStream_t s) {
  const int64_t per = column_rows_per_launch(S::TILES2);
  for (int64_t r0 = 0; r0 < batch; r0 += per) {
    const int64_t rows = batch - r0 < per ? batch - r0 : per;
    const dim3 grid((unsigned)(rows * S::TILES2)), block(S::C2::THREADS);
    if (inverse)
      k_columns_second<S, true, LD><<<grid, block, 0, s>>>(y + r0 * S::N, out + r0 * S::N, tab);
    else
      k_columns_second<S, false, LD><<<grid, block, 0, s>>>(y + r0 * S::N, out + r0 * S::N, tab);
  }
  return hipGetLastError();
}

template <class S>
hipError_t launch_columns_first(const void* x, void* y, const void* /*tw*/, const void* tab, int64_t batch,
                                bool inverse, hipStream_t s) {
  return (columns_stream(batch, S::N) ? launch_columns_first_as<S, kNT> : launch_columns_first_as<S, 0>)(
      static_cast<const c32*>(x), static_cast<c32*>(y), static_cast<const c32*>(tab), batch, inverse, s);
}
template <class S>
hipError_t launch_columns_second(const void* y, void* out, const void* /*tw*/, const void* tab, int64_t batch,
                                 bool inverse, hipStream_t s) {
  return (columns_stream(batch, S::N) ? launch_columns_second_as<S, kNT> : launch_columns_second_as<S, 0>)(
      static_cast<const c32*>(y), static_cast<c32*>(out), static_cast<const c32*>(tab), batch, inverse, s);
}

}  // namespace stockfft
