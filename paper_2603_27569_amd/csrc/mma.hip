// Radix-16 Stockham passes whose 16-point DFTs run on the matrix cores
// (the paper's matrix-multiply DFT of Sections V-C and VII-C, and its
// future-work items on batched matrix-core FFTs and mixed precision,
// Section IX-A), for N = 512 ... 16384 with binary16 or bfloat16 storage.
//
// One pass is 256 butterflies of 16 legs.  Written as real arithmetic, a
// 16-point DFT is a 32 x 32 matrix M acting on the 32 reals of a butterfly
// (real parts of the legs, then imaginary parts):
//   M = [[C, S], [-S, C]],  C[k][r] = cos(2 pi k r / 16),  S[k][r] = sin(...)
// (forward; the backward transform negates S).  A wave takes 32 butterflies
// as the 32 columns of a 32 x 32 operand and forms M times it with two
// v_mfma_f32_32x32x16 products (K = 32 split in two halves of 16): the
// operands are rounded to the 16-bit format, products are exact and the
// sums are FP32.  Each pass's outputs get the next pass's twiddles in FP32 on
// the vector ALUs and are rounded once to the 16-bit format as they go into
// LDS, so the exchange moves 16-bit pairs and the next pass reads its
// operands without converting (the first pass reads them from HBM as
// stored).
//
// Lane layouts of the 32x32x16 products (checked on gfx950): lane l holds
// A[l % 32][8 (l / 32) + e] and B[8 (l / 32) + e][l % 32] for e < 8, and the
// result D[8 (g / 4) + 4 (l / 32) + g % 4][l % 32] in accumulator g < 16.
// So lane (j = l % 32, h = l / 32) supplies legs 8h .. 8h + 7 of butterfly j
// (real parts to the first product, imaginary parts to the second) and gets
// back bins 4h .. 4h + 3 and 8 + 4h .. 8 + 4h + 3 of the same butterfly, real
// parts in accumulators 0 .. 7 and imaginary parts in 8 .. 15.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.hpp"
#include "kernels.hpp"

namespace stockfft {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// N = 16^P * RL: P radix-16 passes on the matrix cores, then (RL > 1) one
// radix-RL pass on the vector ALUs.
template <int N>
struct MmaPlan {
  static constexpr int RL = N == 512 || N == 8192 ? 2 : N == 1024 || N == 16384 ? 4 : N == 2048 ? 8 : 1;
  static constexpr int P = N / RL == 256 ? 2 : 3;
  static constexpr int NB = N / 16;     // butterflies per radix-16 pass
  static constexpr int NL = N / RL;     // butterflies of the last pass (RL > 1)
  static constexpr int LDS = N + N / 16;  // one pad slot per 16 against bank conflicts
  static_assert(N / RL == (P == 2 ? 256 : 4096) && NB % 32 == 0, "unsupported length");
  // Offset of pass p's twiddle table (entries [r - 1][k], as the host builds it).
  static constexpr int tw_off(int p) {
    int o = 0, ns = 16;
    for (int i = 1; i < p; ++i, ns *= 16) o += 15 * ns;
    return o;
  }
};

__device__ __forceinline__ int pidx(int i) { return i + (i >> 4); }

// The 16-bit operand format: binary16 storage multiplies binary16 operands,
// bfloat16 storage bfloat16 operands.
template <class IO>
struct MmaOps;

template <>
struct MmaOps<IoF16> {
  typedef _Float16 E;
  typedef f16x8 V;
  __device__ __forceinline__ static f32x16 mma(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

template <>
struct MmaOps<IoBF16> {
  typedef __bf16 E;
  typedef bf16x8 V;
  __device__ __forceinline__ static f32x16 mma(V a, V b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};

// M as the two A operands, one 32-byte record per lane: row l % 32, columns
// 8 (l / 32) + e (real legs, first product), then 16 + 8 (l / 32) + e.  Two
// 16-byte loads per lane from a 2 KiB table that stays in the caches, in
// flight with the first rows; formed from cosines in registers it took a
// lookup, a sign and a conversion for each of the 16 entries.
template <class IO, bool INV>
struct DftMatrix {
  alignas(16) typename MmaOps<IO>::E e[64][16];
  constexpr DftMatrix() : e() {
    // cos(2 pi m / 16) from the FP64 values; sin(2 pi m / 16) is entry m + 12.
    constexpr float c1 = 0.92387953251128674, c2 = 0.70710678118654757, c3 = 0.38268343236508978;
    constexpr float t[16] = {1.f, c1, c2, c3, 0.f, -c3, -c2, -c1, -1.f, -c1, -c2, -c3, 0.f, c3, c2, c1};
    for (int l = 0; l < 64; ++l)
      for (int i = 0; i < 16; ++i) {
        const int row = l & 31, leg = 8 * (l >> 5) + (i & 7), m = (row & 15) * leg & 15;
        const float c = t[m], s = INV ? -t[(m + 12) & 15] : t[(m + 12) & 15];
        const bool re_row = row < 16, re_leg = i < 8;
        e[l][i] = (typename MmaOps<IO>::E)(re_row == re_leg ? c : re_row ? s : -s);
      }
  }
};
template <class IO, bool INV>
__device__ const DftMatrix<IO, INV> kDftMatrix{};

// The 8 real parts (lo) or imaginary parts (hi) of 8 stored 16-bit pairs as
// one operand: dword i of the operand is half 0 or 1 of pairs 2i and 2i + 1.
template <class V>
__device__ __forceinline__ V gather_halves(const uint32_t (&d)[8], bool hi) {
  const unsigned sel = hi ? 0x07060302u : 0x05040100u;
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], sel);
  return __builtin_bit_cast(V, w);
}

// Twiddles of the 8 bins that lane half h holds of pass p's butterfly j.  Bin
// k goes to x = (j / Ns) Ns 16 + j mod Ns + k Ns.  The next pass (radix R',
// Ns' = 16 Ns, N / R' butterflies) reads it as leg r' = x / (N / R') of
// butterfly j' = x mod (N / R'), whose twiddle there is W_{Ns' R'}^{r' (j' mod
// Ns')}: table entry tw_off + (r' - 1) Ns' + j' mod Ns'.  k Ns never carries
// into r' or out of j' mod Ns', so all bins of a butterfly share r' and their
// entries lie k Ns apart: one lane offset, constant steps, and for Ns = 1 two
// bins in one 16-byte load.  Leg 0 has no entry: it reads leg 1's and takes 1
// instead.
template <class M>
__device__ __forceinline__ void next_twiddles(c32 (&wn)[8], const char* table, int p, int j, int h) {
  const int ns = p == 0 ? 1 : p == 1 ? 16 : 256;
  const bool last16 = p + 1 == M::P;
  if (last16 && M::RL == 1) return;
  const int nsn = 16 * ns;
  const int span = last16 ? M::NL : M::NB;  // N / R' (a power of two)
  const int off = M::tw_off(p + 1);
  const int base = (j / ns) * ns * 16 + (j & (ns - 1));
  const int r = base / span;
  const unsigned voff = 8u * ((r > 0 ? r - 1 : 0) * nsn + (base & (nsn - 1)) + 4 * h * ns);
  if (ns == 1) {
#pragma unroll
    for (int q = 0; q < 8; q += 2) {
      const u32x4 v = *reinterpret_cast<const u32x4*>(table + 8 * (off + q + (q & 4)) + voff);
      wn[q] = c32{__uint_as_float(v.x), __uint_as_float(v.y)};
      wn[q + 1] = c32{__uint_as_float(v.z), __uint_as_float(v.w)};
    }
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const u32x2 v = *reinterpret_cast<const u32x2*>(table + 8 * (off + (q + (q & 4)) * ns) + voff);
      wn[q] = c32{__uint_as_float(v.x), __uint_as_float(v.y)};
    }
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) wn[q] = r > 0 ? wn[q] : c32{1.f, 0.f};
}

// a w, or a conj(w) for the backward transform, with its fused operations spelled
// out: left to the compiler they come out differently with four blocks per
// wave, and the bits of a row would depend on the size of its batch.
template <bool INV>
__device__ __forceinline__ c32 twiddled(c32 a, c32 w) {
  if constexpr (INV) return {__builtin_fmaf(a.x, w.x, a.y * w.y), __builtin_fmaf(a.y, w.x, -(a.x * w.y))};
  else return {__builtin_fmaf(a.x, w.x, -(a.y * w.y)), __builtin_fmaf(a.x, w.y, a.y * w.x)};
}

// Waves per SIMD to leave registers for.  Two blocks' products and twiddles
// fit the 64 registers of 8 waves when the blocks go one after the other
// (512's unrolled radix-2 pass needs a few more), four together those of 4.
constexpr int mma_waves(int n, int blocks) { return blocks == 4 ? 4 : n == 512 && blocks == 2 ? 6 : 8; }

// TPWG transforms per workgroup of THREADS lanes, each wave taking kBlocks
// blocks of 32 butterflies of one transform or, for short transforms, of
// several.  Bound by the latency of a pass (matrix products of 16 cycles an
// instruction, an LDS round trip and the twiddles from L1 / L2) until enough
// waves are in flight, then by memory.
template <int N, int THREADS, int TPWG, bool INV, class IO>
__global__ __launch_bounds__(THREADS, mma_waves(N, TPWG * (N / 512) / (THREADS / 64))) void
k_stockham_mma(const uint32_t* in, uint32_t* out, const c32* __restrict__ tw, int64_t rows,
               int stream) {
  using M = MmaPlan<N>;
  constexpr int NB = M::NB;
  constexpr int BPT = NB / 32;  // blocks per transform
  constexpr int kBlocks = TPWG * BPT / (THREADS / 64);
  static_assert(M::RL > 1 || TPWG == 1, "the last radix-16 pass stores every slot");
  static_assert(kBlocks >= 1 && kBlocks * (THREADS / 64) == TPWG * BPT, "lanes per transform");
  constexpr int G = kBlocks == 4 ? 4 : 1;  // blocks whose products are in flight together
  using Ops = MmaOps<IO>;
  using V = typename Ops::V;
  __shared__ alignas(16) uint32_t lds[TPWG * M::LDS];  // 16-bit pairs, one pad per 16
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int jl = lane & 31;
  const int h = lane >> 5;
  const int64_t row0 = (int64_t)blockIdx.x * TPWG;
  if (row0 >= rows) return;  // whole workgroup, before any barrier

  // Block b of this wave: transform tr[b] of the workgroup, butterfly j[b];
  // rows past the batch (a last, partial workgroup) store nothing.
  int j[kBlocks], tr[kBlocks];
  bool live[kBlocks];
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
  for (int b = 0; b < kBlocks; ++b) {
    const int g = wave * kBlocks + b;
    tr[b] = TPWG > 1 ? g / BPT : 0;
    j[b] = 32 * (g - tr[b] * BPT) + jl;
    live[b] = TPWG == 1 || row0 + tr[b] < rows;  // one transform: row0 < rows
  }

  // Legs 8h + e of each butterfly as stored pairs: the first pass takes its
  // operands straight from HBM, the later ones from LDS, where the writer has
  // already applied their twiddles and rounded.  Rows, tables and results go
  // through buffer descriptors: every access is a lane part plus a constant.
  // A slot past the last row loads the workgroup's first row instead.
  uint32_t d[kBlocks][8];
  {
    const Buf src(in + row0 * N);
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
      const int voff = 4 * ((live[b] ? tr[b] : 0) * N + j[b] + 8 * h * NB);
      if (stream) {
#pragma unroll
        for (int e = 0; e < 8; ++e) d[b][e] = src.ld32<kNT>(voff, 4 * e * NB);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) d[b][e] = src.ld32(voff, 4 * e * NB);
      }
    }
  }
  const V* const m = reinterpret_cast<const V*>(kDftMatrix<IO, INV>.e[lane]);
  const V a_re = m[0], a_im = m[1];
  const char* const table = reinterpret_cast<const char*>(tw);

#pragma unroll
  for (int p = 0; p < M::P; ++p) {
    const int ns = 1 << (4 * p);  // Ns of this pass
    const bool last16 = p == M::P - 1;
    // With one pad element per 16 the padded slots are affine in k: pidx(x) =
    // pidx(x at k = 0) + k for Ns = 1 (x = 16 j + k) and + 17 Ns / 16 k for
    // Ns >= 16, so every write is a base address plus a constant.
    const int step = p == 0 ? 1 : 17 * ns / 16;
#pragma unroll
    for (int b0 = 0; b0 < kBlocks; b0 += G) {
      c32 wn[G][8];
      f32x16 acc[G];
#pragma unroll
      for (int g = 0; g < G; ++g) next_twiddles<M>(wn[g], table, p, j[b0 + g], h);
#pragma unroll
      for (int g = 0; g < G; ++g)
        acc[g] = Ops::mma(a_re, gather_halves<V>(d[b0 + g], false), f32x16{});
#pragma unroll
      for (int g = 0; g < G; ++g)
        acc[g] = Ops::mma(a_im, gather_halves<V>(d[b0 + g], true), acc[g]);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const int b = b0 + g;
        if (last16 && M::RL == 1) {
          // Last pass (Ns = N / 16): bin k of butterfly j is element j + k N / 16.
          const Buf dst(out + row0 * N);
          const int voff = 4 * (tr[b] * N + j[b] + 4 * h * NB);
#pragma unroll
          for (int q = 0; q < 8; ++q)
            dst.st32<kNT>(IO::store(c32{acc[g][q], acc[g][8 + q]}), voff, 4 * (q + (q & 4)) * NB);
        } else {
          uint32_t* wr = lds + tr[b] * M::LDS + pidx((j[b] / ns) * ns * 16 + (j[b] & (ns - 1))) +
                         step * 4 * h;
#pragma unroll
          for (int q = 0; q < 8; ++q)
            wr[step * (q + (q & 4))] = IO::store(twiddled<INV>(c32{acc[g][q], acc[g][8 + q]}, wn[g][q]));
        }
      }
    }
    if (last16 && M::RL == 1) return;
    __syncthreads();
    if (!last16) {
      // pidx(j + r N / 16) = pidx(j) + 17 N / 256 r.
#pragma unroll
      for (int b = 0; b < kBlocks; ++b) {
        const uint32_t* rd = lds + tr[b] * M::LDS + pidx(j[b]) + (17 * NB / 16) * 8 * h;
#pragma unroll
        for (int e = 0; e < 8; ++e) d[b][e] = rd[(17 * NB / 16) * e];
      }
      __syncthreads();
    }
  }
  if constexpr (M::RL > 1) {
    // The radix-RL pass (Ns = N / RL) on the vector ALUs in FP32: butterfly j
    // reads legs j + r N / RL (twiddles already applied) and writes bin k to
    // element j + k N / RL.
    constexpr int R = M::RL, NL = M::NL;
    static_assert(NL % 16 == 0 && (NL % THREADS == 0 || THREADS % NL == 0), "whole pad rows");
    const Buf dst(out + row0 * N);
#pragma unroll
    for (int i = tid; i < TPWG * NL; i += THREADS) {
      const int t = i / NL, jb = i - t * NL;
      if (TPWG > 1 && row0 + t >= rows) continue;
      const uint32_t* rd = lds + t * M::LDS + pidx(jb);
      c32 v[R];
#pragma unroll
      for (int r = 0; r < R; ++r) v[r] = IO::load(rd[r * (NL + NL / 16)]);
      Dft<R, INV>::run(v);
      const int voff = 4 * (t * N + jb);
#pragma unroll
      for (int k = 0; k < R; ++k) dst.st32<kNT>(IO::store(v[k]), voff, 4 * k * NL);
    }
  }
}

// Loads (stream_rows).  Up to 44 MiB in and out, two thirds of a generation of
// waves, the hint is faster or level wherever the rows are; above 192 MiB the
// cache holds no part worth having.  us on an MI355X, rows from HBM / just
// written, hint against ordinary: 4096 x 1050 9.7 / 9.0 against 10.0 / 9.3, 2048
// x 2500 10.5 / 9.8 against 11.0 / 10.0, bfloat16 2048 x 3000 12.9 / 11.9 against
// 13.4 / 10.2, 4096 x 2048 14.6 / 13.8 against 15.4 / 13.9, 4096 x 2500 21.5 /
// 20.2 against 22.1 / 16.5, 2048 x 8000 31.9 / 30.6 against 32.7 / 24.1, 4096 x
// 6000 45.5 / 44.4 against 46.2 / 45.9.
constexpr int64_t kOrdinaryFrom = int64_t(44) << 20, kOrdinaryTo = int64_t(192) << 20;

template <int N, int THREADS, class IO, int TPWG = 1>
hipError_t launch_mma_threads(const void* in, void* out, const void* tw, int64_t batch,
                              bool inverse, hipStream_t s) {
  const int64_t cap = max_groups_per_launch() * TPWG;  // rows per launch
  const int stream = stream_rows(2 * batch * N * (int64_t)sizeof(uint32_t), kOrdinaryFrom, kOrdinaryTo);
  for (int64_t r0 = 0; r0 < batch; r0 += cap) {
    const int64_t rows = batch - r0 < cap ? batch - r0 : cap;
    const uint32_t* ip = static_cast<const uint32_t*>(in) + r0 * N;
    uint32_t* op = static_cast<uint32_t*>(out) + r0 * N;
    const c32* twp = static_cast<const c32*>(tw);
    const dim3 grid((unsigned)((rows + TPWG - 1) / TPWG)), block(THREADS);
    if (inverse)
      k_stockham_mma<N, THREADS, TPWG, true, IO><<<grid, block, 0, s>>>(ip, op, twp, rows, stream);
    else
      k_stockham_mma<N, THREADS, TPWG, false, IO><<<grid, block, 0, s>>>(ip, op, twp, rows, stream);
  }
  return hipGetLastError();
}

// Blocks of 32 butterflies per wave, by the blocks of the launch (the chip has
// 1024 SIMDs).  Device time per launch with 1 / 2 / 4 per wave (4: products
// together), binary16, input in the Infinity Cache, microseconds:
//   up to four waves of one block per SIMD a pass's latency decides, and one
//   block is the shortest chain: 512 x 129 2.25 / 3.2 / 4.9, 2048 x 513 4.1 /
//   4.9 / 5.4, 4096 x 257 4.6 / 4.8 / 5.8, 8192 x 129 6.5 / 6.8 / 7.6;
//   beyond, two blocks share the matrix operands and leave fewer waves to
//   start: 512 x 6145 7.2 / 6.7 / 8.1, 2048 x 4097 16.4 / 15.6 / 16.8, 8192 x
//   3201 69.6 / 67.5 / 70.7;
//   512 and 1024 gain from whole transforms per wave once all waves are full
//   (1024 x 8193 15.9 / 15.7 / 14.2, x 25601 51.6 / 52.1 / 46.3); at 2048 and
//   4096 four blocks keep a launch of 12 to 16 blocks per SIMD in one generation
//   of half the waves (2 / 4 per wave, rows from HBM, then just written): 4096 x
//   1500 12.3 / 12.3, 10.6 / 11.6, x 1625 15.9 / 13.0, 11.9 / 12.2, x 2048 18.9 /
//   15.4, 13.6 / 13.8, x 2500 22.1 / 24.2, 16.5 / 18.1; 2048 x 3500 17.5 / 14.0,
//   12.2 / 12.7.  bfloat16, whose rounding takes more operations, gains at 4096
//   (x 2048 18.1 / 16.6, 13.5 / 13.1) but not at 2048 (x 3250 15.8 / 13.4, 10.7 /
//   12.4); 8192 does not gain (x 1024 19.0 / 19.1, 18.1 / 18.2).
// 16384 has no one-block form (2048 lanes).  The kernel before this one (four
// blocks, 102 ... 168 registers, 64-bit addresses and the matrix formed in
// registers) took 6.9 at 512 x 129, 5.6 at 2048 x 513, 5.2 at 4096 x 257, 7.9 at
// 8192 x 129, 11.7 at 512 x 6145, 19.4 at 2048 x 4097, 19.6 at 1024 x 8193, 17.6
// at 4096 x 2048 and 93.2 at 16384 x 1601 (now 70.5).
template <class IO>
hipError_t launch_mma(int64_t n, const void* in, void* out, const void* tw, int64_t batch,
                      bool inverse, hipStream_t s) {
  const int64_t blocks = batch * (n / 512);
  const bool one = blocks <= 4096, four = n <= 1024 ? blocks > 8192 : blocks > 12288 && blocks <= 16384;
  switch (n) {
    case 512:
      if (one) return launch_mma_threads<512, 64, IO, 1>(in, out, tw, batch, inverse, s);
      if (!four) return launch_mma_threads<512, 64, IO, 2>(in, out, tw, batch, inverse, s);
      return launch_mma_threads<512, 64, IO, 4>(in, out, tw, batch, inverse, s);
    case 1024:
      if (one) return launch_mma_threads<1024, 128, IO>(in, out, tw, batch, inverse, s);
      if (!four) return launch_mma_threads<1024, 64, IO>(in, out, tw, batch, inverse, s);
      return launch_mma_threads<1024, 64, IO, 2>(in, out, tw, batch, inverse, s);
    case 2048:
      if (one) return launch_mma_threads<2048, 256, IO>(in, out, tw, batch, inverse, s);
      if constexpr (std::is_same<IO, IoF16>::value)
        if (four) return launch_mma_threads<2048, 64, IO>(in, out, tw, batch, inverse, s);
      return launch_mma_threads<2048, 128, IO>(in, out, tw, batch, inverse, s);
    case 4096:
      if (one) return launch_mma_threads<4096, 512, IO>(in, out, tw, batch, inverse, s);
      if (four) return launch_mma_threads<4096, 128, IO>(in, out, tw, batch, inverse, s);
      return launch_mma_threads<4096, 256, IO>(in, out, tw, batch, inverse, s);
    case 8192:
      if (one) return launch_mma_threads<8192, 1024, IO>(in, out, tw, batch, inverse, s);
      return launch_mma_threads<8192, 512, IO>(in, out, tw, batch, inverse, s);
    default: return launch_mma_threads<16384, 1024, IO>(in, out, tw, batch, inverse, s);
  }
}

}  // namespace

bool mma_supported(int64_t n) {
  return n == 512 || n == 1024 || n == 2048 || n == 4096 || n == 8192 || n == 16384;
}

const char* mma_table_variant(int64_t n) {
  switch (n) {
    case 512: return "n512_e16_b2_p4_r16.16.2";
    case 1024: return "n1024_e16_b1_p4_r16.16.4";
    case 2048: return "n2048_e16_b1_p4_r16.16.8";
    case 4096: return "n4096_e16_b1_p4_r16.16.16";
    case 8192: return "n8192_e32_b1_p4_r16.16.16.2";
    case 16384: return "n16384_e16_b1_p4_r16.16.16.4";
    default: return nullptr;
  }
}

hipError_t launch_mma_f16(int64_t n, const void* in, void* out, const void* tw, int64_t batch,
                          bool inverse, hipStream_t s) {
  return launch_mma<IoF16>(n, in, out, tw, batch, inverse, s);
}

hipError_t launch_mma_bf16(int64_t n, const void* in, void* out, const void* tw, int64_t batch,
                           bool inverse, hipStream_t s) {
  return launch_mma<IoBF16>(n, in, out, tw, batch, inverse, s);
}

}  // namespace stockfft
