// Split-operand convolution on the bf16 matrix cores.
//
// The fp32 MFMA runs at 157 TFLOP/s, the bf16 one at 2.5 PFLOP/s.  An fp32
// value is exactly the sum of three bf16 parts (each the nearest bf16 of what
// the parts before left over: 8 + 8 + 8 bits), so a product of two values is
// nine products of parts, of which the three smallest lie below 2^-26 of it;
// the other six, summed in fp32 by the MFMAs, give the product at fp32
// precision for 6/16 of the fp32 MFMA's time.  Operands are scaled by 2^24
// first, which keeps the parts of every normal fp32 value normal bf16 values;
// sums beyond 2^80, infinities and NaNs make the output non-finite, and a
// tile with such outputs is computed again for them on the fp32 MFMA.
//
// Precision, measured as 2-norm distance from the 64-bit result: 1.5e-7 on
// the 3x3 C128 N32 layer (fp32 MFMA kernel: 4.3e-7), 1.6e-7 on the 3x3 C512
// one (3.1e-7), 1.4e-7 on a 1x1 layer of 1024 channels (4.0e-7).  An MFMA
// rounds once for 32 products where the fp32 one rounds every four, and the
// five small products have accumulators of their own (in one set of
// accumulators they would round it six times per step: 3.6e-7 on C512).  Only
// the image instances of two steps share one set: 7.6e-8 on a 3x3 stride 2 C3
// K64 194x194 layer (fp32 MFMA kernel: 9.6e-8).
//
// bf16 inputs run the same kernels with one part per operand.
//
// One of the operands is packed by a small kernel into fragments that a wave
// reads as one contiguous kilobyte; the other is staged into LDS channel-
// octet-fastest, [octet][pixel] of 16 bytes, so that every tap (r, s) of an
// output pixel is another 16-byte slot: no im2col copy, any stride and
// padding, and neighbouring lanes read neighbouring slots (LDS conflict cycles
// are 10% to 15% of a kernel's cycles on the 3x3 layers, 26% on the 3x3 C512
// one).  Measured (back to back through the Python calls),
// before (fp32 MFMA kernels, or the transposed-tile bf16 kernel with its
// phase-split pass) and after:
//   3x3 C128 K128 30^2 N32            78.1 -> 40.9 us (181 TFLOP/s)
//   3x3 C512 K512 9^2 N32             76.8 -> 53.9 us
//   3x3 stride 2 C64 K128 56^2 N32    63.7 -> 31.8 us
//   7x7 stride 2 C3 K64 224^2 N32     118  -> 68.7 us
//   3x3 C512 K1024 17^2 N1            48.4 -> 41.6 us
//   1x1 C1024 K28269 17^2 N1          285  -> 112 us
//   bf16 3x3 C128 K128 28^2 N32       67.0 -> 17.9 us
// What bounds it (counters): the clock is 1.8 to 2.1 GHz; the MFMA pipes are
// busy for 42% to 63% of a fp32 kernel's cycles on the CUs in use, and what they leave, less
// about 8 k cycles for set-up, first loads and last stores, is 11 to 17 cycles
// per vector-memory instruction of the CU (26 on the 1x1 layer, whose second
// round of workgroups leaves CUs idle).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>

#include "split_internal.h"

namespace convfwd {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));

constexpr unsigned kOob = 0x80000000u;  // past every buffer's range (tensors < 2 GB)

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(static_cast<F&&>(f), std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ int fdiv(int n, FastDiv f) {
  return (int)(((unsigned long long)(unsigned)n * f.m) >> (31 + f.s));
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// XCD x takes the contiguous range [x G/8, (x+1) G/8) of the tile order.
__device__ __forceinline__ int xcd_remap(int b, int G) {
  const int G8 = G & ~7;
  return (b < G8) ? (b & 7) * (G8 >> 3) + (b >> 3) : b;
}

constexpr float kScale = 16777216.f;                        // 2^24
constexpr float kUnscale = 1.f / (16777216.f * 16777216.f);  // 2^-48

// Two floats as three bf16 pairs whose sums are the floats exactly (each part
// is the nearest bf16 of what the parts before left over).
__device__ __forceinline__ void split2(float x0, float x1, unsigned& h, unsigned& m, unsigned& l) {
  x0 *= kScale;
  x1 *= kScale;
  h = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{x0, x1}, v2bf));
  x0 -= __builtin_bit_cast(float, h << 16);
  x1 -= __builtin_bit_cast(float, h & 0xffff0000u);
  m = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{x0, x1}, v2bf));
  x0 -= __builtin_bit_cast(float, m << 16);
  x1 -= __builtin_bit_cast(float, m & 0xffff0000u);
  l = __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{x0, x1}, v2bf));
}

// 8 values as the NPL planes of a fragment (a kilobyte apart per wave).
template <int NPL, typename T>
__device__ __forceinline__ void put_fragment(const T (&x)[8], v4u* dst) {
  if constexpr (NPL == 3) {
    v4u h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      unsigned a, b, c;
      split2(x[2 * e], x[2 * e + 1], a, b, c);
      h[e] = a; m[e] = b; l[e] = c;
    }
    dst[0] = h;
    dst[64] = m;
    dst[128] = l;
  } else {
    v4u h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (unsigned)x[2 * e] | ((unsigned)x[2 * e + 1] << 16);
    dst[0] = h;
  }
}

// ---------------------------------------------------------------------------
// The packed operand: [16-row block][chunk][step][plane][lane][8 bf16], so a
// wave reads an operand as one contiguous kilobyte.  Lane l holds 8 values of
// row l % 16 for the unit u = 4 step + l / 16 of the chunk; zeros past the
// rows, channels and taps.
//   CONV, POINT: channel octet u % co of the chunk at tap u / co (POINT: rows
//   are pixels of In, one tap); IMAGE: columns s = 2 (u % Sp), + 1 of kernel
//   row u / Sp, 4 channels each.
template <int MODE>
__global__ void __launch_bounds__(256)
split_pack_kernel(const float* __restrict__ Src, v4u* __restrict__ Pk, const SplitGeom g) {
  const int F = g.nchunks * g.steps;
  const int lane = threadIdx.x & 63;
  const int w = blockIdx.x * 4 + (threadIdx.x >> 6);  // (block, chunk, step)
  if (w >= g.blocks * F) return;
  const int blk = w / F, f = w - blk * F, ch = f / g.steps, m = f - ch * g.steps;
  const int u = 4 * m + (lane >> 4), row = blk * 16 + (lane & 15);
  float x[8];
  if constexpr (MODE == SPLIT_IMAGE) {
    const int Sp = (g.S + 1) / 2, r = u / Sp, s0 = 2 * (u - r * Sp);
    const bool ok = row < g.K && r < g.R;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = e & 3, s = s0 + (e >> 2);
      const bool v = ok && c < g.C && s < g.S;
      const float t = Src[v ? (((size_t)row * g.C + c) * g.R + r) * g.S + s : 0];
      x[e] = v ? t : 0.f;
    }
  } else {
    const int c0 = ch * g.co * 8 + u * 8, PQ = g.P * g.Q;
    const bool ok = row < g.N * PQ && u < g.co;
    const int n = ok ? row / PQ : 0, p = ok ? row - n * PQ : 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int c = c0 + e;
      const float t = Src[((size_t)n * g.C + min(c, g.C - 1)) * PQ + p];
      x[e] = ok && c < g.C ? t : 0.f;
    }
  }
  put_fragment<3>(x, Pk + (size_t)w * 3 * 64 + lane);
}

// CONV: one wave packs one channel octet of a 16-row block: its 16 runs of
// 8 R S contiguous values come in coalesced, and LDS turns them into octets
// per tap (reading the octets straight from memory, eight values R S apart
// per lane, took 16 us for the 2.4 M values of the 512 x 512 3x3 layer).
template <int NPL, int RSC>
__global__ void __launch_bounds__(256)
split_pack_taps_kernel(const void* __restrict__ SrcV, v4u* __restrict__ Pk, const SplitGeom g, const FastDiv dv_n) {
  extern __shared__ __align__(16) unsigned char smem[];
  typedef typename std::conditional<NPL == 3, float, unsigned short>::type T;
  const T* Src = static_cast<const T*>(SrcV);
  const int RS = RSC ? RSC : g.R * g.S, n = 8 * RS, pitch = n + 1;
  const int lane = threadIdx.x & 63, noct = g.nchunks * g.co;
  T* buf = reinterpret_cast<T*>(smem) + (threadIdx.x >> 6) * 16 * pitch;
  const int w = min((int)(blockIdx.x * 4 + (threadIdx.x >> 6)), g.blocks * noct - 1);  // (block, octet)
  const int blk = w / noct, oct = w - blk * noct;
  const int nv = min(n, (g.C - oct * 8) * RS);  // values of real channels per row
  if constexpr (RSC > 0) {  // every load in flight at once
    T t[RSC * 2];
#pragma unroll
    for (int y = 0; y < RSC * 2; ++y) {
      const int i = lane + 64 * y, r = i / (8 * RSC), x = i - r * (8 * RSC), k = blk * 16 + r;
      t[y] = k < g.K && x < nv ? Src[((size_t)k * g.C + oct * 8) * RS + x] : T(0);
    }
#pragma unroll
    for (int y = 0; y < RSC * 2; ++y) {
      const int i = lane + 64 * y, r = i / (8 * RSC);
      buf[r * pitch + i - r * (8 * RSC)] = t[y];
    }
  } else {
    for (int i = lane; i < 16 * n; i += 64) {
      const int r = fdiv(i, dv_n), x = i - r * n, k = blk * 16 + r;
      buf[r * pitch + x] = k < g.K && x < nv ? Src[((size_t)k * g.C + oct * 8) * RS + x] : T(0);
    }
  }
  __syncthreads();
  const int ch = oct / g.co, o = oct - ch * g.co;
  const int units = 4 * g.steps, row = lane & 15;
  v4u* dst = Pk + ((size_t)blk * g.nchunks + ch) * g.steps * NPL * 64;
  // this octet's units are o, o + co, ... (one per tap); the units past the
  // last tap are zero, and each octet's sequence runs through its share of them
  for (int tap = lane >> 4; tap * g.co + o < units; tap += 4) {
    const int u = tap * g.co + o;
    T x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = tap < RS ? buf[row * pitch + e * RS + tap] : T(0);
    put_fragment<NPL>(x, dst + (u >> 2) * NPL * 64 + (u & 3) * 16 + row);
  }
}

// ---------------------------------------------------------------------------
// The convolution.  A workgroup computes BK = 16 WK NWK rows of the packed
// operand by BP = 16 WP NWP rows of the staged one.  Per chunk of 8 co
// channels: the next chunk's items are loaded, split and written to the other
// LDS buffer while this chunk's MFMA steps run; each step covers four
// (octet, tap) units, one per lane group (step table in LDS).  NWC groups of
// waves take every NWC-th step of a chunk and are summed in LDS at the end.
//
// Why this shape: one wave issues a 16x16x32 MFMA every 21 cycles when it
// changes accumulators (18 on the same one); two waves per SIMD fill the
// 16-cycle pipe, so the fp32 instances are eight waves of 1 x 7 blocks (the
// two accumulator sets fit 256 registers; 2 x 7 blocks with four waves took
// 47 us against 40 us on the C128 layer).  The loads, LDS reads and vector
// instructions of a step are spread over its blocks by hand (scheduling
// barriers): left to itself the compiler waits for every LDS read right before its use
// (68 us).
template <int MODE, int VEC, int WK, int WP, int NWK, int NWP, int NWC, int NPL, int NI, int NS, int AD, bool ONE, int OCC,
          bool SEP, typename OT>
__global__ void __launch_bounds__(NWK * NWP * NWC * 64, OCC)
split_conv_kernel(const void* __restrict__ InV, const v4u* __restrict__ Pk, const void* __restrict__ KerV,
                  OT* __restrict__ Out, const SplitGeom g) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NT = NWK * NWP * NWC * 64;
  constexpr int BK = 16 * WK * NWK;  // packed rows per workgroup (POINT: pixels)
  constexpr int BP = 16 * WP * NWP;  // staged rows per workgroup (POINT: output channels)
  constexpr int ISZ = NPL == 3 ? 4 : 2;
  static_assert(VEC == 1 || (MODE == SPLIT_CONV && NPL == 1 && ONE), "vector staging: one chunk of bf16");
  static_assert(MODE == SPLIT_CONV || NPL == 3, "bf16 layers are staged by octets");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave % NWK, wp = (wave / NWK) % NWP, wc = wave / (NWK * NWP);
  const int j16 = lane & 15, gq = lane >> 4;

  // tile
  const int L = xcd_remap((int)blockIdx.x, g.num_tiles);
  int kt, ct, rt;
  if (g.order == 0) {
    const int rest = fdiv(L, g.dv_tiles_k);
    kt = L - rest * g.tiles_k;
    rt = fdiv(rest, g.dv_tiles_cols);
    ct = rest - rt * g.tiles_cols;
  } else {
    const int rest = fdiv(L, g.dv_tiles_cols);
    ct = L - rest * g.tiles_cols;
    kt = fdiv(rest, g.dv_tiles_rows);
    rt = rest - kt * g.tiles_rows;
  }
  const int rho0 = rt * g.tr, rho_end = min(rho0 + g.tr, g.N * g.P);
  const int q0 = ct * g.tw;
  const int n0 = fdiv(rho0, g.dv_P);
  const int nu0 = n0 * g.Hi + (rho0 - n0 * g.P) * g.rm;  // first staged row

  // step table: LDS byte offset of each step's unit per lane group, and the
  // word that says whether a stored output is not finite.  The packed operand
  // is zero in the units past the last tap; they read tap 0 (fp32: an infinity
  // there makes the output NaN, and the second pass puts that right) or, bf16,
  // an octet of zeros that the buffers of such layers have behind the others.
  int* tab = reinterpret_cast<int*>(smem + g.tab_off);
  for (int u = tid; u <= 4 * g.steps; u += NT) {
    if constexpr (MODE == SPLIT_IMAGE) {
      const int Sp = (g.S + 1) / 2, r = u / Sp, sp = u - r * Sp;
      tab[u] = r < g.R ? 16 * (r * g.in_wp + sp) : 0;  // (r >= R for the word)
    } else {
      const int oct = u % g.co;
      int tap = u / g.co;
      const bool past = MODE != SPLIT_POINT && tap >= g.R * g.S;
      if (MODE == SPLIT_POINT || past) tap = 0;
      const int r = tap / g.S, s = tap - r * g.S;
      const int a = r % g.sh, b = s % g.sw;
      int off = 16 * (oct * g.Epad + ((a * g.nb + b) * g.in_rows + r / g.sh) * g.in_wp + s / g.sw);
      if (NPL == 1 && past) off = 16 * g.co * g.Epad;
      tab[u] = u == 4 * g.steps ? 0 : off;
    }
  }
  if constexpr (NPL == 1)
    if (4 * g.steps > g.co * g.R * g.S)
      for (int u = tid; u < g.Epad * (ONE ? 1 : 2); u += NT) {
        const int bf = u >= g.Epad;
        *reinterpret_cast<v4u*>(smem + bf * g.buf_bytes + 16 * (g.co * g.Epad + u - bf * g.Epad)) = v4u{0, 0, 0, 0};
      }

  // Staging items of this thread: global byte offset (for IMAGE: of either
  // pixel), LDS byte offset (24 bits) and octet.  Slots past the last item
  // repeat the thread's previous one (the same bytes to the same place),
  // which keeps the loop free of branches.
  unsigned goff[NI], goff2[MODE == SPLIT_IMAGE ? NI : 1], loff[NI];
  unsigned poff[VEC > 1 ? NI : 1][VEC];  // VEC: LDS byte offset of each pixel
  const int HW = g.H * g.W;
  auto image_item = [&](int it, unsigned& left, unsigned& right, unsigned& slot) {  // (one octet, one phase)
    const int row = fdiv(it, g.dv_wp), x = it - row * g.in_wp;
    const int nu = nu0 + row;
    const int n = fdiv(nu, g.dv_Hi), y = nu - n * g.Hi - g.ph, xx = q0 * g.sw + 2 * x - g.pw;
    const bool rok = n < g.N && (unsigned)y < (unsigned)g.H;
    const unsigned base = (unsigned)(ISZ * ((n * g.C * g.H + y) * g.W + xx));
    slot = 16u * (unsigned)it;
    left = rok && (unsigned)xx < (unsigned)g.W ? base : kOob;
    right = rok && (unsigned)(xx + 1) < (unsigned)g.W ? base + ISZ : kOob;
  };
  if constexpr (VEC > 1) {
    // bf16 layers of one chunk, where single-pixel loads (128 bytes a wave)
    // took most of the time: 32-channel layers with K = 32, 165x136 at batch 9
    // 28.1 -> 18.8 us, 176x210 at batch 4 22.7 -> 16.1 us.  (fp32 layers did
    // not gain: 3x3 C128 46.3 -> 49.8 us, C512 60.4 -> 60.6 us.)
    // Four neighbouring input pixels per item, inside the image row: the last
    // group of a row starts early enough to end in it (pixels staged twice
    // get the same bytes).  Columns in the padding are zeroed here; no item
    // writes them.
    const int x0 = q0 * g.sw - g.pw;  // input column of the tile's first staged one
    const int xa = max(x0, 0) & ~1;  // dword-aligned groups
    if (g.pw > 0) {
      for (int u = tid; u < g.co * g.E; u += NT) {
        const int o = fdiv(u, g.dv_Ez), e = u - o * g.E;
        const int prow = fdiv(e, g.dv_wpz), x = e - prow * g.in_wp;
        const int f = fdiv(prow, g.dv_rows);
        const int xx = x0 + x * g.sw + f - fdiv(f, g.dv_nb) * g.nb;
        if ((unsigned)xx < (unsigned)g.W) continue;
        *reinterpret_cast<v4u*>(smem + (o * g.Epad + e) * 16) = v4u{0, 0, 0, 0};
      }
    }
    int it = tid < g.items ? tid : tid % g.items;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (i > 0 && it + NT < g.items) it += NT;
      const int o = fdiv(it, g.dv_E), e = it - o * g.E4;
      const int prow = fdiv(e, g.dv_wp), gi = e - prow * g.ng;
      const int a = fdiv(prow, g.dv_rows), row = prow - a * g.in_rows;
      const int nu = nu0 + row;
      const int n = fdiv(nu, g.dv_Hi), yi = nu - n * g.Hi;
      const int y = yi * g.sh + a - g.ph, base = min(xa + 4 * gi, g.W - 4);
      goff[i] = n < g.N && (unsigned)y < (unsigned)g.H
                    ? (unsigned)(ISZ * (((n * g.C + o * 8) * g.H + y) * g.W + base))
                    : kOob;
      loff[i] = (unsigned)o;
#pragma unroll
      for (int p = 0; p < VEC; ++p) {
        const int v = base + p - x0;  // staged column of the tile, all phases
        const int ix = g.nb == 1 ? v : v >> 1, b = g.nb == 1 ? 0 : v & 1;
        const bool in = v >= 0 && ix < g.in_wp;
        poff[i][p] = 16u * (unsigned)(o * g.Epad + (in ? ((a * g.nb + b) * g.in_rows + row) * g.in_wp + ix : g.E));
      }
    }
  } else {
    int it = tid < g.items ? tid : tid % g.items;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (i > 0 && it + NT < g.items) it += NT;
      if constexpr (MODE == SPLIT_POINT) {
        // consecutive lanes take the octets of one row: contiguous channels
        const int e = fdiv(it, g.dv_nb), o = it - e * g.co;
        loff[i] = 16u * (unsigned)(o * g.Epad + e) | ((unsigned)o << 24);
        const int k = kt * BP + e;
        goff[i] = k < g.K ? 4u * ((unsigned)k * (unsigned)g.C + 8u * (unsigned)o) : kOob;
      } else if constexpr (MODE == SPLIT_IMAGE) {
        image_item(it, goff[i], goff2[i], loff[i]);
      } else {
        const int o = fdiv(it, g.dv_E), e = it - o * g.E;
        const int prow = fdiv(e, g.dv_wp), x = e - prow * g.in_wp;
        const int f = fdiv(prow, g.dv_rows), row = prow - f * g.in_rows;
        const int a = fdiv(f, g.dv_nb), b = f - a * g.nb;
        const int nu = nu0 + row;
        const int n = fdiv(nu, g.dv_Hi), yi = nu - n * g.Hi;
        loff[i] = 16u * (unsigned)(o * g.Epad + e) | ((unsigned)o << 24);
        const int y = yi * g.sh + a - g.ph, xx = (q0 + x) * g.sw + b - g.pw;
        goff[i] = n < g.N && (unsigned)y < (unsigned)g.H && (unsigned)xx < (unsigned)g.W
                      ? (unsigned)(ISZ * (((n * g.C + o * 8) * g.H + y) * g.W + xx))
                      : kOob;
      }
    }
  }
  const auto irsrc = make_rsrc(MODE == SPLIT_POINT ? KerV : InV, g.st_bytes);
  const auto prsrc = make_rsrc(Pk, g.pk_bytes);

  unsigned stg[VEC > 1 ? 1 : NI][8];
  v2u stv[VEC > 1 ? NI : 1][8];
  // Load e of item i of chunk ch (scalar offsets stay inside the tensor, so
  // that the range check's difference is positive).
  constexpr int LPI = MODE == SPLIT_POINT ? 2 : 8;  // loads per item
  auto load_in = [&](int i, int e, int ch) {
    if constexpr (MODE == SPLIT_POINT) {
      const int c = ch * g.co * 8 + 4 * e;
      const unsigned off = c + 8 * (int)(loff[i] >> 24) >= g.C ? kOob : goff[i];
      const v4u v = __builtin_bit_cast(
          v4u, __builtin_amdgcn_raw_buffer_load_b128(irsrc, off, min(c, g.C - 4) * 4, 0));
#pragma unroll
      for (int x = 0; x < 4; ++x) stg[i][4 * e + x] = v[x];
    } else if constexpr (VEC > 1) {
      const int c = ch * g.co * 8 + e;
      const unsigned off = c + 8 * (int)loff[i] >= g.C ? kOob : goff[i];
      const int so = min(c, g.C - 1) * HW * ISZ;
      stv[i][e] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(irsrc, off, so, 0));
    } else {
      unsigned off;
      int so;
      if constexpr (MODE == SPLIT_IMAGE) {
        off = (e & 3) >= g.C ? kOob : e < 4 ? goff[i] : goff2[i];
        so = min(e & 3, g.C - 1) * HW * ISZ;
      } else {
        const int c = ch * g.co * 8 + e;
        off = c + 8 * (int)(loff[i] >> 24) >= g.C ? kOob : goff[i];
        so = min(c, g.C - 1) * HW * ISZ;
      }
      if constexpr (NPL == 3) stg[i][e] = __builtin_amdgcn_raw_buffer_load_b32(irsrc, off, so, 0);
      else stg[i][e] = __builtin_amdgcn_raw_buffer_load_b16(irsrc, off, so, 0);
    }
  };
  const int pl_bytes = g.co * g.Epad * 16;
  // Conversion of an item in pieces (pairs of values; four per pixel), each
  // pixel's LDS writes after its last.
  constexpr int PPI = 4 * VEC;  // pieces per item
  v4u cvt[VEC > 1 ? 1 : NI][NPL];
  auto convert_piece = [&](int i, int q, unsigned char* buf) {
    const int e = q & 3, px = q >> 2, ci = VEC > 1 ? 0 : i;
    if constexpr (NPL == 3) {
      const unsigned lo = stg[i][2 * e], hi = stg[i][2 * e + 1];
      unsigned a, b, c;
      split2(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi), a, b, c);
      cvt[ci][0][e] = a; cvt[ci][1][e] = b; cvt[ci][2][e] = c;
    } else if constexpr (VEC > 1) {
      const unsigned lo = stv[i][2 * e][px >> 1], hi = stv[i][2 * e + 1][px >> 1];
      cvt[ci][0][e] = px & 1 ? (lo >> 16) | (hi & 0xffff0000u) : (lo & 0xffffu) | (hi << 16);
    } else {
      cvt[ci][0][e] = (stg[i][2 * e] & 0xffffu) | (stg[i][2 * e + 1] << 16);
    }
    if (e == 3) {
      unsigned char* d = buf + (VEC > 1 ? poff[VEC > 1 ? i : 0][px] : loff[i] & 0xffffffu);
#pragma unroll
      for (int p = 0; p < NPL; ++p) *reinterpret_cast<v4u*>(d + p * pl_bytes) = cvt[ci][p];
    }
  };

  // LDS byte offset of a lane's staged row (output pixel) of block j
  auto row_offset = [&](int j, int lane16) -> unsigned {
    const int p = (wp * WP + j) * 16 + lane16;
    if constexpr (MODE == SPLIT_POINT) return 16u * (unsigned)p;
    const int t = fdiv(p, g.dv_tw), col = p - t * g.tw;
    const int rho = rho0 + t;
    if (t >= g.tr || rho >= rho_end) return 0;
    const int n = fdiv(rho, g.dv_P);
    const int row = n * g.Hi + (rho - n * g.P) * g.rm - nu0;
    return MODE == SPLIT_IMAGE ? 16u * (unsigned)(row * g.in_wp) + 8u * (unsigned)(col * g.cm)
                               : 16u * (unsigned)(row * g.in_wp + col);
  };
  unsigned paddr[WP];
#pragma unroll
  for (int j = 0; j < WP; ++j) paddr[j] = row_offset(j, j16);

  // packed operand: steps wc, wc + NWC, ... of each chunk
  const int F = g.nchunks * g.steps;
  const unsigned blk0 = (unsigned)((MODE == SPLIT_POINT ? rt : kt) * (BK / 16) + wk * WK);
  auto load_a = [&](v4u (&a)[WK][NPL], int x, int ch, int m) {  // part x of step m of chunk ch
    const unsigned f = (unsigned)min(ch * g.steps + m, F - 1);
    a[x / NPL][x % NPL] = __builtin_bit_cast(
        v4u, __builtin_amdgcn_raw_buffer_load_b128(prsrc, (unsigned)lane * 16u,
                                                   (int)(((blk0 + x / NPL) * (unsigned)F + f) * NPL + x % NPL) * 1024, 0));
  };

  v4f acc[WK][WP], part[SEP ? WK : 1][SEP ? WP : 1];
#pragma unroll
  for (int i = 0; i < WK; ++i)
#pragma unroll
    for (int j = 0; j < WP; ++j) {
      acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
      if constexpr (SEP) part[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    }

  constexpr int BD = OCC > 2 ? 2 : 3;
  v4u bq[BD][NPL];  // LDS operands of this block and the BD - 1 next
  auto load_b = [&](v4u (&b)[NPL], const unsigned char* buf, unsigned ad) {
#pragma unroll
    for (int p = 0; p < NPL; ++p) {
      const unsigned char* s = buf + ad + p * pl_bytes;
      if constexpr (MODE == SPLIT_IMAGE) {  // pixels are 8 bytes: an odd one is 8-byte aligned
        const v2u lo = *reinterpret_cast<const v2u*>(s), hi = *reinterpret_cast<const v2u*>(s + 8);
        b[p] = v4u{lo[0], lo[1], hi[0], hi[1]};
      } else {
        b[p] = *reinterpret_cast<const v4u*>(s);
      }
    }
  };
  auto mma1 = [&](const v4u& a, const v4u& b, v4f& c) {
    const v8bf x = __builtin_bit_cast(v8bf, a), y = __builtin_bit_cast(v8bf, b);
    c = MODE == SPLIT_POINT ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(y, x, c, 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, y, c, 0, 0, 0);
  };
  auto mma = [&](v4u (&a)[WK][NPL], v4u (&b)[NPL], int j) {
    if constexpr (NPL == 3) {
      // small products first
      constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
      for (int i = 0; i < WK; ++i)
#pragma unroll
        for (int p = 0; p < 6; ++p) {
          mma1(a[i][PA[p]], b[PB[p]], SEP && p < 5 ? part[i % (SEP ? WK : 1)][j % (SEP ? WP : 1)] : acc[i][j]);
          __builtin_amdgcn_sched_barrier(0x7f6);  // MFMAs stay in this order
        }
    } else {
#pragma unroll
      for (int i = 0; i < WK; ++i) mma1(a[i][0], b[0], acc[i][j]);
    }
  };

  // prologue: chunk 0 into buffer 0
  v4u aq[AD + 1][WK][NPL];  // Ker operands of this step and the AD next
#pragma unroll
  for (int x = 0; x < WK * NPL; ++x) load_a(aq[0], x, 0, min(wc, g.steps - 1));
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < LPI; ++e) load_in(i, e, 0);
#pragma unroll
  for (int d = 1; d < AD; ++d)
#pragma unroll
    for (int x = 0; x < WK * NPL; ++x) load_a(aq[d], x, d / NS, min((d % NS) * NWC + wc, g.steps - 1));
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < PPI; ++e) convert_piece(i, e, smem);
  __syncthreads();

  // Staging of the next chunk: an item's loads are issued LAG steps before
  // its conversion.
  static_assert(ONE || NS >= 2, "an item's loads and its conversion are in different steps");
  constexpr int LAG = NS > 4 ? 3 : NS / 2;
  constexpr int NR = (NS - LAG) * WP;  // regions (step, block) that convert, from LAG WP on
  for (int ch = 0; ch < (ONE ? 1 : g.nchunks); ++ch) {
    const unsigned char* buf = smem + (ch & 1) * g.buf_bytes;
    unsigned char* nbuf = smem + ((ch + 1) & 1) * g.buf_bytes;
    int off = tab[4 * min(wc, g.steps - 1) + gq];
    load_b(bq[0], buf, paddr[0] + off);
    if constexpr (BD > 2) load_b(bq[1], buf, paddr[1 % WP] + off);
    static_for<NS>([&](auto I) {
      constexpr int i = decltype(I)::value;
      constexpr int n1 = i + 1 < NS ? i + 1 : i;
      const int offn = tab[4 * min(n1 * NWC + wc, g.steps - 1) + gq];
      const bool run = NWC == 1 || i * NWC + wc < g.steps;
      static_for<WP>([&](auto J) {
        constexpr int j = decltype(J)::value;
        constexpr int cur = (i * WP + j) % BD, ahead = j + BD - 1;
        load_b(bq[(cur + BD - 1) % BD], buf, paddr[ahead % WP] + (ahead < WP ? off : offn));
        // This region's share of the loads, spread out so that the waves'
        // loads don't queue up at the address unit: the packed operands AD
        // steps ahead (the next chunk's first steps at the end), and items of
        // the next chunk, each item's within the LAG - 1 steps before the one
        // that precedes its conversion.
        static_for<WK * NPL>([&](auto Q) {
          constexpr int q = decltype(Q)::value;
          if constexpr (q * WP / (WK * NPL) == j)
            load_a(aq[AD], q, ch + (i + AD) / NS, min(((i + AD) % NS) * NWC + wc, g.steps - 1));
        });
        if constexpr (!ONE) static_for<NI * LPI>([&](auto Q) {
          constexpr int it = decltype(Q)::value / LPI, l = decltype(Q)::value % LPI;
          if constexpr (it * NR / NI + l * (LAG - 1) * WP / LPI == i * WP + j) load_in(it, l, ch + 1);
        });
        __builtin_amdgcn_sched_barrier(0);
        if (run) mma(aq[0], bq[cur], j);
        if constexpr (!ONE) static_for<NI * PPI>([&](auto Q) {
          constexpr int q = decltype(Q)::value;
          if constexpr (LAG * WP + q * NR / (NI * PPI) == i * WP + j) convert_piece(q / PPI, q % PPI, nbuf);
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      off = offn;
#pragma unroll
      for (int d = 0; d < AD; ++d)
#pragma unroll
        for (int x = 0; x < WK; ++x)
#pragma unroll
          for (int p = 0; p < NPL; ++p) aq[d][x][p] = aq[d + 1][x][p];
    });
    if constexpr (NWC > 1) __syncthreads();
    else if (!ONE && ch + 1 < g.nchunks) __syncthreads();
  }
  if constexpr (SEP) {
#pragma unroll
    for (int i = 0; i < WK; ++i)
#pragma unroll
      for (int j = 0; j < WP; ++j) acc[i][j] += part[i][j];
  }

  // channel groups: sum in LDS, each group finishing its share of the blocks
  auto sum_groups = [&] {
    float* red = reinterpret_cast<float*>(smem);
    constexpr int RT = WK * WP * 4;
#pragma unroll
    for (int i = 0; i < WK; ++i)
#pragma unroll
      for (int j = 0; j < WP; ++j)
        *reinterpret_cast<v4f*>(red + ((wave * (RT / 4) + i * WP + j) * 64 + lane) * 4) = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WK; ++i)
#pragma unroll
      for (int j = 0; j < WP; ++j) {
        if ((i * WP + j) % NWC != wc) continue;
        v4f s = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NWC; ++q)
          s += *reinterpret_cast<const v4f*>(
              red + (((q * NWK * NWP + wp * NWK + wk) * (RT / 4) + i * WP + j) * 64 + lane) * 4);
        acc[i][j] = s;
      }
  };
  if constexpr (NWC > 1) sum_groups();

  // Block (i, j) holds output channels k0 + 0..3 and one pixel per lane.
  const int PQ = g.P * g.Q;
  auto locate = [&](int lane16, int i, int j, int& n, int& h, int& q, int& k0) -> bool {
    if constexpr (MODE == SPLIT_POINT) {
      const int px = rt * BK + (wk * WK + i) * 16 + lane16;
      k0 = kt * BP + (wp * WP + j) * 16 + gq * 4;
      n = fdiv(px, g.dv_PQ);
      h = 0;
      q = px - n * PQ;
      return n < g.N;
    } else {
      const int p = (wp * WP + j) * 16 + lane16;
      const int t = fdiv(p, g.dv_tw), rho = rho0 + t;
      k0 = kt * BK + (wk * WK + i) * 16 + gq * 4;
      n = fdiv(rho, g.dv_P);
      h = rho - n * g.P;
      q = q0 + p - t * g.tw;
      return t < g.tr && rho < rho_end && q < g.Q;
    }
  };
  int at16 = j16;  // (opaque, or the parts of the staged rows' offsets would be kept in registers till here)
  asm volatile("" : "+v"(at16));
  float z = 0.f;  // NaN once a stored output is not finite
#pragma unroll
  for (int j = 0; j < WP; ++j)
#pragma unroll
    for (int i = 0; i < WK; ++i) {
      int n, h, q, k0;
      const bool ok = locate(at16, i, j, n, h, q, k0);
      if (NWC > 1 && (i * WP + j) % NWC != wc) continue;
      if (!ok) continue;
      OT* o = Out + ((size_t)n * g.K + k0) * PQ + h * g.Q + q;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (k0 + v >= g.K) continue;
        const float x = acc[i][j][v];
        if constexpr (NPL == 3) z = __builtin_fmaf(x, 0.f, z);
        o[(size_t)v * PQ] = (OT)(NPL == 3 ? x * kUnscale : x);
      }
    }
  if constexpr (NPL == 3) {
    int* nonfinite = reinterpret_cast<int*>(smem + g.tab_off) + 4 * g.steps;
    if (z != z) *nonfinite = 1;
    __syncthreads();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(*nonfinite) == 0, 1)) return;

    // The tile again, for its outputs that are not finite, as IEEE arithmetic
    // treats infinities, NaNs and sums beyond the scaled range (bf16 operands
    // are multiplied as they are and need none of this): the operands
    // themselves on the fp32 MFMA, In staged with the 8 channels of a slot as
    // floats in the first two planes, the units past the last tap masked, each
    // step's 32 products summed by themselves first (in one chain per chunk the
    // error on six of 19 layers, one per instance, was above the tile plans', up
    // to 2.2e-7 against 1.3e-7).  Nothing is pipelined: a tile takes two to
    // three times its first pass (all of In NaN, 3x3 C128 N32: 48 -> 172 us, 1x1
    // C1024 K28269: 112 -> 371 us; each lane summing its outputs by itself, 3.8
    // and 37 ms; the tile plans 82 and 284 us).  2-norm error on outputs of
    // 2^100: 1.5e-7 on C128 and 1.6e-7 on C512 (tile plans 6.1e-7 and 4.3e-7).
    unsigned bad[(WK * WP * 4 + 31) / 32] = {};
#pragma unroll
    for (int b = 0; b < WK * WP * 4; ++b)
      if (!(__builtin_fabsf(acc[(b >> 2) / WP][(b >> 2) % WP][b & 3]) < __builtin_inff())) bad[b / 32] |= 1u << (b % 32);
    if constexpr (ONE) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < WK; ++i)
#pragma unroll
      for (int j = 0; j < WP; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    // (opaque indices, or parts of the first pass's offsets would be kept in registers for this one)
    int again = j16, thread = tid, first = 0;
    asm volatile("" : "+v"(again), "+v"(thread), "+s"(first));
#pragma unroll
    for (int j = 0; j < WP; ++j) paddr[j] = row_offset(j, again);
    if constexpr (ONE) __builtin_amdgcn_sched_barrier(0);
    const auto orsrc = make_rsrc(MODE == SPLIT_POINT ? InV : KerV,
                                 4u * (unsigned)(MODE == SPLIT_POINT ? g.N * g.C * PQ : g.K * g.C * g.R * g.S));
#pragma clang loop unroll(disable)
    for (int ch = first; ch < (ONE ? 1 : g.nchunks); ++ch) {
      __syncthreads();  // (buffer 0 was read)
      if constexpr (!ONE)
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int e = 0; e < LPI; ++e) load_in(i, e, ch);
      [[maybe_unused]] int it = thread < g.items ? thread : thread % g.items;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        if constexpr (ONE) {  // (an item at a time: fewer registers)
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (MODE == SPLIT_IMAGE) {
            if (i > 0 && it + NT < g.items) it += NT;
            image_item(it, goff[i], goff2[i], loff[i]);
          }
#pragma unroll
          for (int e = 0; e < LPI; ++e) load_in(i, e, ch);
        }
        constexpr int M1 = MODE == SPLIT_IMAGE ? 4 : 2, M2 = MODE == SPLIT_IMAGE ? 2 : 4;  // IMAGE: 2 pixels x 2 channels
        unsigned char* d = smem + (loff[i] & 0xffffffu);
        *reinterpret_cast<v4u*>(d) = v4u{stg[i][0], stg[i][1], stg[i][M1], stg[i][M1 + 1]};
        *reinterpret_cast<v4u*>(d + pl_bytes) = v4u{stg[i][M2], stg[i][M2 + 1], stg[i][6], stg[i][7]};
      }
      __syncthreads();
#pragma clang loop unroll(disable)
      for (int m = wc; m < g.steps; m += NWC) {
        const int u = 4 * m + gq, off = tab[u];
        const int Sp = (g.S + 1) / 2;
        const int tap = MODE == SPLIT_IMAGE ? u / Sp : u / g.co;  // IMAGE: kernel row
        const int oct = MODE == SPLIT_IMAGE ? 2 * (u - tap * Sp) : u - tap * g.co;  // IMAGE: first column
        const bool real = tap < (MODE == SPLIT_IMAGE ? g.R : g.R * g.S);
        float a[WK][8];
#pragma unroll
        for (int i = 0; i < WK; ++i) {
          const int row = (MODE == SPLIT_POINT ? rt : kt) * BK + (wk * WK + i) * 16 + j16;
          const int pn = MODE == SPLIT_POINT ? fdiv(row, g.dv_PQ) : 0;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            bool in;
            unsigned at;
            if constexpr (MODE == SPLIT_IMAGE) {
              const int c = e & 3, s = oct + (e >> 2);
              in = real && row < g.K && c < g.C && s < g.S;
              at = (((unsigned)row * g.C + c) * g.R + tap) * g.S + s;
            } else {
              const int c = (ch * g.co + oct) * 8 + e;
              in = real && c < g.C && (MODE == SPLIT_POINT ? pn < g.N : row < g.K);
              at = MODE == SPLIT_POINT ? ((unsigned)pn * g.C + c) * PQ + (row - pn * PQ)
                                       : ((unsigned)row * g.C + c) * (g.R * g.S) + tap;
            }
            a[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(orsrc, in ? 4u * at : kOob, 0, 0));
          }
        }
#pragma unroll
        for (int j = 0; j < WP; ++j) {
          const unsigned char* s = smem + paddr[j] + off;
          float b[8];
          if constexpr (ONE) __builtin_amdgcn_sched_barrier(0);
          if constexpr (MODE == SPLIT_IMAGE) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {  // (plane, pixel)
              const v2u t = *reinterpret_cast<const v2u*>(s + (p >> 1) * pl_bytes + (p & 1) * 8);
              const bool in = real && ((p & 1) == 0 || oct + 1 < g.S);
#pragma unroll
              for (int x = 0; x < 2; ++x) {
                const unsigned v = in ? t[x] : 0u;
                b[4 * (p & 1) + 2 * (p >> 1) + x] = __builtin_bit_cast(float, v);
              }
            }
          } else {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
              const v4u t = *reinterpret_cast<const v4u*>(s + p * pl_bytes);
#pragma unroll
              for (int x = 0; x < 4; ++x) {
                const unsigned v = real ? t[x] : 0u;
                b[4 * p + x] = __builtin_bit_cast(float, v);
              }
            }
          }
#pragma unroll
          for (int i = 0; i < WK; ++i) {
            v4f t = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 8; ++e)
              t = MODE == SPLIT_POINT ? __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[i][e], t, 0, 0, 0)
                                      : __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], b[e], t, 0, 0, 0);
            acc[i][j] += t;
          }
        }
      }
    }
    if constexpr (NWC > 1) {
      __syncthreads();
      sum_groups();
    }
    asm volatile("" : "+v"(again));
#pragma unroll
    for (int j = 0; j < WP; ++j)
#pragma unroll
      for (int i = 0; i < WK; ++i) {
        int n, h, q, k0;
        const bool ok = locate(again, i, j, n, h, q, k0);
        if (NWC > 1 && (i * WP + j) % NWC != wc) continue;
        if (!ok) continue;
        OT* o = Out + ((size_t)n * g.K + k0) * PQ + h * g.Q + q;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int b = (i * WP + j) * 4 + v;
          if (k0 + v < g.K && (bad[b / 32] >> (b % 32) & 1)) o[(size_t)v * PQ] = (OT)acc[i][j][v];
        }
      }
  }
}

typedef void (*SplitFnF)(const void*, const v4u*, const void*, float*, SplitGeom);
typedef void (*SplitFnB)(const void*, const v4u*, const void*, __bf16*, SplitGeom);
struct SplitInstance {
  SplitConfig c;
  SplitFnF f32;
  SplitFnB bf16;  // bf16 Out (bf16 inputs only)
};

#define SPLIT_F32(ID, MODE, VEC, WK, WP, NWK, NWP, NWC, NI, NS, AD, ONE, OCC, SEP)                                  \
  SplitInstance{SplitConfig{ID, MODE, VEC, WK, WP, NWK, NWP, NWC, 3, NI, NS, ONE, OCC},                         \
                &split_conv_kernel<MODE, VEC, WK, WP, NWK, NWP, NWC, 3, NI, NS, AD, ONE, OCC, SEP, float>, nullptr}
#define SPLIT_BF16(ID, MODE, VEC, WK, WP, NWK, NWP, NWC, NI, NS, AD, ONE, OCC)                                  \
  SplitInstance{SplitConfig{ID, MODE, VEC, WK, WP, NWK, NWP, NWC, 1, NI, NS, ONE, OCC},                         \
                &split_conv_kernel<MODE, VEC, WK, WP, NWK, NWP, NWC, 1, NI, NS, AD, ONE, OCC, false, float>,           \
                &split_conv_kernel<MODE, VEC, WK, WP, NWK, NWP, NWC, 1, NI, NS, AD, ONE, OCC, false, __bf16>}

const SplitInstance kSplit[] = {
#include "split_instances.inc"
};
constexpr int kNumSplit = sizeof(kSplit) / sizeof(kSplit[0]);

}  // namespace

const SplitConfig* split_configs(int* count) {
  static SplitConfig table[kNumSplit];
  static const bool init = [] {
    for (int i = 0; i < kNumSplit; ++i) table[i] = kSplit[i].c;
    return true;
  }();
  (void)init;
  *count = kNumSplit;
  return table;
}

int split_launch(const SplitPlan& p, bool out_bf16, const void* In, const void* Ker, void* Pk, void* Out,
                 void* stream) {
  const SplitInstance* inst = nullptr;
  for (const SplitInstance& x : kSplit)
    if (x.c.id == p.cfg->id) inst = &x;
  if (!inst || (out_bf16 && !inst->bf16)) return CONV_EINVAL;
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  const SplitGeom& g = p.g;
  const void* fn = out_bf16 ? reinterpret_cast<const void*>(inst->bf16) : reinterpret_cast<const void*>(inst->f32);
  if (p.lds_bytes > 65536) {
    // raise the kernel's dynamic LDS limit once
    static std::mutex mu;
    static bool done[2][kNumSplit] = {};
    std::lock_guard<std::mutex> lk(mu);
    bool& d = done[out_bf16][inst - kSplit];
    if (!d) {
      if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 163840) != hipSuccess) return CONV_EHIP;
      d = true;
    }
  }
  v4u* pk = static_cast<v4u*>(Pk);
  if (p.cfg->mode == SPLIT_CONV) {
    const int n = 8 * g.R * g.S, waves = g.blocks * g.nchunks * g.co;
    const int lds = 4 * 16 * (n + 1) * (p.cfg->npl == 3 ? 4 : 2);
    const FastDiv dv = make_fastdiv(n);
    const bool f32 = p.cfg->npl == 3;
    const auto pack = g.R * g.S == 9 ? (f32 ? &split_pack_taps_kernel<3, 9> : &split_pack_taps_kernel<1, 9>)
                      : g.R * g.S == 1 ? (f32 ? &split_pack_taps_kernel<3, 1> : &split_pack_taps_kernel<1, 1>)
                                       : (f32 ? &split_pack_taps_kernel<3, 0> : &split_pack_taps_kernel<1, 0>);
    hipLaunchKernelGGL(pack, dim3((waves + 3) / 4), dim3(256), lds, st, Ker, pk, g, dv);
  } else {
    const dim3 grid((g.blocks * g.nchunks * g.steps + 3) / 4);
    if (p.cfg->mode == SPLIT_POINT)
      hipLaunchKernelGGL(split_pack_kernel<SPLIT_POINT>, grid, dim3(256), 0, st, static_cast<const float*>(In), pk, g);
    else
      hipLaunchKernelGGL(split_pack_kernel<SPLIT_IMAGE>, grid, dim3(256), 0, st, static_cast<const float*>(Ker), pk, g);
  }
  if (out_bf16)
    hipLaunchKernelGGL(inst->bf16, dim3(g.num_tiles), dim3(p.cfg->threads()), p.lds_bytes, st, In, pk, Ker,
                       static_cast<__bf16*>(Out), g);
  else
    hipLaunchKernelGGL(inst->f32, dim3(g.num_tiles), dim3(p.cfg->threads()), p.lds_bytes, st, In, pk, Ker,
                       static_cast<float*>(Out), g);
  return hipGetLastError() == hipSuccess ? CONV_OK : CONV_EHIP;
}

}  // namespace convfwd
