// Wave-level MFMA tile products shared by the pair kernels and the node mixing kernel.
#pragma once

#include <hip/hip_runtime.h>

namespace tn {

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// mfma4 with the activation fragment a and the weight fragment b; with TR the weights are the
// instruction's first operand, so the accumulator holds the product transposed: entry t of
// acc[rb][cb] in lane l is D_rb[l%16][col0 + cb*16 + 4(l/16) + t], four consecutive columns of one
// row, which a row-major store or load moves in one vector access.
template <bool TR>
__device__ __forceinline__ floatx4 mfma4_ab(float a, float b, floatx4 c) {
  return TR ? mfma4(b, a, c) : mfma4(a, b, c);
}

// BF16 operands, FP32 accumulation (v_mfma_f32_16x16x32_bf16): lane l holds
// A[l%16][8(l/16)..8(l/16)+7] and B[8(l/16)..+7][l%16]; the result layout is that of mfma4.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
constexpr int kPadB = 8;   // LDS row padding of BF16 operand tiles (elements)

__device__ __forceinline__ floatx4 mfma_bf16(const bf16x8 &a, const bf16x8 &b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// Four consecutive values (16-byte aligned FP32, 8-byte aligned BF16) as one vector access.
__device__ __forceinline__ floatx4 ld4(const float *p) { return *reinterpret_cast<const floatx4 *>(p); }
__device__ __forceinline__ floatx4 ld4(const __bf16 *p) {
  const bf16x4 v = *reinterpret_cast<const bf16x4 *>(p);
  return floatx4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ __forceinline__ void st4(float *p, const floatx4 &v) { *reinterpret_cast<floatx4 *>(p) = v; }
__device__ __forceinline__ void st4(__bf16 *p, const floatx4 &v) {
  bf16x4 o;
#pragma unroll
  for (int t = 0; t < 4; ++t) o[t] = (__bf16)v[t];
  *reinterpret_cast<bf16x4 *>(p) = o;
}

// FP32 products on the BF16 matrix instructions.  An FP32 number x is the sum of three BF16 numbers of its
// sign and exponent range: h = bf16(x), m = bf16(x - h) and l = x - h - m, all rounded to nearest.
// Both differences are exact, and l has the bits that are left of the 24 (|m| <= 2^-8 |x|, |l| <=
// 2^-17 |x|), so h + m + l is x itself, with no scale to choose and whatever other entries its
// matrix or row has (for |x| >= 2^-110; below, l ends at BF16's smallest number, 2^-133; and up to the
// largest BF16 number, 2^128 - 2^120: h of the last FP32 numbers above it may be infinite).  A product
// is the six largest of the nine BF16 products with FP32 accumulation; the three left out (m l, l m,
// l l) are at most 2^-24 of it together, of either sign, and 2^-27.4 in RMS.  Six
// v_mfma_f32_16x16x32_bf16 do the work of eight v_mfma_f32_16x16x4_f32 in 96 matrix cycles instead
// of 256.  Two parts are not enough: of FP16's 11 bits each they hold 23, and a rounding of a weight is the
// same in every pair and atom.
constexpr int kPadH = 8;   // LDS row padding of split operand tiles (elements)

// V values (1, 2 or 4) as their three parts, each as one store at p, p + plane and p + 2 plane.  The
// remainders are those of the rounded x: a product that ends in x may not be fused into them.
template <int V>
__device__ __forceinline__ void st_split(__bf16 *p, int plane, const float (&x)[V]) {
#pragma clang fp contract(off)
  typedef __bf16 part __attribute__((ext_vector_type(V)));
  float r[V];
#pragma unroll
  for (int t = 0; t < V; ++t) r[t] = x[t];
#pragma unroll
  for (int n = 0; n < 3; ++n) {
    part o;
#pragma unroll
    for (int t = 0; t < V; ++t) {
      o[t] = (__bf16)r[t];
      r[t] -= (float)o[t];
    }
    *reinterpret_cast<part *>(p + n * plane) = o;
  }
}
__device__ __forceinline__ void st4_split(__bf16 *p, int plane, const floatx4 &v) {
  const float x[4] = {v[0], v[1], v[2], v[3]};
  st_split<4>(p, plane, x);
}

// One fragment's three parts.
struct Frag3 {
  bf16x8 h, m, l;
};
__device__ __forceinline__ Frag3 ld_frag3(const __bf16 *p, int plane) {
  return Frag3{*reinterpret_cast<const bf16x8 *>(p), *reinterpret_cast<const bf16x8 *>(p + plane),
               *reinterpret_cast<const bf16x8 *>(p + 2 * plane)};
}

// t[n] += W(n) A(n) over one chunk of 32 along K: the six products, smallest first.  The N chains are
// independent; each instruction of a chain waits for the one before.
template <int N, class FW, class FA>
__device__ __forceinline__ void mfma_split(FW &&W, FA &&A, floatx4 (&t)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).l, A(n).h, t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).h, A(n).l, t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).m, A(n).m, t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).m, A(n).h, t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).h, A(n).m, t[n]);
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = mfma_bf16(W(n).h, A(n).h, t[n]);
}
// The same from zero: added to a running sum afterwards, a chunk rounds that once (its instructions would six
// times, FP32 ones eight).  Used where it costs nothing: the channel mixings, and dE/de in the reverse pair
// kernel, whose sums run over all channels.  Against 64 bits (600 atoms, F = 128, two layers) forces 6.6e-7 ->
// 3.6e-7, energies of 22 atoms without layers 1.8e-8 -> 8.2e-9 an atom; in the pair kernels' other products
// it changes neither and takes 3 to 15 % of their time.
template <int N, class FW, class FA>
__device__ __forceinline__ void mfma_split_zero(FW &&W, FA &&A, floatx4 (&t)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) t[n] = floatx4{0.f, 0.f, 0.f, 0.f};
  mfma_split(W, A, t);
}

// This wave's weights of a product in KC chunks of 32 along K: column blocks cb0 .. cb0 + NB - 1, packed by
// fragment (k_split_pack): block (column block, chunk) holds 64 lanes x 8 h, then m, then l, so a
// wave's loads are 1 KB without gaps.  The first PD chunks are loaded at once: before the stores and barriers
// that precede the product, whose end the wait for a later load would also wait for.
constexpr int kSplitBlock = 3 * 512;
template <int NB, int KC, int PD>
struct SplitWeights {
  const __bf16 *p;
  Frag3 next[PD][NB];
  __device__ __forceinline__ void load(int kc, Frag3 (&f)[NB]) const {
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) f[cb] = ld_frag3(p + ((size_t)cb * KC + kc) * kSplitBlock, 512);
  }
  __device__ __forceinline__ SplitWeights(const __bf16 *__restrict__ B, int cb0)
      : p(B + (size_t)cb0 * KC * kSplitBlock + (threadIdx.x & 63) * 8) {
#pragma unroll
    for (int d = 0; d < PD; ++d)
      if (d < KC) load(d, next[d]);
  }
};

// acc[rb][cb] += act_rb * Bt^T from split operands: row i of the activations starts at act + i*ld
// (LDS, h; m and l `plane` and 2 `plane` elements further).  The weights are the instruction's first
// operand: entry t of acc[rb][cb] in lane l is D[rb*16 + l%16][(cb0 + cb)*16 + 4(l/16) + t].
// The weights of the next PD chunks are in flight while the current chunk's products run.  SUMS: every chunk is
// summed from zero and then added; otherwise the products go straight to acc, which spares the partial sums'
// registers and additions.
template <bool SUMS, int RB, int NB, int KC, int PD>
__device__ __forceinline__ void wave_mm_split(const __bf16 *act, int plane, int ld, SplitWeights<NB, KC, PD> &B,
                                              floatx4 (&acc)[RB][NB]) {
  const int lane = threadIdx.x & 63;
  const __bf16 *ap = act + (lane & 15) * ld + 8 * (lane >> 4);
  auto chunk = [&](int kc, Frag3 (&f)[NB]) {
    Frag3 w[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) w[cb] = f[cb];
    if (kc + PD < KC) B.load(kc + PD, f);
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const Frag3 a = ld_frag3(ap + rb * 16 * ld + 32 * kc, plane);
      auto W = [&](int n) -> const Frag3 & { return w[n]; };
      auto A = [&](int) -> const Frag3 & { return a; };
      if constexpr (SUMS) {
        floatx4 t[NB];
        mfma_split_zero(W, A, t);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) acc[rb][cb] += t[cb];
      } else {
        mfma_split(W, A, acc[rb]);
      }
    }
  };
  if constexpr (PD == 1) {
    for (int kc = 0; kc < KC; ++kc) chunk(kc, B.next[0]);
  } else {
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) chunk(kc, B.next[kc % PD]);
  }
}

// acc[rb][cb] += act_rb[16 x Kin] * Bt^T for rb < RB, where row i of block rb starts at
// act + rb*rbs + i*ld (LDS) and Bt is [ncol][Kin] in global memory (row stride Kin); this wave
// covers columns col0 .. col0 + 16*NB - 1 (v_mfma_f32_16x16x4f32).  Inside each 16-wide K
// chunk, lane group q takes k = 4q..4q+3, so one 16-byte load feeds four MFMAs for both
// operands; the weight fragments of the next chunk are loaded while the current chunk's MFMAs
// run.  Element t of acc[rb][cb] in lane l is D_rb[4*(l/16) + t][col0 + cb*16 + l%16].
template <int RB, int NB, bool TR = false>
__device__ __forceinline__ void wave_mm_rows(const float *act, int ld, int rbs, int Kin, const float *__restrict__ Bt,
                                             int col0, floatx4 (&acc)[RB][NB]) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
  const float *ap = act + r * ld + 4 * q;
  const float *bp = Bt + (size_t)(col0 + r) * Kin + 4 * q;
  const size_t bstride = (size_t)16 * Kin;
  float4 bn[NB];
#pragma unroll
  for (int cb = 0; cb < NB; ++cb) bn[cb] = *reinterpret_cast<const float4 *>(bp + cb * bstride);
  for (int k0 = 0; k0 < Kin; k0 += 16) {
    float4 b[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) b[cb] = bn[cb];
    if (k0 + 16 < Kin) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) bn[cb] = *reinterpret_cast<const float4 *>(bp + cb * bstride + k0 + 16);
    }
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float4 a = *reinterpret_cast<const float4 *>(ap + rb * rbs + k0);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        acc[rb][cb] = mfma4_ab<TR>(a.x, b[cb].x, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.y, b[cb].y, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.z, b[cb].z, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.w, b[cb].w, acc[rb][cb]);
      }
    }
  }
}

// The same product with this wave's weight fragments already in registers: b[kc][cb] holds
// Bt[col0 + cb*16 + l%16][16 kc + 4(l/16) .. +3] for the KC = Kin/16 chunks (TR: transposed
// accumulator, as mfma4_ab).
template <int RB, int NB, int KC, bool TR = false>
__device__ __forceinline__ void wave_mm_rows_breg(const float *act, int ld, int rbs, const float4 (&b)[KC][NB],
                                                  floatx4 (&acc)[RB][NB]) {
  const int lane = threadIdx.x & 63;
  const int r = lane & 15, q = lane >> 4;
  const float *ap = act + r * ld + 4 * q;
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
      const float4 a = *reinterpret_cast<const float4 *>(ap + rb * rbs + 16 * kc);
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        acc[rb][cb] = mfma4_ab<TR>(a.x, b[kc][cb].x, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.y, b[kc][cb].y, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.z, b[kc][cb].z, acc[rb][cb]);
        acc[rb][cb] = mfma4_ab<TR>(a.w, b[kc][cb].w, acc[rb][cb]);
      }
    }
  }
}

// Loads this wave's weight fragments for wave_mm_rows_breg.
template <int NB, int KC>
__device__ __forceinline__ void load_bfrag(const float *__restrict__ Bt, int Kin, int col0, float4 (&b)[KC][NB]) {
  const int lane = threadIdx.x & 63;
  const float *bp = Bt + (size_t)(col0 + (lane & 15)) * Kin + 4 * (lane >> 4);
#pragma unroll
  for (int kc = 0; kc < KC; ++kc)
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) b[kc][cb] = *reinterpret_cast<const float4 *>(bp + (size_t)cb * 16 * Kin + 16 * kc);
}

template <int RB, int NB>
__device__ __forceinline__ void zero_acc_rb(floatx4 (&acc)[RB][NB]) {
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) acc[rb][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
}

}  // namespace tn
