// The node steps between the gathers, for tiles of 16 or 4 atoms (FP32, F = 64 or 128).
//
// A step of the network's node part is a per-part channel mixing (a product over channels, on the
// matrix cores) between maps of one channel's nine coordinates (gating, normalisation, 3x3
// products).  With the weights as the instruction's first operand a lane ends a mixing with four
// channels of one atom, and with one accumulator per coordinate it holds all nine coordinates of
// them: the channel maps run on the accumulators, and the next mixing's operand goes from
// registers to LDS.  So everything between two gathers is one launch that reads and writes each
// [N, 9, F] array once:
//   forward  embedding mixing, gate, [normalise, W1 mixing]            Xr, g -> T0, X, Y
//            W2 mixing, residual, [normalise, W1 mixing]               Pb, X -> D, X', Y'
//            (last: the part norms and their LayerNorm instead)
//   reverse  the LayerNorm's and part norms' adjoint, residual adjoint, W2^T mixing, product adjoint
//            W1^T mixing, normalisation adjoint, then the same of the layer below
//            W1^T mixing, normalisation adjoint, gate adjoint, embedding mixing's adjoint
// Bound by those reads and writes: for a 100,000-atom box at F = 128 and two layers 37 arrays of
// 461 MB, 3.6 ms at the rate of a large copy; the six launches take 5.1 ms, one launch per step (61
// arrays, ten of them mixings on FP32 instructions) 6.4 ms.  A large tile alone on its compute unit is
// bound by its vector instructions and the memory-side cache's latency: 27 us on average for 22 atoms
// at F = 128, of which the maps and staging about half, the mixings' weights the rest; the small
// tile takes 12.7 us (a call 370 -> 281 us).
//
// The mixings run on split operands (tn_mfma.h).
#pragma once

#include "tn_internal.h"
#include "tn_device.h"
#include "tn_mfma.h"

namespace tn {

// One mixing's three matrices as split weights.
struct MixSplit {
  const __bf16 *W[3] = {nullptr, nullptr, nullptr};
};

struct NodeFwdArgs {
  int64_t N = 0;
  const float *in = nullptr;     // first: Xr (embedding sums); else Pb
  const float *X = nullptr;      // not first: the layer's input features
  const double *g = nullptr;     // first: the gates [N, 3F]
  float *mid = nullptr;          // first: T0, the mixed embedding; else D, the mixed product
  float *Xo = nullptr;           // the features that leave
  float *Y = nullptr;            // not last: the next layer's mixed input
  // last: LayerNorm of the part norms [N, 3F]: weights, output, normalised values, 1 / deviation
  const double *ln_g = nullptr, *ln_b = nullptr;
  double *q = nullptr, *xhat = nullptr, *rstd = nullptr;
  MixSplit A, B;                 // the embedding's or W2; W1 of the next layer
};

struct NodeBwdArgs {
  int64_t N = 0;
  const float *X = nullptr;      // the features entering the layer above (top: leaving the network)
  // top: the adjoint entering the part norms' LayerNorm, what its forward stored, its weights
  const double *dq = nullptr, *xhat = nullptr, *rstd = nullptr, *ln_g = nullptr;
  float *dX = nullptr;           // not top: read; not bottom: written
  float *dY = nullptr;           // not top: adjoint of the layer above's Y, read; not bottom: written
  const float *D = nullptr, *Y = nullptr, *M = nullptr;   // not bottom: of the layer below
  float *dM = nullptr;           // not bottom
  const float *T0 = nullptr;     // bottom
  const double *g = nullptr, *ez = nullptr;
  double *dez = nullptr;
  float *dXr = nullptr;
  MixSplit A, B;                 // W1^T of the layer above; W2^T of the layer below or the embedding's
};

// ---------------------------------------------------------------- one channel's maps
// A number whose operations round one by one: the compiler would otherwise contract a b + c d into a
// fused multiply-add either way round, and differently where the code around it differs, while a
// result may not depend on the tile that formed it.  Fused operations are written out (fma below).
template <class T>
struct Fp {
  T v;
  Fp() = default;
  template <class U> __device__ __forceinline__ explicit Fp(U x) : v((T)x) {}
};
#define TN_FP_OP(OP)                                                                    \
  template <class T> __device__ __forceinline__ Fp<T> operator OP(Fp<T> a, Fp<T> b) {  \
    _Pragma("clang fp contract(off)") return Fp<T>(a.v OP b.v);                         \
  }
TN_FP_OP(+)
TN_FP_OP(-)
TN_FP_OP(*)
TN_FP_OP(/)
#undef TN_FP_OP
template <class T> __device__ __forceinline__ Fp<T> operator-(Fp<T> a) { return Fp<T>(-a.v); }
__device__ __forceinline__ Fp<float> fma(Fp<float> a, Fp<float> b, Fp<float> c) { return Fp<float>(__builtin_fmaf(a.v, b.v, c.v)); }
__device__ __forceinline__ Fp<double> fma(Fp<double> a, Fp<double> b, Fp<double> c) { return Fp<double>(__builtin_fma(a.v, b.v, c.v)); }
// The 3x3 products with fused operations (C = A B, A^T B, A B^T), added to C with ADD.
template <bool ADD, bool TA, bool TB, class T>
__device__ __forceinline__ void mm_fma(const Fp<T> A[9], const Fp<T> B[9], Fp<T> C[9]) {
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const Fp<T> a0 = A[TA ? r : r * 3], b0 = B[TB ? q * 3 : q];
      Fp<T> s = ADD ? fma(a0, b0, C[r * 3 + q]) : a0 * b0;
#pragma unroll
      for (int k = 1; k < 3; ++k) s = fma(A[TA ? k * 3 + r : r * 3 + k], B[TB ? q * 3 + k : k * 3 + q], s);
      C[r * 3 + q] = s;
    }
}

using F32 = Fp<float>;
using F64 = Fp<double>;
template <class T, class U>
__device__ __forceinline__ void to_fp(const U x[9], Fp<T> o[9]) {
#pragma unroll
  for (int q = 0; q < 9; ++q) o[q] = Fp<T>(x[q]);
}

// The forward maps run in FP64 and round once, to the FP32 features that leave (the energy is most
// sensitive to the features' rounding; the launches wait on memory, and the FP64 rate is FP32's).
__device__ __forceinline__ void normalize_channel(F64 x[9]) {   // x / (||x|| + 1)
  const F64 s = F64(1) / (norm9(x) + F64(1));
#pragma unroll
  for (int q = 0; q < 9; ++q) x[q] = x[q] * s;
}
__device__ __forceinline__ void residual_channel(const float d[9], float x[9]) {   // xb + d + d d
  F64 D[9], Dm[9], Q[9], qc[9], v[9];
  to_fp(d, D);
  to_fp(x, v);
  normalize_channel(v);
  rec(D, Dm);
  mm_fma<false, false, false>(Dm, Dm, Q);
  dec(Q, qc);
#pragma unroll
  for (int q = 0; q < 9; ++q) x[q] = (float)(v[q] + (D[q] + qc[q])).v;
}

// g = dX -> dD = dX + rec^T(dQ D^T + D^T dQ), dQ = dec^T(dX)
__device__ __forceinline__ void residual_bwd_channel(const float d[9], float g[9]) {
  F32 D[9], G[9], Dm[9], dQ[9], A[9], r[9];
  to_fp(d, D);
  to_fp(g, G);
  rec(D, Dm);
  dec_adj(G, dQ);
  mm_fma<false, false, true>(dQ, Dm, A);
  mm_fma<true, true, false>(Dm, dQ, A);
  rec_adj(A, r);
#pragma unroll
  for (int q = 0; q < 9; ++q) g[q] = (G[q] + r[q]).v;
}

// g through x / (||x|| + 1): g s - <g, x> s^2 grad||x||, s = 1 / (||x|| + 1)
__device__ __forceinline__ void normalize_bwd_channel(const F32 x[9], F32 g[9]) {
  const F32 s = F32(1) / (norm9(x) + F32(1));
  F32 gn[9], dot = g[0] * x[0];
#pragma unroll
  for (int q = 1; q < 9; ++q) dot = fma(g[q], x[q], dot);
  norm_grad_parts(x, F32(1), F32(1), F32(1), gn);
  const F32 w = -(dot * s * s);
#pragma unroll
  for (int q = 0; q < 9; ++q) g[q] = fma(g[q], s, w * gn[q]);
}

// g = dPb through Pb = P / (||P|| + 1), P = Y M + M Y -> y = dY, m = dM (in place)
__device__ __forceinline__ void product_bwd_channel(const float gf[9], float y[9], float m[9]) {
  F32 g[9], t[9], Ym[9], Mm[9], A[9], p[9], dP[9];
  to_fp(gf, g);
  to_fp(y, t);
  rec(t, Ym);
  to_fp(m, t);
  rec(t, Mm);
  mm_fma<false, false, false>(Ym, Mm, A);
  mm_fma<true, false, false>(Mm, Ym, A);
  dec(A, p);
  normalize_bwd_channel(p, g);
  dec_adj(g, dP);
  mm_fma<false, false, true>(dP, Mm, A);   // dY = dP M^T + M^T dP
  mm_fma<true, true, false>(Mm, dP, A);
  rec_adj(A, t);
#pragma unroll
  for (int q = 0; q < 9; ++q) y[q] = t[q].v;
  mm_fma<false, true, false>(Ym, dP, A);   // dM = Y^T dP + dP Y^T
  mm_fma<true, false, true>(dP, Ym, A);
  rec_adj(A, t);
#pragma unroll
  for (int q = 0; q < 9; ++q) m[q] = t[q].v;
}

// V consecutive doubles (V = 1 or 4).
template <int V>
__device__ __forceinline__ void ldd(const double *p, double (&o)[V]) {
  if constexpr (V == 4) {
    const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
    o[0] = a.x;
    o[1] = a.y;
    o[2] = b.x;
    o[3] = b.y;
  } else {
    o[0] = p[0];
  }
}
template <int V>
__device__ __forceinline__ void std_(double *p, const double (&o)[V]) {
  if constexpr (V == 4) {
    reinterpret_cast<double2 *>(p)[0] = make_double2(o[0], o[1]);
    reinterpret_cast<double2 *>(p)[1] = make_double2(o[2], o[3]);
  } else {
    p[0] = o[0];
  }
}

// ---------------------------------------------------------------- the tile
// NW waves; wave w holds channels [w F / NW, (w + 1) F / NW) in NB blocks of 16, lane l of block cb
// the channels cb*16 + 4(l/16) .. +3 of atom l%16.
template <int F, int WAVES>
struct NodeTile {
  static constexpr int NW = WAVES;
  static constexpr int NB = F / (16 * NW), KC = F / 32, LD = F + kPadH, PL = 9 * 16 * LD;
  static_assert(F % (16 * NW) == 0 && F % 32 == 0, "whole blocks per wave");
  static constexpr size_t bytes = 3 * PL * sizeof(__bf16) + 2 * F * sizeof(double);
  static constexpr int TA = 16, VT = 4;   // atoms; channels of a lane in a block
  static constexpr int CG = NB == 1 ? 3 : 1;   // coordinates whose products run side by side
  static constexpr bool kEarly = false;
  using Feat = floatx4[9][NB];
  struct Frags {};
  __device__ __forceinline__ void weights(const MixSplit &, Frags &) const {}

  __bf16 *sA;
  double *sSum;  // [2][16 atoms][F / 16]
  int wave, r16, q;

  __device__ __forceinline__ explicit NodeTile(char *smem) {
    sA = reinterpret_cast<__bf16 *>(smem);
    sSum = reinterpret_cast<double *>(smem + 3 * PL * sizeof(__bf16));
    wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    r16 = threadIdx.x & 15;
    q = (threadIdx.x & 63) >> 4;
  }
  __device__ __forceinline__ int col(int cb) const { return (wave * NB + cb) * 16 + 4 * q; }
  // rows past the last atom read it again and are not stored
  __device__ __forceinline__ bool live(int navail) const { return r16 < navail; }
  __device__ __forceinline__ bool leader() const { return wave == 0 && q == 0; }   // one lane per atom
  __device__ __forceinline__ int64_t row(int64_t a0, int navail) const { return a0 + (r16 < navail ? r16 : navail - 1); }

  __device__ __forceinline__ void load(const float *X, int64_t i, Feat &x) const {
#pragma unroll
    for (int c = 0; c < 9; ++c)
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) x[c][cb] = ld4(X + (i * 9 + c) * F + col(cb));
  }
  __device__ __forceinline__ void store(float *X, int64_t i, int navail, const Feat &x) const {
    if (r16 < navail) {
#pragma unroll
      for (int c = 0; c < 9; ++c)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) st4(X + (i * 9 + c) * F + col(cb), x[c][cb]);
    }
  }
  // Sum over an atom's channels: of four neighbours, of the four fours of a block of 16, of the blocks
  // in order; `at` (0 or 1) is not used twice without a barrier in between.
  __device__ __forceinline__ double atom_sum(const double (&part)[NB][VT], int at) const {
    double *s = sSum + (at * 16 + r16) * (F / 16);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      double v = (part[cb][0] + part[cb][1]) + (part[cb][2] + part[cb][3]);
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (q == 0) s[wave * NB + cb] = v;
    }
    __syncthreads();
    double v = 0.0;
#pragma unroll
    for (int b = 0; b < F / 16; ++b) v += s[b];
    return v;
  }

  // x to LDS as split operands
  __device__ __forceinline__ void stage(const Feat &x) {
    __syncthreads();   // the last mixing has read sA
#pragma unroll
    for (int c = 0; c < 9; ++c)
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) st4_split(sA + (c * 16 + r16) * LD + col(cb), PL, x[c][cb]);
    __syncthreads();
  }
  // y = the staged operand times the part's matrix
  __device__ __forceinline__ void product(const MixSplit &m, const Frags &, Feat &y) const {
    const int lane = threadIdx.x & 63;
    const __bf16 *ap = sA + r16 * LD + 8 * q;
    Frag3 next[3][NB];
    auto weights = [&](int kc) {
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb)
          next[p][cb] = ld_frag3(m.W[p] + (size_t)((wave * NB + cb) * KC + kc) * kSplitBlock + lane * 8, 512);
    };
    weights(0);
#pragma unroll
    for (int c = 0; c < 9; ++c)
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) y[c][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
    // (two blocks per wave, in the molecule kernel: unrolled, the chunks' loads fill registers and it spills)
    constexpr int kUnroll = NB > 1 ? 1 : KC;
#pragma unroll kUnroll
    for (int kc = 0; kc < KC; ++kc) {
      Frag3 w[3][NB];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) w[p][cb] = next[p][cb];
      if (kc + 1 < KC) weights(kc + 1);
#pragma unroll
      for (int c0 = 0; c0 < 9; c0 += CG) {   // two or three chains side by side
        Frag3 a[CG];
#pragma unroll
        for (int n = 0; n < CG; ++n) a[n] = ld_frag3(ap + (c0 + n) * 16 * LD + 32 * kc, PL);
        floatx4 t[CG * NB];
        mfma_split_zero([&](int n) -> const Frag3 & { return w[coord_part(c0 + n / NB)][n % NB]; },
                        [&](int n) -> const Frag3 & { return a[n / NB]; }, t);
#pragma unroll
        for (int n = 0; n < CG * NB; ++n) y[c0 + n / NB][n % NB] += t[n];
      }
    }
  }
};

// The same steps for tiles of four atoms, F threads each: a thread holds one channel of one atom, a
// mixing's rows are packed into four blocks of 16 (I: 4 rows, A: 12, S: 20) and its result goes
// through LDS to the thread that maps it.  Every number is formed by the operations of the tile
// above in their order.  For few atoms: the maps, most of a lone tile's time, spread over four times
// the lanes, and with one channel's registers a mixing's weights are all in flight while the rows are
// staged (a lone tile otherwise waits for the memory-side cache at every chunk).
template <int F>
struct NodeTileSmall {
  static constexpr int TA = 4, VT = 1, NB = 1, NW = TA * F / 64, KC = F / 32, LD = F + kPadH, PL = 64 * LD, LDY = F + 4;
  static_assert(16 * NW == F && F % 64 == 0, "a wave per 16 columns, whole waves per atom");
  static constexpr bool kEarly = true;
  static constexpr size_t bytes = 3 * PL * sizeof(__bf16) + 64 * LDY * sizeof(float) + 2 * TA * (F / 16) * sizeof(double);
  using Feat = float[9][1][1];
  struct Frags {
    Frag3 w[KC][3];
  };

  __bf16 *sA;
  float *sY;
  double *sSum;  // [2][TA][F / 16]
  int wave, atom, ch;

  __device__ __forceinline__ explicit NodeTileSmall(char *smem) {
    sA = reinterpret_cast<__bf16 *>(smem);
    smem += 3 * PL * sizeof(__bf16);
    sY = reinterpret_cast<float *>(smem);
    smem += 64 * LDY * sizeof(float);
    sSum = reinterpret_cast<double *>(smem);
    wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    atom = wave * 64 / F;
    ch = threadIdx.x % F;
  }
  __device__ __forceinline__ int col(int) const { return ch; }
  __device__ __forceinline__ bool live(int navail) const { return atom < navail; }
  __device__ __forceinline__ bool leader() const { return ch == 0; }
  __device__ __forceinline__ int64_t row(int64_t a0, int navail) const { return a0 + (atom < navail ? atom : navail - 1); }
  // an operand row's place in the blocks
  __device__ __forceinline__ int at(int c) const { return (c == 0 ? 0 : c < 4 ? 16 + TA * (c - 1) : 32 + TA * (c - 4)) + atom; }

  __device__ __forceinline__ void load(const float *X, int64_t i, Feat &x) const {
#pragma unroll
    for (int c = 0; c < 9; ++c) x[c][0][0] = X[(i * 9 + c) * F + ch];
  }
  __device__ __forceinline__ void store(float *X, int64_t i, int navail, const Feat &x) const {
    if (live(navail)) {
#pragma unroll
      for (int c = 0; c < 9; ++c) X[(i * 9 + c) * F + ch] = x[c][0][0];
    }
  }
  __device__ __forceinline__ double atom_sum(const double (&part)[1][1], int at) const {
    double *s = sSum + (at * TA + atom) * (F / 16);
    double v = part[0][0];
#pragma unroll
    for (int m = 1; m < 16; m *= 2) v += __shfl_xor(v, m, 64);
    if (ch % 16 == 0) s[ch / 16] = v;
    __syncthreads();
    v = 0.0;
#pragma unroll
    for (int b = 0; b < F / 16; ++b) v += s[b];
    return v;
  }
  __device__ __forceinline__ void stage(const Feat &x) {
    __syncthreads();   // the last mixing has read sA
#pragma unroll
    for (int c = 0; c < 9; ++c) st_split<1>(sA + at(c) * LD + ch, PL, x[c][0]);
    __syncthreads();
  }
  __device__ __forceinline__ void weights(const MixSplit &m, Frags &f) const {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        f.w[kc][p] = ld_frag3(m.W[p] + (size_t)(wave * KC + kc) * kSplitBlock + lane * 8, 512);
  }
  __device__ __forceinline__ void product(const MixSplit &, const Frags &f, Feat &y) const {
    const int r16 = threadIdx.x & 15, q = (threadIdx.x & 63) >> 4;
    const __bf16 *ap = sA + r16 * LD + 8 * q;
    floatx4 acc[4];
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) acc[rb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) {
      Frag3 a[4];
      floatx4 t[4];
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) a[rb] = ld_frag3(ap + rb * 16 * LD + 32 * kc, PL);
      mfma_split_zero([&](int rb) -> const Frag3 & { return f.w[kc][rb < 2 ? rb : 2]; },
                 [&](int rb) -> const Frag3 & { return a[rb]; }, t);
#pragma unroll
      for (int rb = 0; rb < 4; ++rb) acc[rb] += t[rb];
    }
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) st4(sY + (rb * 16 + r16) * LDY + wave * 16 + 4 * q, acc[rb]);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 9; ++c) y[c][0][0] = sY[at(c) * LDY + ch];
  }
};

// ---------------------------------------------------------------- the steps
// One lane's channels of a tile: fn(block, channel in the lane, the nine coordinates, in and out).
template <class NT, class Fn>
__device__ __forceinline__ void channels(typename NT::Feat &x, Fn &&fn) {
#pragma unroll
  for (int cb = 0; cb < NT::NB; ++cb)
#pragma unroll
    for (int t = 0; t < NT::VT; ++t) {
      float v[9];
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = x[c][cb][t];
      fn(cb, t, v);
#pragma unroll
      for (int c = 0; c < 9; ++c) x[c][cb][t] = v[c];
    }
}
template <class NT>
__device__ __forceinline__ void channel(const typename NT::Feat &x, int cb, int t, float (&v)[9]) {
#pragma unroll
  for (int c = 0; c < 9; ++c) v[c] = x[c][cb][t];
}

template <class NT, int F, bool FIRST, bool LAST>
__device__ __forceinline__ void node_fwd_tile(NT &nt, const NodeFwdArgs &a, int64_t a0, int navail) {
  constexpr int NB = NT::NB, VT = NT::VT;
  const int64_t i = nt.row(a0, navail);
  typename NT::Feat x, y, z;
  typename NT::Frags w;
  double g[FIRST ? NB : 1][3][VT];
  auto operands = [&]() {   // what the first mixing's result meets
    if constexpr (!FIRST) {
      nt.load(a.X, i, z);
    } else {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb)
#pragma unroll
        for (int p = 0; p < 3; ++p) ldd<VT>(a.g + i * 3 * F + p * F + nt.col(cb), g[cb][p]);
    }
  };
  nt.load(a.in, i, x);
  nt.weights(a.A, w);
  if constexpr (NT::kEarly) operands();
  nt.stage(x);
  if constexpr (!NT::kEarly && !FIRST) operands();
  nt.product(a.A, w, y);
  if constexpr (!LAST) nt.weights(a.B, w);
  nt.store(a.mid, i, navail, y);
  if constexpr (!NT::kEarly && FIRST) operands();
  if constexpr (FIRST) {   // the gating product is formed in FP64 and rounded once
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int c = 0; c < 9; ++c)
#pragma unroll
        for (int t = 0; t < VT; ++t) x[c][cb][t] = (float)(g[cb][coord_part(c)][t] * (double)y[c][cb][t]);
  } else {
    channels<NT>(x, [&](int cb, int t, float (&v)[9]) {
      float d[9];
      channel<NT>(y, cb, t, d);
      channel<NT>(z, cb, t, v);
      residual_channel(d, v);
    });
  }
  nt.store(a.Xo, i, navail, x);
  if constexpr (LAST) {   // LayerNorm of the part norms (population variance, eps 1e-5)
    double n[NB][3][VT], sum[NB][VT];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        float f[9];
        F64 v[9];
        channel<NT>(x, cb, t, f);
        to_fp(f, v);
        const F64 n0 = norm_I(v), n1 = norm_A(v), n2 = norm_S(v);
        n[cb][0][t] = n0.v;
        n[cb][1][t] = n1.v;
        n[cb][2][t] = n2.v;
        sum[cb][t] = (n0 + n1 + n2).v;
      }
    const double mean = nt.atom_sum(sum, 0) / (3 * F);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        F64 s(0);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const F64 d = F64(n[cb][p][t]) - F64(mean);
          s = fma(d, d, s);
          n[cb][p][t] = d.v;
        }
        sum[cb][t] = s.v;
      }
    const double rs = 1.0 / sqrt(nt.atom_sum(sum, 1) / (3 * F) + 1e-5);
    if (nt.live(navail)) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb)
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const int k = p * F + nt.col(cb);
          double g[VT], b[VT], o[VT];
          ldd<VT>(a.ln_g + k, g);
          ldd<VT>(a.ln_b + k, b);
#pragma unroll
          for (int t = 0; t < VT; ++t) {
            n[cb][p][t] *= rs;
            o[t] = __builtin_fma(n[cb][p][t], g[t], b[t]);
          }
          std_<VT>(a.xhat + i * 3 * F + k, n[cb][p]);
          std_<VT>(a.q + i * 3 * F + k, o);
        }
      if (nt.leader()) a.rstd[i] = rs;
    }
  } else {
    channels<NT>(x, [&](int, int, float (&v)[9]) {
      F64 u[9];
      to_fp(v, u);
      normalize_channel(u);
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = (float)u[c].v;
    });
    nt.stage(x);
    nt.product(a.B, w, y);
    nt.store(a.Y, i, navail, y);
  }
}

template <class NT, int F, bool TOP, bool BOTTOM>
__device__ __forceinline__ void node_bwd_tile(NT &nt, const NodeBwdArgs &a, int64_t a0, int navail) {
  constexpr int NB = NT::NB, VT = NT::VT;
  const int64_t i = nt.row(a0, navail);
  typename NT::Feat x, y, z, u, d0, y0, m0;
  typename NT::Frags w;
  auto below = [&]() {   // of the layer below
    if constexpr (!BOTTOM) {
      nt.load(a.Y, i, y0);
      nt.load(a.M, i, m0);
    }
  };
  auto mixed = [&]() {   // D, or the mixed embedding
    nt.load(BOTTOM ? a.T0 : a.D, i, d0);
  };
  if constexpr (TOP) {   // the adjoints of the LayerNorm and of the part norms
    nt.load(a.X, i, z);
    double gd[NB][3][VT], h[NB][3][VT], s1[NB][VT], s2[NB][VT];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      double g[3][VT];
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const int k = p * F + nt.col(cb);
        ldd<VT>(a.dq + i * 3 * F + k, gd[cb][p]);
        ldd<VT>(a.xhat + i * 3 * F + k, h[cb][p]);
        ldd<VT>(a.ln_g + k, g[p]);
      }
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        F64 a1(0), a2(0);
#pragma unroll
        for (int p = 0; p < 3; ++p) {
          const F64 v = F64(gd[cb][p][t]) * F64(g[p][t]);
          a1 = a1 + v;
          a2 = fma(v, F64(h[cb][p][t]), a2);
          gd[cb][p][t] = v.v;
        }
        s1[cb][t] = a1.v;
        s2[cb][t] = a2.v;
      }
    }
    if constexpr (NT::kEarly) {
      mixed();
      nt.weights(a.B, w);
      below();
    }
    const double m1 = nt.atom_sum(s1, 0) / (3 * F), m2 = nt.atom_sum(s2, 1) / (3 * F), rs = a.rstd[i];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int t = 0; t < VT; ++t) {
        float f[9];
        F64 v[9], d[9], n[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) n[p] = F64(rs) * fma(-F64(h[cb][p][t]), F64(m2), F64(gd[cb][p][t]) - F64(m1));
        channel<NT>(z, cb, t, f);
        to_fp(f, v);
        norm_grad_parts(v, n[0], n[1], n[2], d);
#pragma unroll
        for (int c = 0; c < 9; ++c) x[c][cb][t] = (float)d[c].v;
      }
  } else {
    auto above = [&]() {
      nt.load(a.dX, i, u);
      nt.load(a.X, i, z);
    };
    nt.load(a.dY, i, x);
    nt.weights(a.A, w);
    if constexpr (NT::kEarly) {
      above();
      mixed();
      below();
    }
    nt.stage(x);
    if constexpr (!NT::kEarly) above();
    nt.product(a.A, w, y);
    nt.weights(a.B, w);
    channels<NT>(x, [&](int cb, int t, float (&v)[9]) {
      float p[9], q[9], e[9];
      F32 g[9], X[9];
      channel<NT>(u, cb, t, p);
      channel<NT>(y, cb, t, q);
      channel<NT>(z, cb, t, e);
      to_fp(e, X);
#pragma unroll
      for (int c = 0; c < 9; ++c) g[c] = F32(p[c]) + F32(q[c]);
      normalize_bwd_channel(X, g);
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = g[c].v;
    });
  }
  if constexpr (!NT::kEarly) mixed();
  if constexpr (BOTTOM) {
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        const int64_t o = i * 3 * F + p * F + nt.col(cb);
        double g[VT], ez[VT], s[VT] = {};
        ldd<VT>(a.g + o, g);
        ldd<VT>(a.ez + o, ez);
#pragma unroll
        for (int c = 0; c < 9; ++c)
          if (coord_part(c) == p) {
#pragma unroll
            for (int t = 0; t < VT; ++t) {
              const double d = (double)x[c][cb][t];
              s[t] = __builtin_fma(d, (double)d0[c][cb][t], s[t]);
              x[c][cb][t] = (float)(g[t] * d);
            }
          }
#pragma unroll
        for (int t = 0; t < VT; ++t) s[t] *= silu_grad(ez[t]);
        if (nt.live(navail)) std_<VT>(a.dez + o, s);
      }
    nt.stage(x);
    nt.product(a.B, w, y);
    nt.store(a.dXr, i, navail, y);
  } else {
    nt.store(a.dX, i, navail, x);
    channels<NT>(x, [&](int cb, int t, float (&v)[9]) {
      float d[9];
      channel<NT>(d0, cb, t, d);
      residual_bwd_channel(d, v);
    });
    nt.stage(x);
    if constexpr (!NT::kEarly) below();
    nt.product(a.B, w, y);
    channels<NT>(y, [&](int cb, int t, float (&v)[9]) {
      float yc[9], mc[9];
      channel<NT>(y0, cb, t, yc);
      channel<NT>(m0, cb, t, mc);
      product_bwd_channel(v, yc, mc);
#pragma unroll
      for (int c = 0; c < 9; ++c) {
        y0[c][cb][t] = yc[c];
        m0[c][cb][t] = mc[c];
      }
    });
    nt.store(a.dY, i, navail, y0);
    nt.store(a.dM, i, navail, m0);
  }
}

// The waves of a tile in a launch of its own: 16 channels each.
constexpr int node_waves(int F) { return F / 16; }

int launch_node_fwd(hipStream_t s, int F, bool first, bool last, const NodeFwdArgs &a);
int launch_node_bwd(hipStream_t s, int F, bool top, bool bottom, const NodeBwdArgs &a);

// A mixing's split weights.
MixSplit split_mix(const tn_model *m, const SplitMix &x);

}  // namespace tn
