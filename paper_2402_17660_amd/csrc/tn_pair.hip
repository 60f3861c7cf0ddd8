// Launchers of the fused per-pair MFMA kernels (the tile code is in tn_pairtile.h).
#include "tn_pairtile.h"

namespace tn {

bool pair_kernels_support(int F, int K, int L, bool bf16) {
  const bool k_ok = bf16 ? (K == 32 || K == 64) : (K == 16 || K == 32 || K == 48 || K == 64);
  return (F == 64 || F == 128) && k_ok && L >= 0 && L <= kMaxLayers;
}

// ============================================================================ launchers
// Tile shapes: pairs per tile = 16 RB, NW waves per workgroup; MINB, the launch bound's
// minimum waves per SIMD, caps the registers at 512 / MINB per lane and so allows MINB * 4 / NW
// workgroups per compute unit (LDS permitting).  Every shape computes each pair with the same
// arithmetic in the same order, so results do not depend on the shape; tn_autotune picks the
// fastest.  Pairs, waves and workgroups per CU, with the time of a launch on the 100,000-atom box
// (2.6 M pairs) and on a 22-atom molecule (180 pairs; both F = 128, two layers):
//   FP32 forward: 0 = 32, 8, 2 (9.0 ms, 37 us); 1 = 48, 8, 2 (8.3 ms, 48 us; F = 64: 32, 4, 3); 2 = 16, 8, 2
//     (12.9 ms, 27 us); 3 = 16, 16, 1 with two chunks of weights in flight (16.6 ms, 26 us); 4 = 48, 4, 2
//     (8.5 ms, 56 us)
//   FP32 reverse: 0 = 32, 4, 2 (14.6 ms, 65 us; F = 64: 48, 8, 2); 1 = 32, 8, 2 (14.9 ms, 59 us); 2 = 16, 8, 2
//     (19.8 ms, 39 us); 3 = 16, 16, 1 with three chunks in flight (28.3 ms, 40 us); 4 = 64, 8, 1 (14.5 ms,
//     87 us; F = 64: 32, 4, 2)
//   BF16: 0 = 64 pairs, 4 waves, 1 per CU; 1 = 32, 4, 2; 2 = 48, 4, 2; 3, 4: below
// With the products on FP32 instructions the best shapes took 13.7 and 18.7 ms, and 64 and 94 us.
int pair_variant_count(bool bf16) { return bf16 ? 5 : 5; }

// The shape of a call that was neither tuned nor forced, from the pair budget (the pairs
// themselves are known on the device only; molecules fill about half of 32 pairs per atom, boxes
// nearly all).  FP32: a budget of up to 1.5 tiles of 16 pairs per CU is a latency chain, one tile per CU
// and most CUs idle: sixteen waves per tile share its rows and weight loads (166 atoms, 2700 pairs:
// 28.6 and 44.6 us in shape 3, 29.3 and 49.2 in 2, 36 and 58 in the best of the others).  Up to 16384
// there are one or two tiles per CU, and the fewer waves of shape 2 let two of them share one
// (400 atoms, 7500 pairs: 44 and 63 us, 58 and 91 in shape 3, 40 and 62 in the best of the others; F = 64
// 22.6 and 31.3, 29 and 48, 23 and 36).  Beyond, the tile's reuse of each weight fragment and the waves
// that hide its gathers decide, as at 2.6 M pairs: forward shape 1 (800 atoms, 20,900 pairs: 86 us, 96 in
// 0 and 125 in 2; 6000 atoms 473, 539 in 0), reverse shape 1 (136 us, 144 in 0 and 183 in 2; 895 and 925 in
// 0), and shape 0 for F = 64 (20,000 atoms 1142 us, 1233 in 1; 800 atoms 54 and 67).
// BF16, forward and
// reverse: 35 and 51 us in shape 1 at 180 pairs (38 and 75 in 0); 4.0 and 8.6 ms in shapes 4 and
// 3 at 2.6 M pairs (5.6 and 12.1 in 0), shape 3 forward below 100,000 (132 against 145 us at
// 65,000); for F = 64 shapes 2 and 1 (575 and 1203 us at 785,000 pairs, 582 and 1402 in 0).
int pair_default_variant(int F, bool bf16, int64_t max_pairs, bool reverse) {
  if (bf16) {
    if (max_pairs <= 16384) return 1;
    if (F != 128) return reverse ? 1 : 2;
    return reverse || max_pairs <= 100000 ? 3 : 4;
  }
  if (max_pairs <= 6144) return 3;
  if (max_pairs <= 16384) return 2;
  return !reverse || F == 128 ? 1 : 0;
}

template <int TILE>
static unsigned tile_grid(int64_t max_pairs) {
  return (unsigned)((max_pairs + TILE - 1) / TILE);
}

template <int F, int K, int RB, int NW, int MINB, int PD = 1>
static int launch_fwd_v(hipStream_t s, const PairFwdArgs &a) {
  const unsigned grid = tile_grid<16 * RB>(a.max_pairs);
  if (grid == 0) return TN_OK;
  TimedScope ts("edge_fwd", s);
  hipLaunchKernelGGL((k_pair_fwd<F, K, RB, NW, MINB, PD>), dim3(grid), dim3(64 * NW), 0, s, a);
  TN_LAUNCH_CHECK();
  return TN_OK;
}

template <int F, int K, int RB, int NW, int MINB, int PD = 1>
static int launch_bwd_v(hipStream_t s, const PairBwdArgs &a) {
  const unsigned grid = tile_grid<16 * RB>(a.max_pairs);
  if (grid == 0) return TN_OK;
  TimedScope ts("edge_bwd", s);
  hipLaunchKernelGGL((k_pair_bwd<F, K, RB, NW, MINB, PD>), dim3(grid), dim3(64 * NW), 0, s, a);
  TN_LAUNCH_CHECK();
  return TN_OK;
}

template <int F, int K, int RB, int MINB, int NW = 4>
static int launch_fwd_bf16_v(hipStream_t s, const PairFwdArgsB &a) {
  const unsigned grid = tile_grid<16 * RB>(a.max_pairs);
  if (grid == 0) return TN_OK;
  TimedScope ts("edge_fwd", s);
  hipLaunchKernelGGL((k_pair_fwd_bf16<F, K, RB, MINB, NW>), dim3(grid), dim3(64 * NW), 0, s, a);
  TN_LAUNCH_CHECK();
  return TN_OK;
}

template <int F, int K, int RB, int MINB, int NW = 4, int PF = 2>
static int launch_bwd_bf16_v(hipStream_t s, const PairBwdArgsB &a) {
  const unsigned grid = tile_grid<16 * RB>(a.max_pairs);
  if (grid == 0) return TN_OK;
  TimedScope ts("edge_bwd", s);
  hipLaunchKernelGGL((k_pair_bwd_bf16<F, K, RB, MINB, NW, PF>), dim3(grid), dim3(64 * NW), 0, s, a);
  TN_LAUNCH_CHECK();
  return TN_OK;
}

template <int F, int K>
static int launch_fwd(hipStream_t s, const PairFwdArgs &a, int v) {
  constexpr bool wide = F == 128;
  switch (v) {
    case 1: return launch_fwd_v<F, K, wide ? 3 : 2, wide ? 8 : 4, wide ? 4 : 3>(s, a);
    case 2: return launch_fwd_v<F, K, 1, 8, 4>(s, a);
    case 3: return launch_fwd_v<F, K, 1, 16, 4, 2>(s, a);
    case 4: return launch_fwd_v<F, K, 3, 4, 2>(s, a);
    default: return launch_fwd_v<F, K, 2, 8, 4>(s, a);
  }
}

template <int F, int K>
static int launch_bwd(hipStream_t s, const PairBwdArgs &a, int v) {
  constexpr bool wide = F == 128;
  switch (v) {
    case 1: return launch_bwd_v<F, K, 2, 8, 4>(s, a);
    case 2: return launch_bwd_v<F, K, 1, 8, 4>(s, a);
    case 3: return launch_bwd_v<F, K, 1, 16, 4, 3>(s, a);
    case 4: return launch_bwd_v<F, K, wide ? 4 : 2, wide ? 8 : 4, 2>(s, a);
    default: return launch_bwd_v<F, K, wide ? 2 : 3, wide ? 4 : 8, wide ? 2 : 4>(s, a);
  }
}

// BF16 shapes 3 and 4 (F = 128): eight-wave tiles, one workgroup per CU, each weight fragment
// read once for twice (or more) the rows of the four-wave tiles: forward 96 and 112 pairs
// (4.9 against 6.0 ms per launch on 100k atoms); reverse 96 pairs, its prologues loading one row
// ahead or none (about as fast as shape 2: its gathers, not its weight reads, set its time;
// 112 pairs spill).  F = 64 takes shape 2 for them.
template <int F, int K>
static int launch_fwd_bf16(hipStream_t s, const PairFwdArgsB &a, int v) {
  if (v == 1) return launch_fwd_bf16_v<F, K, 2, 2>(s, a);
  if (v == 2) return launch_fwd_bf16_v<F, K, 3, 2>(s, a);
  if constexpr (F == 128) {
    if (v == 3) return launch_fwd_bf16_v<F, K, 6, 1, 8>(s, a);
    if (v == 4) return launch_fwd_bf16_v<F, K, 7, 1, 8>(s, a);
  }
  if (v >= 3) return launch_fwd_bf16_v<F, K, 3, 2>(s, a);
  return launch_fwd_bf16_v<F, K, 4, 1>(s, a);
}

template <int F, int K>
static int launch_bwd_bf16(hipStream_t s, const PairBwdArgsB &a, int v) {
  if (v == 1) return launch_bwd_bf16_v<F, K, 2, 2>(s, a);
  if (v == 2) return launch_bwd_bf16_v<F, K, 3, 2>(s, a);
  if constexpr (F == 128 && K <= 128) {
    if (v == 3) return launch_bwd_bf16_v<F, K, 6, 1, 8, 1>(s, a);
    if (v == 4) return launch_bwd_bf16_v<F, K, 6, 1, 8, 0>(s, a);
  }
  if (v >= 3) return launch_bwd_bf16_v<F, K, 3, 2>(s, a);
  return launch_bwd_bf16_v<F, K, 4, 1>(s, a);
}

#define TN_PAIR_DISPATCH(FN)                                         \
  switch (F * 1000 + K) {                                            \
    case 64016: return FN<64, 16>(s, a, v);                          \
    case 64032: return FN<64, 32>(s, a, v);                          \
    case 64048: return FN<64, 48>(s, a, v);                          \
    case 64064: return FN<64, 64>(s, a, v);                          \
    case 128016: return FN<128, 16>(s, a, v);                        \
    case 128032: return FN<128, 32>(s, a, v);                        \
    case 128048: return FN<128, 48>(s, a, v);                        \
    case 128064: return FN<128, 64>(s, a, v);                        \
    default: return TN_E_UNSUPPORTED;                                \
  }

#define TN_PAIR_DISPATCH_BF16(FN)                                    \
  switch (F * 1000 + K) {                                            \
    case 64032: return FN<64, 32>(s, a, v);                          \
    case 64064: return FN<64, 64>(s, a, v);                          \
    case 128032: return FN<128, 32>(s, a, v);                        \
    case 128064: return FN<128, 64>(s, a, v);                        \
    default: return TN_E_UNSUPPORTED;                                \
  }

int launch_pair_fwd(hipStream_t s, int F, int K, const PairFwdArgs &a, int v) { TN_PAIR_DISPATCH(launch_fwd) }
int launch_pair_bwd(hipStream_t s, int F, int K, const PairBwdArgs &a, int v) { TN_PAIR_DISPATCH(launch_bwd) }
int launch_pair_fwd_bf16(hipStream_t s, int F, int K, const PairFwdArgsB &a, int v) {
  TN_PAIR_DISPATCH_BF16(launch_fwd_bf16)
}
int launch_pair_bwd_bf16(hipStream_t s, int F, int K, const PairBwdArgsB &a, int v) {
  TN_PAIR_DISPATCH_BF16(launch_bwd_bf16)
}

}  // namespace tn
