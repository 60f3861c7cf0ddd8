// Launches of the node steps between the gathers (tn_nodetile.h).
#include "tn_nodetile.h"

namespace tn {

namespace {

template <int F> using Tile = NodeTile<F, node_waves(F)>;

template <class NT, int F, bool FIRST, bool LAST>
__global__ void __launch_bounds__(64 * NT::NW) k_node_fwd(NodeFwdArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[NT::bytes];
  const int64_t a0 = xcd_block() * NT::TA;
  NT nt(smem);
  node_fwd_tile<NT, F, FIRST, LAST>(nt, a, a0, (int)(a.N - a0 < NT::TA ? a.N - a0 : NT::TA));
}

template <class NT, int F, bool TOP, bool BOTTOM>
__global__ void __launch_bounds__(64 * NT::NW) k_node_bwd(NodeBwdArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[NT::bytes];
  const int64_t a0 = xcd_block() * NT::TA;
  NT nt(smem);
  node_bwd_tile<NT, F, TOP, BOTTOM>(nt, a, a0, (int)(a.N - a0 < NT::TA ? a.N - a0 : NT::TA));
}

// Which tile: the small one while a compute unit gets at most two of them (four at F = 64, where they are
// half as large).  A call of energies and forces, two layers, us, small and large tiles (256 compute units):
// F = 128, 22 atoms 281 / 370, 800 618 / 709, 1400 934 / 962, 2000 1163 / 1188, 2489 1440 / 1405, 4000 2121 / 2041;
// F = 64, 48 atoms 195 / 251, 1500 433 / 479, 3000 711 / 743, 4000 886 / 911, 6000 1232 / 1262 (2 % behind the line,
// where the large tile reads the weights a quarter as often).
bool small_tiles(int F, int64_t N) { return N * F <= 2048 * 128; }

}  // namespace

#define TN_NODE_LAUNCH(KERNEL, F, P, Q)                                                                       \
  if (small_tiles(F, a.N)) {                                                                                  \
    using NT = NodeTileSmall<F>;                                                                              \
    hipLaunchKernelGGL((KERNEL<NT, F, P, Q>), dim3((unsigned)((a.N + NT::TA - 1) / NT::TA)), dim3(64 * NT::NW), 0, s, a); \
  } else {                                                                                                    \
    using NT = Tile<F>;                                                                                       \
    hipLaunchKernelGGL((KERNEL<NT, F, P, Q>), dim3((unsigned)((a.N + NT::TA - 1) / NT::TA)), dim3(64 * NT::NW), 0, s, a); \
  }
#define TN_NODE_DISPATCH(KERNEL, P, Q)                                                                        \
  if (a.N <= 0) return TN_OK;                                                                                 \
  if (F == 64) {                                                                                              \
    if (P && Q) { TN_NODE_LAUNCH(KERNEL, 64, true, true) }                                                    \
    else if (P) { TN_NODE_LAUNCH(KERNEL, 64, true, false) }                                                   \
    else if (Q) { TN_NODE_LAUNCH(KERNEL, 64, false, true) }                                                   \
    else { TN_NODE_LAUNCH(KERNEL, 64, false, false) }                                                         \
  } else if (F == 128) {                                                                                      \
    if (P && Q) { TN_NODE_LAUNCH(KERNEL, 128, true, true) }                                                   \
    else if (P) { TN_NODE_LAUNCH(KERNEL, 128, true, false) }                                                  \
    else if (Q) { TN_NODE_LAUNCH(KERNEL, 128, false, true) }                                                  \
    else { TN_NODE_LAUNCH(KERNEL, 128, false, false) }                                                        \
  } else {                                                                                                    \
    return TN_E_UNSUPPORTED;                                                                                  \
  }                                                                                                           \
  TN_LAUNCH_CHECK();                                                                                          \
  return TN_OK;

int launch_node_fwd(hipStream_t s, int F, bool first, bool last, const NodeFwdArgs &a) {
  TN_NODE_DISPATCH(k_node_fwd, first, last)
}
int launch_node_bwd(hipStream_t s, int F, bool top, bool bottom, const NodeBwdArgs &a) {
  TN_NODE_DISPATCH(k_node_bwd, top, bottom)
}

MixSplit split_mix(const tn_model *m, const SplitMix &x) {
  MixSplit r;
  for (int p = 0; p < 3; ++p) r.W[p] = m->wsplit + x.at[p];
  return r;
}

}  // namespace tn
