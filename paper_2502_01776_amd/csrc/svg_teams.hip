// The attention kernel with two teams of four wavefronts to a workgroup: for calls that give a compute unit one query tile at most.
//
// A workgroup of attn_kernel that has its CU to itself, one wavefront to a SIMD, runs at 0.7 of the rate two of them reach together (1.13-1.2
// us a key tile at head dimension 128 against 0.88, 0.75-0.81 against 0.5 at 64): nothing covers a wavefront's softmax, operand reads and
// barriers.  Here the second half of the CU takes every other key tile of the same query tile, with staging buffers of its own, and the two
// results (output, maximum, row sum) are merged through LDS at the end.  Bound as attn_kernel is with two workgroups on a CU, less the
// barrier both teams share: 10-15 % of the rate once there are several workgroups to a CU, so it is taken for the first only.  By passes of 1 to 48
// heads of 1500 to 24000 rows: dense 1.20 times as fast (2 heads of 12142 rows at head dimension 128 214 -> 164 us, 2 of 14545 at 64 171 -> 129),
// exact masks 1.10 (5 of 5140 92 -> 70), sparse 1.06 (3 of 9900 85 -> 68), gathering 1.05 (89 -> 74); where text-row tiles are the time of the pass 0.98-1.01.
#include "svg_attn_kernel.h"

namespace svg {

namespace attn {

// One workgroup to a CU, each text-row tile counted as the four workgroups that may take it in parts (with more of them 0.76-0.96).  Below 24 key
// tiles the merge costs what the shorter chain saves (0.95-1.07).  257 to 3500 query tiles: dense 0.78-0.95, sparse and exact masks 0.7-1.0.
// One line for all passes: a sparse pass over full lists gives the bits of the dense pass, gathering in place those of the layout passes.
bool two_teams(const Geo& g) {
  if (g.bm != 128 || g.nk < 24) return false;
  const SparseOrder so = sparse_order(g.B * g.H, g.nq, g.bm, g.off, g.video_end, g.N, 0, 0, 0, g.nk);
  return (long long)g.B * g.H * (so.nl + 4 * so.nh) <= 256;
}

int launch_teams(const Geo& g, const AttnArgs& a, int mode, hipStream_t stream) {
  const bool wide = g.D == 128;
  switch (mode) {
    case kDense: return wide ? launch_one<128, 4, 64, kDense, 2>(a, g.N, stream) : launch_one<64, 4, 64, kDense, 2>(a, g.N, stream);
    case kSparse: return wide ? launch_one<128, 4, 64, kSparse, 2>(a, g.N, stream) : launch_one<64, 4, 64, kSparse, 2>(a, g.N, stream);
    case kSparseExact: return wide ? launch_one<128, 4, 64, kSparseExact, 2>(a, g.N, stream) : launch_one<64, 4, 64, kSparseExact, 2>(a, g.N, stream);
    default: return wide ? launch_one<128, 4, 64, kSparseGather, 2>(a, g.N, stream) : launch_one<64, 4, 64, kSparseGather, 2>(a, g.N, stream);
  }
}

}  // namespace attn

}  // namespace svg
