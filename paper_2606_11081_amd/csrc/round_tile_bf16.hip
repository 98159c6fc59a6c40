// The tile round kernels for bfloat16 parameters: see round_tile.h.
#include "round_tile.h"

namespace gasloc {

hipError_t launch_gossip_tile_bf16(const GossipArgs& a, const RowSum& sum, bool fused, int form, const LaunchShape& s,
                                  size_t lds, hipStream_t stream) {
  return launch_tile_form<GASLOC_BF16>(a, sum, fused, form, s, lds, stream);
}

}  // namespace gasloc
