// The row-tile attention kernels of head dimension 128 (one of the two sources
// that they are compiled from, side by side).
#include "attn_tiles.h"

namespace pisa {

template hipError_t launch_attn_tiles<128>(const AttnBlockArgs&, int, const uint16_t*, const uint16_t*, const uint16_t*,
                                          const int32_t*, uint16_t*, float*, const uint16_t*, const float*,
                                          hipStream_t);

}  // namespace pisa
