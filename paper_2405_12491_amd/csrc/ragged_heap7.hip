// ragged_heap7.hip -- the padded-heap walk of ragged trees with 7 top levels, 2 trees per batch.
#include "ragged_heap.h"

namespace bridger {

int launch_ragged_heap7(const LaunchArgs &a, int waves, int64_t n_wg, int lds_bytes, void *stream) {
  return launch_heap_lu<7, heap_batch(7)>(a, waves, n_wg, lds_bytes, stream);
}

}  // namespace bridger
