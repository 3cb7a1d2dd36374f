// ragged_heap5.hip -- the padded-heap walk of ragged trees with 5 top levels, 4 trees per batch.
#include "ragged_heap.h"

namespace bridger {

int launch_ragged_heap5(const LaunchArgs &a, int waves, int64_t n_wg, int lds_bytes, void *stream) {
  return launch_heap_lu<5, heap_batch(5)>(a, waves, n_wg, lds_bytes, stream);
}

}  // namespace bridger
