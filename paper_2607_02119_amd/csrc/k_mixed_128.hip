// K1 for a mixed batch in one launch with 65 to 128 text rows (mixed_tile.h).
#include "mixed_tile.h"

namespace mcd {

hipError_t launch_mixed_text_128(const HeadView &hv, const StepView &sv, hipStream_t st) {
  return launch_mixed_text<128>(hv, sv, st);
}

}  // namespace mcd
