// K1 for a mixed batch in one launch with 33 to 64 text rows (mixed_tile.h).
#include "mixed_tile.h"

namespace mcd {

hipError_t launch_mixed_text_64(const HeadView &hv, const StepView &sv, hipStream_t st) {
  return launch_mixed_text<64>(hv, sv, st);
}

}  // namespace mcd
