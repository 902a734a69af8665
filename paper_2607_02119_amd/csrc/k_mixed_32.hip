// K1 for a mixed batch in one launch with at most 32 text rows (mixed_tile.h).
#include "mixed_tile.h"

namespace mcd {

hipError_t launch_mixed_text_32(const HeadView &hv, const StepView &sv, hipStream_t st) {
  return launch_mixed_text<32>(hv, sv, st);
}

}  // namespace mcd
