// The kernel of nadmm_thin.h for rows whose stride is no multiple of 4.
#include "nadmm_thin.h"

namespace nadmm {

hipError_t launch_thin_block(const ThinArgs& ta, int grid, hipStream_t st) { return launch_thin_rows<kBlock>(ta, grid, st); }

}  // namespace nadmm
