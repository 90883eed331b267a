// The patch analysis of 9x9 patches (see patch_kernel.h).
#include "patch_kernel.h"

namespace cs {

hipError_t launch_patch9(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    return launch_patch_p<9>(lc, a, precision);
}

}  // namespace cs
