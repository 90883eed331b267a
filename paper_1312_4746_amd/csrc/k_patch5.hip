// The patch analysis of 5x5 patches (see patch_kernel.h).
#include "patch_kernel.h"

namespace cs {

hipError_t launch_patch5(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    return launch_patch_p<5>(lc, a, precision);
}

}  // namespace cs
