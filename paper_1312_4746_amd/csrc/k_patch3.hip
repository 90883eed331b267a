// The patch analysis of 3x3 patches (see patch_kernel.h).
#include "patch_kernel.h"

namespace cs {

hipError_t launch_patch3(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    return launch_patch_p<3>(lc, a, precision);
}

}  // namespace cs
