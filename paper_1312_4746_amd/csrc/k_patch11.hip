// The patch analysis of 11x11 patches (see patch_kernel.h).
#include "patch_kernel.h"

namespace cs {

hipError_t launch_patch11(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    return launch_patch_p<11>(lc, a, precision);
}

}  // namespace cs
