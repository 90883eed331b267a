// The patch analysis of 7x7 patches (see patch_kernel.h).
#include "patch_kernel.h"

namespace cs {

hipError_t launch_patch7(const LaunchCtx &lc, const AnalyzeArgs &a, int precision) {
    return launch_patch_p<7>(lc, a, precision);
}

}  // namespace cs
