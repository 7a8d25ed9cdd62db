// The one-launch forward for subsampling s = 3 (its own file: the bodies compile side by side).
#include "starred_frame.h"

namespace starred {

hipError_t launch_frames_s3(hipStream_t st, const FftPlanDev &d, const FrameArgs &g, const DensePiece &dp, size_t lds)
{
    return launch_frames<3>(st, d, g, dp, lds);
}

}  // namespace starred
