// Decode kernels with the fp32 MFMA MLP (BCF_FP32 and BCF_FP32_MFMA).
#include "frame_kernels.hpp"

namespace bcf {

hipError_t launch_frame_f32(const FrameArgs &a, const MlpShape &sh, int layout, hipStream_t s)
{
    switch (layout) {
    case kLayoutPacked: return launch_frame_kind<MLP_MFMA_F32, kLayoutPacked>(a, sh, s);
    case kLayoutShared: return launch_frame_kind<MLP_MFMA_F32, kLayoutShared>(a, sh, s);
    default: return launch_frame_kind<MLP_MFMA_F32, kLayoutSplit>(a, sh, s);
    }
}

hipError_t launch_batch_f32(const BatchArgs &a, const MlpShape &sh, unsigned grid, uint32_t waves, hipStream_t s)
{
    return launch_batch_kind<MLP_MFMA_F32>(a, sh, grid, waves, s);
}

}  // namespace bcf
