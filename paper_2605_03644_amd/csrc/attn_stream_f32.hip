// Streaming attention, fp32 models (one translation unit per element type, so that they compile side by side).
#include "attn_stream_kernel.h"

namespace adapshot {

hipError_t launch_attn_stream_f32(const StreamLaunch& s, hipStream_t stream) {
    const bool two = s.row_blocks == 2;
    switch (s.head_dim) {
        case 8: return launch_stream_form<ADAPSHOT_F32, 8, 1>(s, stream);
        case 16: return launch_stream_form<ADAPSHOT_F32, 16, 1>(s, stream);
        case 32: return launch_stream_form<ADAPSHOT_F32, 32, 1>(s, stream);
        case 64: return two ? launch_stream_form<ADAPSHOT_F32, 64, 2>(s, stream) : launch_stream_form<ADAPSHOT_F32, 64, 1>(s, stream);
        case 128: return launch_stream_form<ADAPSHOT_F32, 128, 1>(s, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace adapshot
