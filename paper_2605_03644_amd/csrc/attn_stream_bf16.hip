// Streaming attention, bf16 models.
#include "attn_stream_kernel.h"

namespace adapshot {

hipError_t launch_attn_stream_bf16(const StreamLaunch& s, hipStream_t stream) {
    const bool two = s.row_blocks == 2;
    switch (s.head_dim) {
        case 16: return launch_stream_form<ADAPSHOT_BF16, 16, 1>(s, stream);
        case 32: return launch_stream_form<ADAPSHOT_BF16, 32, 1>(s, stream);
        case 64: return two ? launch_stream_form<ADAPSHOT_BF16, 64, 2>(s, stream) : launch_stream_form<ADAPSHOT_BF16, 64, 1>(s, stream);
        case 128: return launch_stream_form<ADAPSHOT_BF16, 128, 1>(s, stream);
        case 256: return launch_stream_form<ADAPSHOT_BF16, 256, 1>(s, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_attn_stream(const StreamLaunch& s, hipStream_t stream) {
    if (s.n_items < 1 || s.n_items > kStreamItems || s.n_wgs < 1) return hipErrorInvalidValue;
    return s.dtype == ADAPSHOT_BF16 ? launch_attn_stream_bf16(s, stream) : launch_attn_stream_f32(s, stream);
}

}  // namespace adapshot
