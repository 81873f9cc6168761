// Instantiations for f32 keys (two f16 values an element) of the scan with the queries in LDS.
#include "kb_stream.hpp"

namespace kbi {

hipError_t launch_stream_f32(const StreamPlan &p, bool dense, bool once, const StreamArgs &a, hipStream_t s)
{
    return launch_stream<KB_F32_SPLIT>(p, dense, once, a, s);
}

}  // namespace kbi
