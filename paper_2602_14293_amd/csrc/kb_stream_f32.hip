// Instantiations for f32 keys of the scan with the queries in LDS: as two f16 values an element, and as they are for the calls of which some
// query needs that.
#include "kb_stream.hpp"

namespace kbi {

hipError_t launch_stream_f32(const StreamPlan &p, bool split, bool once, const StreamArgs &a, hipStream_t s)
{
    return split ? launch_stream<KB_F32_SPLIT>(p, false, once, a, s) : launch_stream<KB_F32>(p, false, once, a, s);
}

}  // namespace kbi
