// Instantiations for fp8 keys of the scan with the queries in LDS.
#include "kb_stream.hpp"

namespace kbi {

hipError_t launch_stream_fp8(const StreamPlan &p, bool q8, bool dense, bool once, const StreamArgs &a, hipStream_t s)
{
    return q8 ? launch_stream<KB_FP8_Q8>(p, dense, once, a, s) : launch_stream<KB_FP8_E4M3>(p, dense, once, a, s);
}

}  // namespace kbi
