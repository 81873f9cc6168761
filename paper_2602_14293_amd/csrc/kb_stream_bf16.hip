// Instantiations for bf16 keys of the scan with the queries in LDS.
#include "kb_stream.hpp"

namespace kbi {

hipError_t launch_stream_bf16(const StreamPlan &p, bool dense, bool once, const StreamArgs &a, hipStream_t s)
{
    return launch_stream<KB_BF16>(p, dense, once, a, s);
}

}  // namespace kbi
