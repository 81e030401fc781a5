// Weight-streaming grouped GEMM: the e2m1 instantiations of qgemm_stream_fp8.hpp, in a source of their own so that the two are
// compiled side by side.
#include "qgemm_stream_fp8.hpp"

namespace qarl {

namespace stream8 {

int launch_fp4(const StreamParams &p, int epilogue, int MT, hipStream_t s) { return launch_codes<true>(p, epilogue, MT, s); }

}  // namespace stream8

}  // namespace qarl
