// Instantiations of the Log-Int-Softmax unit kernel for rows of 8..20
// chunks of 32 keys; compiled once for each half of the chunk counts
// (FQ_UNIT_HI).
#include "lis_device.h"

namespace fqvit {
namespace lis {

static_assert(kUnitMaxNC == 20, "instantiated chunk counts");

#define FQ_CASE(NC) \
    case NC: return launch_unit_nc<NC>(fused, dtm, false, unit_long_waves(NC), a, p, lds, stream)

#ifndef FQ_UNIT_HI
hipError_t launch_lis_unit_lo(int nc, bool fused, int dtm, const LisArgs& a, const LisLaunch& p,
                              size_t lds, hipStream_t stream) {
    switch (nc) {
        FQ_CASE(8); FQ_CASE(9); FQ_CASE(10); FQ_CASE(11); FQ_CASE(12); FQ_CASE(13); FQ_CASE(14);
        default: return hipErrorInvalidValue;
    }
}
#else
hipError_t launch_lis_unit_hi(int nc, bool fused, int dtm, const LisArgs& a, const LisLaunch& p,
                              size_t lds, hipStream_t stream) {
    switch (nc) {
        FQ_CASE(15); FQ_CASE(16); FQ_CASE(17); FQ_CASE(18); FQ_CASE(19); FQ_CASE(20);
        default: return hipErrorInvalidValue;
    }
}
#endif

}  // namespace lis
}  // namespace fqvit
