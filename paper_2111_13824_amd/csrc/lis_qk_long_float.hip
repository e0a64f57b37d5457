// Instantiations of the integer-only attention kernel for long rows (8..20
// chunks of 32 keys, float path); compiled once for each width of Q and K and
// half of the chunk counts (FQ_QK32_LO, FQ_QK32_HI, FQ_QK64_LO, FQ_QK64_HI).
#include "lis_qk_kernel.h"

namespace fqvit {
namespace lis {

#if defined(FQ_QK32_LO)
#define FQ_LAUNCH launch_qk_long32_lo
#elif defined(FQ_QK32_HI)
#define FQ_LAUNCH launch_qk_long32_hi
#elif defined(FQ_QK64_LO)
#define FQ_LAUNCH launch_qk_long64_lo
#elif defined(FQ_QK64_HI)
#define FQ_LAUNCH launch_qk_long64_hi
#endif

#if defined(FQ_QK32_LO) || defined(FQ_QK32_HI)
constexpr int kDk = 32;
#else
constexpr int kDk = 64;
#endif

#define FQ_CASE(NC) \
    case NC: return launch_qk_nc<kDk, NC>(dtm, false, fp, a, qa, p, lds, stream)

hipError_t FQ_LAUNCH(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                     const LisLaunch& p, size_t lds, hipStream_t stream) {
    switch (nc) {
#if defined(FQ_QK32_LO) || defined(FQ_QK64_LO)
        FQ_CASE(8); FQ_CASE(9); FQ_CASE(10); FQ_CASE(11); FQ_CASE(12); FQ_CASE(13); FQ_CASE(14);
#else
        FQ_CASE(15); FQ_CASE(16); FQ_CASE(17); FQ_CASE(18); FQ_CASE(19); FQ_CASE(20);
#endif
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lis
}  // namespace fqvit
