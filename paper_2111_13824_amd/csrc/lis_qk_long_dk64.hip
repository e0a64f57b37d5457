// Instantiations of the integer-only attention kernel for long rows (8..20
// chunks of 32 keys, float path) and 64-byte features of Q and K; compiled once
// for each half of the chunk counts (FQ_QK_HI).
#include "lis_qk_kernel.h"

namespace fqvit {
namespace lis {

#ifndef FQ_QK_HI
hipError_t launch_qk_long64_lo(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream) {
    switch (nc) {
        case 8: return launch_qk_nc<64, 8>(dtm, false, fp, a, qa, p, lds, stream);
        case 9: return launch_qk_nc<64, 9>(dtm, false, fp, a, qa, p, lds, stream);
        case 10: return launch_qk_nc<64, 10>(dtm, false, fp, a, qa, p, lds, stream);
        case 11: return launch_qk_nc<64, 11>(dtm, false, fp, a, qa, p, lds, stream);
        case 12: return launch_qk_nc<64, 12>(dtm, false, fp, a, qa, p, lds, stream);
        case 13: return launch_qk_nc<64, 13>(dtm, false, fp, a, qa, p, lds, stream);
        case 14: return launch_qk_nc<64, 14>(dtm, false, fp, a, qa, p, lds, stream);
        default: return hipErrorInvalidValue;
    }
}
#else
hipError_t launch_qk_long64_hi(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream) {
    switch (nc) {
        case 15: return launch_qk_nc<64, 15>(dtm, false, fp, a, qa, p, lds, stream);
        case 16: return launch_qk_nc<64, 16>(dtm, false, fp, a, qa, p, lds, stream);
        case 17: return launch_qk_nc<64, 17>(dtm, false, fp, a, qa, p, lds, stream);
        case 18: return launch_qk_nc<64, 18>(dtm, false, fp, a, qa, p, lds, stream);
        case 19: return launch_qk_nc<64, 19>(dtm, false, fp, a, qa, p, lds, stream);
        case 20: return launch_qk_nc<64, 20>(dtm, false, fp, a, qa, p, lds, stream);
        default: return hipErrorInvalidValue;
    }
}
#endif

}  // namespace lis
}  // namespace fqvit
