// Test-only stand-ins for the kernel launchers of libfqvit.  The C ABI's host
// code (argument validation, the I-Exp integer constants, the dyadic
// multiplier of the requantization) is linked against these in the CPU
// sanitizer build (tests/test_sanitizers.py), so every entry point can run to
// its launch without a GPU.  Each stub counts its call and launches nothing;
// that of the Log-Int-Softmax kernels keeps the launch it would make
// (tests/launch_plan.py).
#include "fqvit_internal.h"
#include "lis_dispatch.h"

namespace fqvit {

static int g_launches = 0;

hipError_t launch_ptf_layernorm(const LnArgs&, hipStream_t) { ++g_launches; return hipSuccess; }
static lis::LisPlan g_plan;
hipError_t launch_lis(const LisArgs& a, hipStream_t) {
    ++g_launches;
    g_plan = lis::plan_lis(a);
    return hipSuccess;
}
hipError_t launch_lis_qk(const LisArgs&, const QkInput&, hipStream_t) {
    ++g_launches;
    return hipSuccess;
}
hipError_t launch_attn_v_shift(const AvArgs&, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_attn_v_shift_wide(const AvWideArgs&, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_ptf_calibrate(const PtfCalibArgs&, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_ptf_calibrate_noalloc(const PtfCalibArgs& a, hipStream_t) {
    ++g_launches;
    return a.workspace == nullptr ? hipSuccess : hipErrorInvalidValue;
}
hipError_t launch_ptf_quantize(const PtfQuantArgs&, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_requant(const RequantArgs&, hipStream_t) { ++g_launches; return hipSuccess; }

}  // namespace fqvit

extern "C" int fq_test_launch_count(void) { return fqvit::g_launches; }

// The last Log-Int-Softmax launch: kernel (0 unit, 1 tile, 2 stream), chunks of
// a row, V^T column tiles, half last chunk, wavefronts a workgroup, workgroups
// a unit, workgroups, LDS bytes, float path, LDS bytes of gathered code rows.
extern "C" void fq_test_last_plan(long long* out) {
    const fqvit::lis::LisPlan& s = fqvit::g_plan;
    const long long v[10] = {s.kernel, s.nc, s.dt, s.half, s.waves, s.p.split, s.blocks,
                             (long long)s.lds, s.fp, s.p.codes_ldw};
    for (int i = 0; i < 10; ++i) out[i] = v[i];
}
