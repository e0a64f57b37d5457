// Host side of the integer-only attention from int8 Q and K (kernels in
// lis_qk_kernel.h and lis_qk_long.hip): launch geometry and LDS.
#include <algorithm>

#include "lis_qk_kernel.h"

namespace fqvit {

constexpr size_t kQkLds = 160 * 1024;     // LDS of a CU

hipError_t launch_lis_qk(const LisArgs& a, const QkInput& in, hipStream_t stream) {
    using namespace lis;
    const int nc = (a.Lk + 31) / 32;
    int dt = 2;
    while (16 * dt < a.d) dt <<= 1;
    LisLaunch p{};
    p.ntiles = (a.Lq + 15) / 16;
    p.dpad = 16 * dt;
    p.ncg = dt;
    p.kb = 32 * nc;
    p.ld = p.kb + 8;
    p.vec_ok = (a.d % 16 == 0) && ((reinterpret_cast<uintptr_t>(a.v) & 15) == 0);
    p.vt_bytes = p.dpad * p.ld * (int)sizeof(uint16_t);
    // output rows as 16-byte units (d % 4 == 0 and a 16-byte aligned out)
    p.out_vec = (a.d % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.out) & 15) == 0);
    p.n_logits = 0;
    p.n_bias = a.bias ? (int64_t)a.Hb * a.Lq * a.Lk : 0;
    const size_t lds = (size_t)p.vt_bytes + (size_t)32 * nc * in.dk + (size_t)32 * nc * sizeof(int32_t);
    const bool half = a.Lk - 32 * (nc - 1) <= 16;
    // float path (and its I-Exp without the pre-shift where that is 0) or the
    // integer path
    const int fp = a.k.fp_ok != 0 ? (a.k.s_pre == 0 ? 2 : 1) : 0;
    const QkArgs qa{in.q, in.k, in.zp_q, in.zp_k};
    // Workgroups per unit.  A workgroup's time is its staging plus its
    // wavefronts' tiles one after the other, so where the units alone do not
    // fill the workgroup slots of 256 CUs (by LDS), a unit is dealt to as many
    // as do, at most one tile a wavefront.  Measured on one MI355X: 75 units of
    // 197 x 197, dk = d = 32 (with the requantization) 20.7 us undivided, 13.0
    // us divided; one DeiT-T block (LayerNorm, 3 units of 197 x 197,
    // requantization) 22.0 and 13.6 us; 24 units of 577 x 577 on the integer
    // path 205 and 78 us.
    const bool lng = nc > kQkRegsNC;
    const int waves = lng && fp == 0 ? kQkLongWaves : qk_waves(nc);
    const int64_t slots = 256 * std::max<int64_t>(1, std::min<int64_t>(12 / waves, kQkLds / lds));
    const int64_t most = (p.ntiles + waves - 1) / waves;
    p.split = (int)std::max<int64_t>(1, std::min<int64_t>(most, slots / a.G));
    if (lng && fp == 0) return launch_qk_long_int(in.dk, dt, a, qa, p, lds, stream);
    if (lng && in.dk == 32)
        return nc <= 14 ? launch_qk_long32_lo(nc, dt, fp, a, qa, p, lds, stream)
                        : launch_qk_long32_hi(nc, dt, fp, a, qa, p, lds, stream);
    if (lng)
        return nc <= 14 ? launch_qk_long64_lo(nc, dt, fp, a, qa, p, lds, stream)
                        : launch_qk_long64_hi(nc, dt, fp, a, qa, p, lds, stream);
    if (in.dk == 32) return launch_qk_dk32(nc, dt, half, fp, a, qa, p, lds, stream);
    return launch_qk_dk64(nc, dt, half, fp, a, qa, p, lds, stream);
}

}  // namespace fqvit
