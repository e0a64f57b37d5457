// Integer-only attention from int8 Q and K for long rows (8 to 20 chunks of
// 32 keys, up to 640 keys) on the integer Log-Int-Softmax path, for scales
// outside the float path's bounds (kernels of the float path: lis_qk_kernel.h).
//
// A workgroup of kQkLongWaves wavefronts stages V^T (bf16), K (int8,
// XOR-swizzled as in lis_qk_kernel.h) and each key's zero-point term in LDS.
// The integer path's qL, z of a row of several hundred keys do not fit a lane's
// registers, and its logits cost two MFMAs per 32-key chunk from LDS, so each
// 16-query tile takes the three passes of qk_tile_passes.  The chunk count is a
// run-time value; the last chunk's keys past Lk get P = 0.
#include "lis_qk_kernel.h"

namespace fqvit {
namespace lis {

constexpr int kQkLongBlock = 64 * kQkLongWaves;

// V^T of a whole unit (keys [0, kp), kp a multiple of 32) staged by a workgroup
// of NTHREADS threads, as stage_store does: item = (16-column group, key quad).
template <int DTMAX, int NTHREADS>
__device__ __forceinline__ void long_stage_vt(uint16_t* vt, int ld, const int8_t* vg, int Lk, int d,
                                              int kp, int zp, bool vec_ok) {
    const int nquads = kp / 4;
    const float off = (float)(128 + zp);
    for (int idx = threadIdx.x; idx < nquads * DTMAX; idx += NTHREADS) {
        const int cg = idx / nquads;
        const int jj = 4 * (idx - cg * nquads);
        const int dd = 16 * cg;
        u32x4 w[4];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            w[t] = (dd < d && jj + t < Lk) ? load_v16(vg + (int64_t)(jj + t) * d, dd, d, vec_ok)
                                           : u32x4{0u, 0u, 0u, 0u};
        const int pos = (jj & ~31) + chunk_pos(jj & 31);
#pragma unroll
        for (int t = 0; t < 4; ++t) w[t] ^= 0x80808080u;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            float f[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) f[t] = (float)((w[t][q >> 2] >> (8 * (q & 3))) & 0xFFu) - off;
            *reinterpret_cast<u32x2*>(vt + (16 * cg + q) * ld + pos) =
                u32x2{bf16_pair(f[0], f[1]), bf16_pair(f[2], f[3])};
        }
    }
}

template <int DTMAX, int DK, bool BIAS>
__global__ __launch_bounds__(kQkLongBlock) void lis_qk_long_kernel(LisArgs a, QkArgs qa,
                                                                   LisLaunch p) {
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    const int nc = (a.Lk + 31) >> 5;
    const int kp = 32 * nc;                       // staged keys (zero past Lk)
    uint16_t* vt = reinterpret_cast<uint16_t*>(smem);
    int8_t* kst = reinterpret_cast<int8_t*>(smem + p.vt_bytes);
    int32_t* ck = reinterpret_cast<int32_t*>(smem + p.vt_bytes + kp * DK);
    const int part = (int)blockIdx.y;     // as lis_qk_kernel
    const int64_t g = blockIdx.x;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int r = lane & 15;
    const int kg = lane >> 4;
    const int Lk = a.Lk;

    LisConsts k = a.k;
    k.u_max &= 0xFFFFFFu;
    k.d_ln2 &= 0xFFFFFFu;
    k.magic &= 0xFFFFFFu;

    // V^T, K and the per-key zero-point terms of the unit
    long_stage_vt<DTMAX, kQkLongBlock>(vt, p.ld, a.v + g * (int64_t)Lk * a.d, Lk, a.d, kp, a.zp_v,
                                       p.vec_ok);
    stage_k<DK, kQkLongBlock>(kst, ck, qa.k + g * (int64_t)Lk * DK, Lk, kp, qa.zq);
    __syncthreads();

    const int8_t* q_base = qa.q + g * (int64_t)a.Lq * DK;
    const int32_t* bplane = BIAS ? a.bias + (g % a.Hb) * (int64_t)a.Lq * Lk : nullptr;
    for (int tile = wave + kQkLongWaves * part; tile < p.ntiles; tile += kQkLongWaves * p.split) {
        const int i0 = 16 * tile;
        const int i = min(i0 + r, a.Lq - 1);
        i32x4v qb[DK >= 64 ? DK / 64 : 1];
        int64_t qb8 = 0;
        qb[0] = i32x4v{0, 0, 0, 0};
        qk_load_q<DK>(q_base, i, kg, qb, qb8);
        f32x4 acc[DTMAX];
        qk_tile_passes<DTMAX, DK, BIAS>(acc, kst, ck, vt, p.ld, qb, qb8,
                                        BIAS ? bplane + (int64_t)i * Lk : nullptr, k, nc, Lk, r, kg);
        store_out_t<DTMAX>(acc, a, g, i0, r, kg, p.out_vec);
    }
}

hipError_t launch_qk_long_int(int dk, int dtm, const LisArgs& a, const QkArgs& qa,
                              const LisLaunch& p, size_t lds, hipStream_t stream) {
    const dim3 grid((unsigned)a.G, (unsigned)p.split), block(kQkLongBlock);
#define FQ_QKL(DT, DK)                                                                            \
    do {                                                                                          \
        if (a.bias)                                                                               \
            launch_kernel(lis_qk_long_kernel<DT, DK, true>, grid, block, lds, stream, a, qa, p);  \
        else                                                                                      \
            launch_kernel(lis_qk_long_kernel<DT, DK, false>, grid, block, lds, stream, a, qa, p); \
    } while (0)
    if (dk == 32) {
        if (dtm == 2) FQ_QKL(2, 32);
        else FQ_QKL(4, 32);
    } else {
        if (dtm == 2) FQ_QKL(2, 64);
        else FQ_QKL(4, 64);
    }
#undef FQ_QKL
    return hipGetLastError();
}

}  // namespace lis
}  // namespace fqvit
