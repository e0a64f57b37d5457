// Integer-only multi-head self-attention from int8 queries and keys on gfx950:
// the MinMax-quantized MatMul of Sec. 3.1 (Q K^T as an integer GEMM) feeding
// Log-Int-Softmax and the BitShift Attn x V of Sec. 3.3 (the dataflow of its
// Fig. 4), with the logits never leaving the chip.
//
// A workgroup per attention unit, or several where the units alone would leave
// CUs idle: V^T is staged once in LDS as bf16, K once as int8 with each key's zero-point
// term, and each wavefront walks the unit's 16-query tiles.  For a tile, its
// queries' bytes are the B operand of v_mfma_i32_16x16x{64,32}_i8 and 16 keys
// of K the A operand, so one MFMA gives S^T for 16 keys x 16 queries with lane
// (query r, group kg) holding keys 4 kg .. 4 kg + 3 of the key tile: two key
// tiles make exactly the 8 keys per 32-key chunk that the Log-Int-Softmax
// code of lis_device.h keeps per lane.  Both operands take contiguous bytes of
// the feature dimension in the same lane order, so the dot product covers
// every feature once whatever order the instruction uses inside a lane group.
//
// With zero points (int8 containers; the 2^(b-1) offset cancels):
//   sum_c (q - zq)(k - zk) = S - zk sum_c q - zq sum_c k + dk zq zk,
// S = sum_c q k from the MFMA; the per-key term zq sum_c k is computed once per
// unit (stored negated) and added to S.  The per-query term dk zq zk - zk
// sum_c q is left out: it is the same for every key of a row, and the
// Log-Int-Softmax of a row depends only on the differences of its logits
// (I-Exp takes max - v).  All sums are exact in int32 (|S| <= dk 255^2 < 2^24
// for dk <= 256).
#pragma once

#include "lis_device.h"

namespace fqvit {
namespace lis {

struct QkArgs {
    const int8_t* q;    // [G, Lq, DK] int8 container
    const int8_t* k;    // [G, Lk, DK] int8 container
    int32_t zq;         // zero point of q, container form
    int32_t zk;         // zero point of k: carried, not used (it cancels, see above)
};

typedef int32_t i32x4v __attribute__((ext_vector_type(4)));

// Rows of up to this many 32-key chunks run both Log-Int-Softmax paths in
// registers; longer rows the float path.
constexpr int kQkRegsNC = 7;

// Byte offset of 16-byte unit u of key j in the staged K (DK bytes per key).
// For DK >= 64 the units are XOR-swizzled with bits 2..3 of the key so that
// the 16 keys read by one lane group fall on distinct LDS banks.
template <int DK>
__device__ __forceinline__ int kst_off(int j, int u) {
    if constexpr (DK >= 64) return j * DK + 16 * (u ^ ((j >> 2) & 3));
    return j * DK + 16 * u;
}

// K of the unit into LDS (keys [0, kp), zeros past Lk), and each key's
// zero-point term -zq sum_c k[j][c] (the initial accumulator of its logits).
// The DK / 16 threads that load a key's 16-byte units are neighbours: their
// partial sums meet by DPP in the same pass.  kp DK / 16 is a multiple of 64,
// so a wavefront is all in or all out.
template <int DK, int NTHREADS>
__device__ __forceinline__ void stage_k(int8_t* kst, int32_t* ck, const int8_t* kg_base, int Lk,
                                        int kp, int zq) {
    static_assert(DK == 32 || DK == 64, "two or four lanes a key");
    for (int w = threadIdx.x; w < kp * (DK / 16); w += NTHREADS) {
        const int j = w / (DK / 16);
        const int u = w - j * (DK / 16);
        i32x4v val = {0, 0, 0, 0};
        if (j < Lk) val = *reinterpret_cast<const i32x4v*>(kg_base + (int64_t)j * DK + 16 * u);
        *reinterpret_cast<i32x4v*>(kst + kst_off<DK>(j, u)) = val;
        int s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) s = __builtin_amdgcn_sdot4(val[q], 0x01010101, s, false);
        s += __builtin_amdgcn_update_dpp(0, s, 0xB1, 0xF, 0xF, false);      // quad_perm 1,0,3,2
        if constexpr (DK == 64)
            s += __builtin_amdgcn_update_dpp(0, s, 0x4E, 0xF, 0xF, false);  // quad_perm 2,3,0,1
        if (u == 0) ck[j] = -(zq * s);
    }
}

// The bias of chunk c's logits in their layout (keys past Lk, which only the
// last chunk holds: 0).
__device__ __forceinline__ void qk_load_bias(i32x4v (&b)[2], const int32_t* brow, int c, int kg,
                                             int Lk, bool last) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int j0 = 32 * c + 16 * h + 4 * kg;
        if (!last) {
            const i32x4a4 v = *reinterpret_cast<const i32x4a4*>(brow + j0);
            b[h] = i32x4v{v.x, v.y, v.z, v.w};
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) b[h][t] = j0 + t < Lk ? brow[j0 + t] : 0;
        }
    }
}

// Logits of chunk c for lane (query r, group kg): keys 32 c + 4 kg + t
// (t < 4) and 32 c + 16 + 4 kg + (t - 4), INT_MIN past Lk (only the last chunk
// holds such keys).  The per-key zero-point terms, with the bias b if there is
// one, are the MFMA's initial accumulator (same layout: lane (r, kg) holds
// keys j0 .. j0 + 3): the logits then stay in the four registers that the MFMA
// writes, where adding the bias to them afterwards scattered them and made
// rows of 13 chunks and more spill.  The per-query term zp_q zp_k dk - zp_k
// sum_c q[i][c] is left out: the Log-Int-Softmax of a row depends only on the
// differences of its logits.  HALF: the last chunk holds at most 16 keys.
template <int DK, bool HALF, bool BIAS>
__device__ __forceinline__ void qk_chunk(int (&lg)[8], const int8_t* kst, const int32_t* ck,
                                         const i32x4v (&qb)[DK >= 64 ? DK / 64 : 1], int64_t qb8,
                                         const i32x4v (&b)[2], int c, int r, int kg, int Lk,
                                         bool last) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        if (HALF && last && h == 1) {
#pragma unroll
            for (int t = 4; t < 8; ++t) lg[t] = INT_MIN;
            continue;
        }
        const int kt = 2 * c + h;
        const int key = 16 * kt + r;          // A operand row of this lane
        const int j0 = 16 * kt + 4 * kg;      // keys of s[0..3]
        i32x4v s = *reinterpret_cast<const i32x4v*>(ck + j0);
        if (BIAS) s += b[h];
        if constexpr (DK >= 64) {
#pragma unroll
            for (int m = 0; m < DK / 64; ++m) {
                const i32x4v av = *reinterpret_cast<const i32x4v*>(kst + kst_off<DK>(key, 4 * m + kg));
                s = __builtin_amdgcn_mfma_i32_16x16x64_i8(av, qb[m], s, 0, 0, 0);
            }
        } else {
            const int64_t av = *reinterpret_cast<const int64_t*>(kst + key * DK + 8 * kg);
            s = __builtin_amdgcn_mfma_i32_16x16x32_i8(av, qb8, s, 0, 0, 0);
        }
        if (!last) {
#pragma unroll
            for (int t = 0; t < 4; ++t) lg[4 * h + t] = s[t];
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) lg[4 * h + t] = j0 + t < Lk ? s[t] : INT_MIN;
        }
    }
}

// The query bytes of row i: the B operand of the logits' MFMA (DK / 4 bytes a
// lane).
template <int DK>
__device__ __forceinline__ void qk_load_q(const int8_t* q_base, int i, int kg,
                                          i32x4v (&dst)[DK >= 64 ? DK / 64 : 1], int64_t& dst8) {
    const int8_t* qrow = q_base + (int64_t)i * DK;
    if constexpr (DK >= 64) {
#pragma unroll
        for (int m = 0; m < DK / 64; ++m)
            dst[m] = *reinterpret_cast<const i32x4v*>(qrow + 64 * m + 16 * kg);
    } else {
        dst8 = *reinterpret_cast<const int64_t*>(qrow + 8 * kg);
    }
}

// One 16-query tile on the integer path in three passes over the keys, the
// logits recomputed in each: the row maximum, the exact I-Exp sum, and the
// codes with the product P V.  The chunk count is a run-time value; masked
// keys get P = 0.
template <int DTMAX, int DK, bool BIAS>
__device__ __forceinline__ void qk_tile_passes(f32x4 (&acc)[DTMAX], const int8_t* kst,
                                               const int32_t* ck, const uint16_t* vt, int ld,
                                               const i32x4v (&qb)[DK >= 64 ? DK / 64 : 1],
                                               int64_t qb8, const int32_t* brow,
                                               const LisConsts& k, int nc, int Lk, int r, int kg) {
    int mx = INT_MIN;
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
        int lg[8];
        i32x4v b[2];
        if (BIAS) qk_load_bias(b, brow, c, kg, Lk, c == nc - 1);
        qk_chunk<DK, false, BIAS>(lg, kst, ck, qb, qb8, b, c, r, kg, Lk, c == nc - 1);
#pragma unroll
        for (int t = 0; t < 8; ++t) mx = max(mx, lg[t]);
    }
    mx = row4_max(mx);

    uint64_t sum = 0;
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
        int lg[8];
        i32x4v b[2];
        if (BIAS) qk_load_bias(b, brow, c, kg, Lk, c == nc - 1);
        qk_chunk<DK, false, BIAS>(lg, kst, ck, qb, qb8, b, c, r, kg, Lk, c == nc - 1);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            uint32_t z;
            const uint32_t qL = iexp_qL(lg[t], mx, k, z);
            sum += lg[t] != INT_MIN ? ((uint64_t)qL << (k.n - (int)z)) : 0ull;
        }
    }
    const RowSum rs = row_sum(sum, k);

    const int ptop = (127 + k.top) << 7;
#pragma unroll
    for (int dt = 0; dt < DTMAX; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int c = 0; c < nc; ++c) {
        int lg[8];
        i32x4v b[2];
        if (BIAS) qk_load_bias(b, brow, c, kg, Lk, c == nc - 1);
        qk_chunk<DK, false, BIAS>(lg, kst, ck, qb, qb8, b, c, r, kg, Lk, c == nc - 1);
        uint32_t pbits[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const bool valid = lg[t] != INT_MIN;
            uint32_t z;
            const uint32_t qL = iexp_qL(valid ? lg[t] : mx, mx, k, z);
            pbits[t] = valid ? (uint32_t)(ptop - (lis_code(qL, z, rs, k) << 7)) : 0u;
        }
        const u32x4 pb = {pbits[0] | (pbits[1] << 16), pbits[2] | (pbits[3] << 16),
                          pbits[4] | (pbits[5] << 16), pbits[6] | (pbits[7] << 16)};
        chunk_mfma<DTMAX, false, true>(acc, pb, vt, ld, c, r, kg);
    }
}

// Adds to acc what the exact codes of the chunks in todo differ by from the
// screened ones, the chunks' logits formed again from K in LDS (rolled loops:
// cold code of long rows, whose unrolled form would be longer than the rest of
// the kernel).
template <int NC, int DTMAX, int DK, bool P0, bool BIAS>
__device__ __forceinline__ void qk_fix_chunks(f32x4 (&acc)[DTMAX], uint32_t todo, const int8_t* kst,
                                              const int32_t* ck, const uint16_t* vt, int ld,
                                              const int8_t* q_base, int i, const int32_t* brow,
                                              const ScreenRow& st, const LisConsts& k, int Lk,
                                              int r, int kg) {
    i32x4v qe[DK >= 64 ? DK / 64 : 1];
    int64_t qe8 = 0;
    qk_load_q<DK>(q_base, i, kg, qe, qe8);
    double part = 0.0;
#pragma unroll 1
    for (int c = 0; c < NC; ++c) {
        int lg[8];
        i32x4v b[2];
        if (BIAS) qk_load_bias(b, brow, c, kg, Lk, c == NC - 1);
        qk_chunk<DK, false, BIAS>(lg, kst, ck, qe, qe8, b, c, r, kg, Lk, c == NC - 1);
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const float e = __uint_as_float(screen_iexp<P0>(lg[t], st.mc, k));
            part += lg[t] != INT_MIN ? (double)e : 0.0;
        }
    }
    const RowState ex = screen_exact(row4_sum(part), k);
#pragma unroll 1
    for (uint32_t m = todo; m != 0; m &= m - 1) {
        const int c = __builtin_ctz(m);
        int lg[8];
        i32x4v b[2];
        if (BIAS) qk_load_bias(b, brow, c, kg, Lk, c == NC - 1);
        qk_chunk<DK, false, BIAS>(lg, kst, ck, qe, qe8, b, c, r, kg, Lk, c == NC - 1);
        chunk_mfma<DTMAX, false, true>(acc, chunk_pbits_diff<P0>(lg, st, ex, k), vt, ld, c, r, kg);
    }
}

// Wavefronts per workgroup: four for rows whose V^T and K leave room for
// several workgroups on a CU; eight for longer rows, whose 8 NC logits a lane
// allow two wavefronts per SIMD anyway (one workgroup of ViT-L's 577 keys takes
// 125 of the CU's 160 KB of LDS).  Holding the logits in registers instead of
// forming them again for the maximum, the sum and the codes: 256 units of 577 x
// 577, dk = d = 64, 148 -> 89 us.
constexpr int qk_waves(int NC) { return NC <= 10 ? 4 : 8; }
constexpr int qk_waves_per_simd(int NC, bool FP) {
    if (!FP && NC == 4) return 4;       // some forms take 131 to 134 registers by themselves
    if (FP && NC == 2) return 6;        // 83 (1536 units of 64 x 64 9.8 us, 9.0 with 80)
    return NC <= 8 ? 3 : 2;
}
constexpr int kQkGroup = 3;     // chunks whose K reads and bias are in flight together

// Workgroup (g, part) does part `part` of unit g: the unit's tiles are dealt to
// the wavefronts of its p.split workgroups in turn, each of which stages V^T and
// K.  (Taken from one index, the two cost two divisions before the first load:
// 3072 units of 16 x 16 7.8 -> 7.4 us.)
// BIAS: the call has a bias.  With both forms of the logits in one kernel, the
// 8 NC registers where the two met were copied and spilled (577 keys, dk = d =
// 64: 352 bytes of scratch a lane, most of it written and read in the tile
// loop).  256 units of 577 x 577, dk = d = 64: 82 -> 68 us, with a bias 142 ->
// 90 us.
template <int NC, int DTMAX, bool HALF, bool FP, int DK, bool P0, bool BIAS>
__global__ __launch_bounds__(64 * qk_waves(NC), qk_waves_per_simd(NC, FP)) void lis_qk_kernel(
    LisArgs a, QkArgs qa, LisLaunch p) {
    constexpr int WAVES = qk_waves(NC);
    constexpr int NTHR = 64 * WAVES;
    constexpr int NT = HALF ? 4 : 8;
    constexpr int KP = 32 * NC;                 // staged keys (zero past Lk)
    // Integer path: a group of chunks at a time, and the next queries' bytes
    // requested at the tile's end.  Not rows of three and four chunks, which then
    // take a few registers more than five and four wavefronts a SIMD leave them
    // (1000 units of 100 x 100 at 2^-12 19.4 us, as it is 17.4); of two chunks, 6144
    // units of 49 x 49 39.3 us without and 37.4 with.
    constexpr bool kTight = !FP && NC != 3 && NC != 4;
    extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
    uint16_t* vt = reinterpret_cast<uint16_t*>(smem);
    int8_t* kst = reinterpret_cast<int8_t*>(smem + p.vt_bytes);
    int32_t* ck = reinterpret_cast<int32_t*>(smem + p.vt_bytes + KP * DK);
    const int part = (int)blockIdx.y;
    const int64_t g = blockIdx.x;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int r = lane & 15;
    const int kg = lane >> 4;

    LisConsts k = a.k;
    k.u_max &= 0xFFFFFFu;
    k.d_ln2 &= 0xFFFFFFu;
    k.magic &= 0xFFFFFFu;

    // V^T and K of the unit into LDS
    StageRegs sr;
    stage_load<NTHR>(sr, a.v + g * (int64_t)a.Lk * a.d, a.Lk, a.d, DTMAX, 0, KP, a.zp_v, p.vec_ok);
    const int8_t* kg_base = qa.k + g * (int64_t)a.Lk * DK;
    stage_k<DK, NTHR>(kst, ck, kg_base, a.Lk, KP, qa.zq);
    stage_store<NTHR>(sr, vt, p.ld, DTMAX, KP, a.zp_v);
    __syncthreads();

    const int8_t* q_base = qa.q + g * (int64_t)a.Lq * DK;
    const int32_t* bplane = BIAS ? a.bias + (g % a.Hb) * (int64_t)a.Lq * a.Lk : nullptr;

    i32x4v qb[DK >= 64 ? DK / 64 : 1];
    int64_t qb8 = 0;
    const int step = WAVES * p.split;
    int tile = wave + WAVES * part + (int)(g & 3);
    tile = tile < step ? tile : tile - step;
    if (tile < p.ntiles) qk_load_q<DK>(q_base, min(16 * tile + r, a.Lq - 1), kg, qb, qb8);
    for (; tile < p.ntiles; tile += step) {
        const int i0 = 16 * tile;
        const int i = min(i0 + r, a.Lq - 1);

        // Logits of this tile in the Log-Int-Softmax lane layout, kQkGroup chunks
        // at a time: a few chunks' K reads in flight, not all, and the bias of
        // the next group requested before this one waits for its own.
        int lg[NC][8];
        i32x4v bias[2][kQkGroup][2];
        const int32_t* brow = BIAS ? bplane + (int64_t)i * a.Lk : nullptr;
        auto request = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kQkGroup; ++u)
                if (BIAS && c0 + u < NC)
                    qk_load_bias(bias[c0 / kQkGroup % 2][u], brow, c0 + u, kg, a.Lk, c0 + u == NC - 1);
        };
        request(0);
#pragma unroll
        for (int c0 = 0; c0 < NC; c0 += kQkGroup) {
            request(c0 + kQkGroup);
#pragma unroll
            for (int u = 0; u < kQkGroup; ++u) {
                const int c = c0 + u;
                if (c < NC)
                    qk_chunk<DK, HALF, BIAS>(lg[c], kst, ck, qb, qb8, bias[c0 / kQkGroup % 2][u], c, r, kg,
                                             a.Lk, c == NC - 1);
            }
            if (NC > kQkRegsNC || kTight) __builtin_amdgcn_sched_barrier(0);
        }
        // the next tile's query bytes, in flight during the rest of this tile
        // (kTight: requested at its end, where its registers are free)
        const int nt = min(16 * (tile + step < p.ntiles ? tile + step : tile) + r, a.Lq - 1);
        if (!kTight) qk_load_q<DK>(q_base, nt, kg, qb, qb8);
        f32x4 acc[DTMAX];
#pragma unroll
        for (int dt = 0; dt < DTMAX; ++dt) acc[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (FP) {
            double S;
            const ScreenRow st = tile_iexp_screen<NC, NT, false, P0>(lg, k, S);
            uint32_t todo = 0;      // undecided chunks (long rows)
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                bool undecided;
                u32x4 pb = chunk_pbits_screen<NC, NT, (NC > kQkRegsNC)>(lg, st, c, undecided);
                if constexpr (NC <= kQkRegsNC) {
                    if (__builtin_expect(undecided, 0))
                        pb = chunk_pbits_exact(lg[c], screen_sum<NC, NT>(lg), k);
                } else {
                    todo |= undecided ? 1u << c : 0u;
                }
                if (HALF && c == NC - 1)
                    chunk_mfma<DTMAX, true, true>(acc, pb, vt, p.ld, c, r, kg);
                else
                    chunk_mfma<DTMAX, false, true>(acc, pb, vt, p.ld, c, r, kg);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (NC > kQkRegsNC) {
                if (__builtin_expect(todo != 0, 0))
                    qk_fix_chunks<NC, DTMAX, DK, P0, BIAS>(acc, todo, kst, ck, vt, p.ld, q_base, i,
                                                     BIAS ? bplane + (int64_t)i * a.Lk : nullptr, st,
                                                     k, a.Lk, r, kg);
            }
        } else {
            uint32_t zb[NC][2];
            const RowState st = tile_iexp<NC, FP, NT>(lg, zb, k);
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                const u32x4 pb = chunk_pbits<NC, FP, NT>(lg, zb, st, k, c);
                if (HALF && c == NC - 1)
                    chunk_mfma<DTMAX, true, true>(acc, pb, vt, p.ld, c, r, kg);
                else
                    chunk_mfma<DTMAX, false, true>(acc, pb, vt, p.ld, c, r, kg);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (kTight) qk_load_q<DK>(q_base, nt, kg, qb, qb8);
        store_out_t<DTMAX>(acc, a, g, i0, r, kg, p.out_vec);
    }
}

// fpm: 0 the integer path, 1 the float path, 2 the float path with the
// I-Exp pre-shift 0.  Rows of more than kQkRegsNC chunks: the float path only
// (half: as a full last chunk).
template <int DK, int NC>
hipError_t launch_qk_nc(int dtm, bool half, int fpm, const LisArgs& a, const QkArgs& qa,
                        const LisLaunch& p, size_t lds, hipStream_t stream) {
    const dim3 grid((unsigned)a.G, (unsigned)p.split), block(64 * qk_waves(NC));
#define FQ_QK(DT, H, F, P0)                                                                   \
    do {                                                                                          \
        if (a.bias)                                                                               \
            launch_kernel(lis_qk_kernel<NC, DT, H, F, DK, P0, true>, grid, block, lds, stream, a, qa, p);  \
        else                                                                                      \
            launch_kernel(lis_qk_kernel<NC, DT, H, F, DK, P0, false>, grid, block, lds, stream, a, qa, p); \
    } while (0)
#define FQ_QK_F(DT, H)                          \
    if (fpm == 2) FQ_QK(DT, H, true, true);     \
    else FQ_QK(DT, H, true, false)
    if constexpr (NC > kQkRegsNC) {
        if (dtm == 2) { FQ_QK_F(2, false); }
        else { FQ_QK_F(4, false); }
    } else {
#define FQ_QK_H(DT, H) \
    if (fpm == 0) FQ_QK(DT, H, false, false); else FQ_QK_F(DT, H)
        if (dtm == 2) {
            if (half) { FQ_QK_H(2, true); } else { FQ_QK_H(2, false); }
        } else {
            if (half) { FQ_QK_H(4, true); } else { FQ_QK_H(4, false); }
        }
#undef FQ_QK_H
    }
#undef FQ_QK_F
#undef FQ_QK
    return hipGetLastError();
}

template <int DK>
hipError_t launch_qk_dk(int nc, int dtm, bool half, int fp, const LisArgs& a, const QkArgs& qa,
                        const LisLaunch& p, size_t lds, hipStream_t stream) {
    switch (nc) {
        case 1: return launch_qk_nc<DK, 1>(dtm, half, fp, a, qa, p, lds, stream);
        case 2: return launch_qk_nc<DK, 2>(dtm, half, fp, a, qa, p, lds, stream);
        case 3: return launch_qk_nc<DK, 3>(dtm, half, fp, a, qa, p, lds, stream);
        case 4: return launch_qk_nc<DK, 4>(dtm, half, fp, a, qa, p, lds, stream);
        case 5: return launch_qk_nc<DK, 5>(dtm, half, fp, a, qa, p, lds, stream);
        case 6: return launch_qk_nc<DK, 6>(dtm, half, fp, a, qa, p, lds, stream);
        case 7: return launch_qk_nc<DK, 7>(dtm, half, fp, a, qa, p, lds, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_qk_dk32(int nc, int dtm, bool half, int fp, const LisArgs& a, const QkArgs& qa,
                          const LisLaunch& p, size_t lds, hipStream_t stream);
// Rows of 8 to 20 chunks: the float path (lis_qk_long_float.hip,
// 8..14 and 15..20 chunks), and the integer path, which
// takes the three passes of qk_tile_passes (lis_qk_long.hip).
hipError_t launch_qk_long32_lo(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream);
hipError_t launch_qk_long32_hi(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream);
hipError_t launch_qk_long64_lo(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream);
hipError_t launch_qk_long64_hi(int nc, int dtm, int fp, const LisArgs& a, const QkArgs& qa,
                               const LisLaunch& p, size_t lds, hipStream_t stream);
hipError_t launch_qk_long_int(int dk, int dtm, const LisArgs& a, const QkArgs& qa,
                              const LisLaunch& p, size_t lds, hipStream_t stream);
constexpr int kQkLongWaves = 12;     // integer path: wavefronts per workgroup
hipError_t launch_qk_dk64(int nc, int dtm, bool half, int fp, const LisArgs& a, const QkArgs& qa,
                          const LisLaunch& p, size_t lds, hipStream_t stream);

}  // namespace lis
}  // namespace fqvit
