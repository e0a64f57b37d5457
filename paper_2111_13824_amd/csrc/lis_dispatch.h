// Launch selection of the Log-Int-Softmax kernels (codes and fused head): which
// kernel a call takes, with how many wavefronts and workgroups, and its LDS.
// Host code without a HIP call, so that a test can ask it what a call reaches.
#pragma once

#include <algorithm>

#include "fqvit_internal.h"

namespace fqvit {
namespace lis {

constexpr int kBlock = 256;             // four wavefronts
constexpr int kRowsPerBlock = 64;       // 16 rows per wavefront in the tile kernel
constexpr size_t kMaxLds = 160 * 1024;  // of a CU and of a workgroup on gfx950
constexpr int kSimds = 1024;            // 256 CUs of four SIMDs

constexpr int kUnitShortNC = 7;     // unit kernel: rows instantiated with half last chunks
constexpr int kUnitMaxNC = 20;      // unit kernel: longest rows, in 32-key chunks
// Longest rows of the fused tile kernels, which hold a row in registers on
// the integer path too.  Beyond 9 chunks that path is faster in the stream
// kernel, which reads the logits again instead (d = 64, 64 square units: 300
// keys 30 against 36 us, 384 keys 41 against 61 us; 288 keys 29 against 15 us).
constexpr int kRegsFusedMaxNC = 9;

// LDS dwords of an undecided chunk's keys and the row sums (64 x 8 + 64 x 2).
constexpr int kScreenLds = 640;

// The fused unit kernel's LDS per wavefront: its output block (16 rows of
// 16 dtm + 4 dwords), or kScreenLds dwords where that is more.
constexpr int unit_lds_dwords(int dtm) {
    return 16 * (16 * dtm + 4) > kScreenLds ? 16 * (16 * dtm + 4) : kScreenLds;
}

// Keys of V^T per LDS stage for a padded head dimension dpad: at most 40 KB of
// LDS per workgroup so that several workgroups share a CU.
constexpr int vt_stage_keys(int dpad) { return (40960 / (2 * dpad) - 8) / 32 * 32; }

// Wavefronts per workgroup of rows of more than four chunks: up to 10 chunks
// several workgroups share a CU's LDS, beyond one takes it (V^T of 577 keys and
// d = 64: 79 KB).
constexpr int unit_long_waves(int nc) { return nc <= 10 ? 4 : 8; }

// Wavefronts per workgroup of the unit kernel: units of at most four 16-row
// tiles (and rows of at most four chunks, whose V^T 64 threads can stage) get
// one wavefront per tile up to two, so that the per-wavefront set-up serves
// several tiles.  Measured on Swin-S (6144 units of 49 x 49, d = 32): two
// wavefronts per unit 41.4 us, one 43.7 us, four 46.6-47.3 us.
inline int unit_waves(int nc, int tiles16) {
    if (nc > 4 || tiles16 > 4) return unit_long_waves(nc);
    return tiles16 == 1 ? 1 : 2;
}

// Kernel arguments that follow from the selection.
struct LisLaunch {
    int ntiles;     // tile kernel: row tiles of 64 per unit; unit kernel: 16-row tiles per unit
    int kb;         // keys per V^T stage (multiple of 32)
    int ld;         // LDS row stride of V^T in bf16 elements
    int dpad;       // 16 * (power of two >= ceil(d / 16))
    int ncg;        // dpad / 16: 16-column groups of V
    int vec_ok;     // V rows read as 16-byte vectors (d % 16 == 0, 16-byte aligned V)
    int vt_bytes;   // LDS bytes of one V^T stage (0 for codes only)
    int out_vec;    // output rows written through LDS as 16-byte units (d % 4 == 0, aligned out)
    int64_t n_logits;  // elements of the logits tensor (G Lq Lk)
    int64_t n_bias;    // elements of the bias tensor (Hb Lq Lk), 0 without bias
    int split;         // workgroups per unit (unit and Q K kernels)
    int codes_ldw;     // unit kernel, codes only: LDS bytes per wavefront of the tile's
                       // code rows (dense rows, ld_codes = row bytes), 0: direct stores
};

struct LisPlan {
    enum Kernel { kUnit, kTile, kStream } kernel;
    bool fused;         // with the product (else codes only)
    bool fp;            // float path
    int nc;             // 32-key chunks of a row
    int dt;             // V^T columns / 16 (a power of two, at least 2)
    bool half;          // the last chunk holds at most 16 keys
    int waves;          // wavefronts per workgroup
    int64_t blocks;     // workgroups
    size_t lds;         // dynamic LDS per workgroup
    LisLaunch p;
};

// Workgroups per unit of the fused unit kernel for G units of `tiles` tiles: as
// many as fill the workgroup slots of 256 CUs (by LDS, and three wavefronts a
// SIMD), at most one tile a wavefront, and no more than the tiles that leaves
// each wavefront need.  Each stages V^T.  Measured against one: 6 units of 577 x
// 577, d = 48, 85 -> 24 us; 30 of them with a bias 122 -> 36 us.  Against the
// tile kernel wherever this leaves one tile a wavefront, as the rule was: 2048
// units of 1 x 64 8.8 -> 4.0 us, 2900 of 16 x 16 9.8 -> 4.9, 512 of 60 x 197 12.2
// -> 9.2, 144 of 64 x 256 9.2 -> 7.6, 48 of 197 x 197 7.8 -> 7.5 us; over 16 x 16
// to 288 x 288 and 1 to 6000 units the tile kernel was never more than 6 %
// faster, and that for two sizes.
inline int unit_split(int64_t G, int tiles, int waves, int nc, size_t lds) {
    const int64_t most = (tiles + waves - 1) / waves;
    const int64_t slots =
        256 * std::max<int64_t>(1, std::min<int64_t>(12 / waves, kMaxLds / std::max<size_t>(lds, 1)));
    // workgroups per unit that leave a wavefront t tiles
    auto split_of = [&](int64_t t) { return (tiles + waves * t - 1) / (waves * t); };
    const int64_t fill = std::max<int64_t>(1, std::min<int64_t>(most, slots / G));
    const int64_t even = split_of((tiles + waves * fill - 1) / (waves * fill));
    if (fill > 1 && (nc == 9 || nc == 10)) {
        // Rows of 257 to 320 keys, divided: the CUs that get a workgroup more
        // than the others end last, so a unit's load is its workgroups a CU,
        // rounded up, times the tiles a wavefront and the staging (0.6 of a
        // tile), and 1.3 times that where a SIMD has one wavefront and nothing
        // to run while it waits.  Over 100 to 350 units of 257 to 320 keys this
        // is within 8 % of the best division (200 units of 288 x 288 29.1 us by
        // `even`, 27.7 by this; 180 of 300 x 300 with a bias 29.9 and 26.1).
        auto cost = [&](int64_t split) {
            const int64_t load = (G * split + 255) / 256;
            return (double)load * ((double)((tiles + waves * split - 1) / (waves * split)) + 0.6) *
                   (load == 1 ? 1.3 : 1.0);
        };
        int64_t best = even;
        for (int64_t t = 1; t <= most; ++t)
            if (cost(split_of(t)) < cost(best)) best = split_of(t);
        return (int)best;
    }
    if (fill > 1 || nc < 8 || nc > 9) return (int)even;
    // Rows of 225 to 288 keys, more units than half the slots: the SIMDs that
    // get a wavefront more than the others end last, so the load of one is its
    // wavefronts, rounded up, times the tiles each walks and the staging (0.4 of
    // a tile).  300 units of 288 x 288 38.6 us undivided and 33.5 divided, 520 of
    // 257 x 257 with a bias 84 and 70; 768 of 257 x 257 56 and 73, 400 37.4 and 40.7.
    auto cost = [&](int64_t split) {
        const int64_t load = (G * split * waves + kSimds - 1) / kSimds;
        return (double)load * ((double)((tiles + waves * split - 1) / (waves * split)) + 0.4);
    };
    int64_t best = 1;
    for (int64_t t = std::min<int64_t>(8, most); t >= 1; --t)
        if (cost(split_of(t)) < cost(best)) best = split_of(t);
    return (int)best;
}

// Few tiles, with a partial last chunk: the tile kernel, which stores the codes'
// bytes from the registers, is up to 15 % faster than gathering the rows in LDS
// as long as the wavefronts have the SIMDs (nearly) to themselves: nibble codes
// of up to 288 keys in at most one tile a SIMD (256 units of 49 x 100 4.4 against
// 5.0 us, 96 of 113 x 113 4.2 and 4.9; with full last chunks 192 of 64 x 128 5.9
// against 4.8, and units of a few rows 1024 of 1 x 197 8.0 against 7.1), and
// windows of 49 keys in up to 2.75 (700 of 49 x 49 4.9 against 5.6; 8-bit codes
// 5.2 and 6.0).  Other byte codes store four times the bytes: never (768 x 197 x
// 197 62 against 41 us).
inline bool codes_tile_kernel(int64_t G, int Lq, int nc, int Lk, bool bytes) {
    const int tiles = (Lq + 15) / 16;
    const int64_t most = nc <= 2 && tiles >= 4 ? 2816 : bytes ? 0 : kSimds;
    return nc <= 9 && Lk % 32 != 0 && Lq > 8 && G * tiles > 256 && G * tiles <= most;
}

inline LisPlan plan_lis(const LisArgs& a) {
    LisPlan s{};
    LisLaunch& p = s.p;
    s.fused = a.out != nullptr;
    s.fp = a.k.fp_ok != 0;
    s.nc = (a.Lk + 31) / 32;
    s.half = a.Lk - 32 * (s.nc - 1) <= 16;
    p.ntiles = (a.Lq + kRowsPerBlock - 1) / kRowsPerBlock;
    // V^T columns padded to a power of two, at least 32 (two MFMA tiles).
    s.dt = 2;
    while (s.fused && 16 * s.dt < a.d) s.dt <<= 1;
    p.dpad = 16 * s.dt;
    p.ncg = s.dt;
    p.kb = std::max(32, std::min(s.nc * 32, vt_stage_keys(p.dpad)));
    p.ld = p.kb + 8;
    p.vec_ok = s.fused && (a.d % 16 == 0) && ((reinterpret_cast<uintptr_t>(a.v) & 15) == 0);
    p.vt_bytes = s.fused ? p.dpad * p.ld * (int)sizeof(uint16_t) : 0;
    p.out_vec = s.fused && (a.d % 4 == 0) && ((reinterpret_cast<uintptr_t>(a.out) & 15) == 0);
    p.n_logits = a.G * (int64_t)a.Lq * a.Lk;
    p.n_bias = a.bias ? (int64_t)a.Hb * a.Lq * a.Lk : 0;
    p.split = 1;
    p.codes_ldw = 0;
    s.waves = kBlock / 64;
    s.blocks = a.G * (int64_t)p.ntiles;

    // Unit kernel: rows of up to 640 keys on the float path, planes of less
    // than 2^31 bytes; the fused product for d <= 64 and no codes output; codes
    // only of more than 224 keys for dense code rows.
    const int tiles16 = (a.Lq + 15) / 16;
    const int row_bytes = a.k.top > 15 ? a.Lk : (a.Lk + 1) / 2;
    const bool dense = !s.fused && a.ld_codes == row_bytes;
    const bool unit_ok = s.fp && a.G <= 0x7FFFFFFF && (int64_t)a.Lq * a.Lk < ((int64_t)1 << 29) &&
                         s.nc <= kUnitMaxNC &&
                         (s.fused ? a.codes == nullptr && s.dt <= 4 : dense || s.nc <= kUnitShortNC);
    if (unit_ok) {
        LisLaunch u = p;
        u.ntiles = tiles16;
        u.kb = s.nc * 32;
        u.ld = u.kb + 8;
        u.vt_bytes = s.fused ? u.dpad * u.ld * (int)sizeof(uint16_t) : 0;
        const int waves = s.fused ? unit_waves(s.nc, tiles16) : 1;
        const size_t wave_lds = (size_t)(s.fused ? unit_lds_dwords(s.dt) : kScreenLds) * sizeof(int32_t);
        size_t lds = (size_t)u.vt_bytes + wave_lds * waves;
        // codes only, dense rows: each wavefront gathers its tile's code rows
        // in LDS and writes them as one span
        if (dense) {
            u.codes_ldw = (16 * row_bytes + 8 + 15) / 16 * 16;
            lds += (size_t)waves * u.codes_ldw;
        }
        // Codes only: nothing is shared between a unit's tiles, so a workgroup
        // is one wavefront with one tile (several beyond the grid's limit).
        // Against workgroups of eight wavefronts for rows of more than 320 keys
        // and two or four below, several tiles each: 3000 units of 16 x 577
        // 138 -> 42 us, 300 of 400 x 400 75 -> 46, 144 of 325 x 325 33 -> 22, and
        // 8-bit codes of 768 x 197 x 197 unchanged.
        u.split = std::min(s.fused ? unit_split(a.G, tiles16, waves, s.nc, lds) : tiles16, 65535);
        if (s.fused || !codes_tile_kernel(a.G, a.Lq, s.nc, a.Lk, a.k.top > 15)) {
            s.kernel = LisPlan::kUnit;
            s.p = u;
            s.waves = waves;
            s.blocks = a.G * u.split;
            s.lds = lds;
            return s;
        }
    }
    // Tile kernels: codes only for rows of up to 640 keys, the fused product
    // (without a codes output, d <= 64) for rows of up to 288: on the integer
    // path, and of planes too large for the unit kernel.
    if (s.fused ? s.nc <= kRegsFusedMaxNC && a.codes == nullptr && s.dt <= 4 : s.nc <= 20) {
        s.kernel = LisPlan::kTile;
        // with the row-wise output stores: one 16 x (dpad + 4) int32 block per wavefront
        s.lds = (size_t)p.vt_bytes +
                (p.out_vec ? (size_t)4 * 16 * (p.dpad + 4) * sizeof(int32_t) : 0);
        return s;
    }
    s.kernel = LisPlan::kStream;
    s.lds = (size_t)p.vt_bytes;
    return s;
}

}  // namespace lis
}  // namespace fqvit
