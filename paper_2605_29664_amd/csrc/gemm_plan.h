// Choice of tile and of the number of parts of the contraction for a plain
// product on gemm_mfma_dl_kernel. Host only.
#pragma once
#include <algorithm>
#include <cstddef>

namespace amdp {

enum DlTileId { DL_256, DL_256x128, DL_128, DL_128_PAIR, DL_64_DEEP, DL_64, DL_TILES };

// The estimate below is a model of the launch in microseconds, with constants fitted to
// measurements on MI355X (192 products of stages from d_model 128 to 4096 with 400 to
// 8192 tokens, operands not cache-resident; every tile on every product). It is within
// 10 % of a tile's own time, and the tile it picks is on average 1 % slower than the
// fastest of all measured ones (worst 1.27x, where the output's memory time dominates).
//   per_cu   workgroups of the tile that share a compute unit
//   launch   launch and first loads
//   round    per round of workgroups: what does not depend on the contraction
//   heavy    added to it when the output is fp32 or the epilogue reads or writes a second matrix
//   ktile    one k-tile (64) with one workgroup on the unit
//   share    added per further workgroup on the unit
// Why six: the 256x256 tile moves the least data per flop and wins wherever it fills the
// GPU; 256x128 has twice the tiles at 1.3 times the time per flop and wins where 256x256
// leaves part of a round idle ([2048, 4096] outputs: 65 against 80 us); 128x128 runs as
// one eight-wave workgroup per unit with three tiles in LDS ([4096, 1024] outputs, 43
// against 55 us) or as two four-wave workgroups (short contractions, several rounds);
// 64x64 is for outputs too small for those, with four tiles in LDS while at most two
// workgroups share a unit (latency: 512x512x4096, 15 against 25 us) and two beyond.
struct DlTileModel { int bm, bn, per_cu; double launch, round, heavy, ktile, share; };
constexpr DlTileModel DL_MODEL[DL_TILES] = {
    {256, 256, 1, 0.0, 16.3, 7.8, 1.327, 0.0},   {256, 128, 1, 0.0, 8.2, 2.9, 0.869, 0.0},
    {128, 128, 1, 1.5, 3.6, 1.7, 0.577, 0.0},    {128, 128, 2, 0.9, 4.8, 2.2, 0.734, 0.273},
    {64, 64, 2, 2.8, 1.3, 0.5, 0.226, 0.238},    {64, 64, 5, 1.9, 1.8, 0.7, 0.496, 0.152},
};

inline double dl_tile_time(DlTileId t, long M, long N, long K, bool heavy, int parts, int n_cu) {
    const DlTileModel& m = DL_MODEL[t];
    const long tiles = ((M + m.bm - 1) / m.bm) * ((N + m.bn - 1) / m.bn) * parts;
    const double nk = (double)(((K + parts - 1) / parts + 63) / 64);
    const double fix = m.round + (heavy ? m.heavy : 0.0);
    const long slots = (long)m.per_cu * n_cu;
    double us = m.launch + (double)(tiles / slots) * (fix + nk * (m.ktile + m.share * (m.per_cu - 1)));
    if (const long rest = tiles % slots; rest) {
        // a round that leaves units idle runs faster on the others (memory, clock)
        const double used = std::min(1.0, (double)rest / n_cu);
        const int together = (int)((rest + n_cu - 1) / n_cu);
        us += fix * (0.5 + 0.5 * used) + nk * (m.ktile + m.share * (together - 1)) * (0.72 + 0.28 * used);
    }
    return us;
}

struct DlPlan { DlTileId tile; int parts; int k_part; };

// Length of a part when K is cut into `parts` (a multiple of the 64-long k-tile).
inline int dl_part_length(long K, int parts) { return (int)(((K + parts - 1) / parts + 63) / 64 * 64); }

// A product with few output tiles and a long contraction may run in 2, 4 or 8 parts
// into fp32 scratch, added in order by a second kernel (2.5 us, and 4 bytes per part and
// output element at the rate measured for scratch that was just written): 640x640x8192 39
// -> 20 us, [1000, 2048] outputs with an 8192-long contraction 67 -> 46 us. The parts must
// be at least 256 long and win by 10 %: inside a stage the scratch also displaces the
// caches' other contents.
inline DlPlan dl_plan(long M, long N, long K, bool heavy, bool may_split, size_t scratch_bytes, int n_cu) {
    DlPlan best{DL_64, 1, (int)K};
    double best_us = 1e30;
    for (int t = 0; t < DL_TILES; ++t) {
        const double us = dl_tile_time((DlTileId)t, M, N, K, heavy, 1, n_cu);
        if (us < best_us) { best_us = us; best = {(DlTileId)t, 1, (int)K}; }
    }
    if (!may_split) return best;
    for (int parts = 2; parts <= 8; parts *= 2) {
        if (K / parts < 256 || (size_t)M * N * 4 * parts > scratch_bytes) break;
        const int k_part = dl_part_length(K, parts);
        if ((long)k_part * (parts - 1) >= K) break;
        const double reduce = 2.5 + (double)M * N * (4.0 * parts + 4.0) / 9.5e6;
        for (int t = 0; t < DL_TILES; ++t) {
            const double us = 1.1 * (dl_tile_time((DlTileId)t, M, N, K, true, parts, n_cu) + reduce);
            if (us < best_us) { best_us = us; best = {(DlTileId)t, parts, k_part}; }
        }
    }
    return best;
}

}  // namespace amdp
