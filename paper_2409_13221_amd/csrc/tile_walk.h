// Workgroup -> tile mapping of the compute-bound GEMM launches.
#pragma once
#include <hip/hip_runtime.h>

namespace rlhf {

// The tile grid is cut into panels of kGroupM tile rows.  Inside a panel the tile columns are dealt to
// the 8 XCDs (workgroup id modulo 8, the order in which the dispatcher deals workgroups to XCDs) in
// contiguous groups, and an XCD walks its group column by column.  Two things follow.  The workgroups
// resident on one XCD at a time cover a compact block of kGroupM x 4 tiles, so its L2 re-serves the A
// rows and W rows they share.  And all XCDs work on the SAME panel of A rows at the same time, each on W
// columns of its own: an A panel is requested by the eight L2s within a short time of each other (one
// fetch from HBM, the others from the memory-side cache even while a decode stream sweeps its weights
// through that cache) and every W column is fetched by one XCD only, once per panel.  (Before, each XCD
// walked its own contiguous eighth of the panel-ordered tile list; the eight of them then sat on up to
// four different A panels and up to eight W ranges, and with the memory-side cache swept by the decode
// stream the scoring GEMMs pulled several times their operands from HBM.)
constexpr int kGroupM = 8;
__host__ __device__ inline int xcd_cols(int tiles_n) { return (tiles_n + 7) >> 3; }   // tile columns per XCD
inline int xcd_grid(int tiles_m, int tiles_n) { return 8 * tiles_m * xcd_cols(tiles_n); }
__host__ __device__ __forceinline__ bool xcd_tile_of(int bid, int tiles_m, int tiles_n, int& tm, int& tn) {
    const int xcd = bid & 7, slot = bid >> 3;
    const int cx = xcd_cols(tiles_n);
    const int c_lo = xcd * cx;
    const int c_n = min(tiles_n, c_lo + cx) - c_lo;          // this XCD's columns (may be <= 0 at the end)
    if (c_n <= 0) return false;
    const int per_panel = kGroupM * c_n;
    const int full = tiles_m / kGroupM;
    int panel = slot / per_panel, r = slot - panel * per_panel, rows = kGroupM;
    if (panel >= full) {                                     // the last, shorter panel
        panel = full;
        r = slot - full * per_panel;
        rows = tiles_m - full * kGroupM;
        if (rows <= 0 || r >= rows * c_n) return false;
    }
    tm = panel * kGroupM + r % rows;
    tn = c_lo + r / rows;
    return true;
}

}  // namespace rlhf
