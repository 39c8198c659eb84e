// Many-order passes over ribbons of up to 48 rows, held in registers
// (ribbon_tile_walk.h, ribbon_tile.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "chain_tile.h"
#include "internal.h"
#include "pipe.h"

namespace chebtd {

constexpr int kTileRows = 48;   // most rows of a ribbon
constexpr int kTileDepth = 48;  // most orders of a pass (32 own columns left of 128)

// rows per wavefront for a ribbon of W <= 48 rows (at most eight wavefronts)
inline int ribbon_tile_rows(int64_t W) { return W <= 16 ? 2 : W <= 32 ? 4 : 6; }

inline int ribbon_tile_waves(int64_t W)
{
    const int r = ribbon_tile_rows(W);
    return (int)((W + r - 1) / r);
}
inline int64_t ribbon_tile_blocks(int64_t L, int D)
{
    const int S = 128 - 4 * ((D + 1) / 2);
    return (L + S - 1) / S;
}
// LDS of a workgroup of NW wavefronts
constexpr size_t kTileEdgeBytes = 4 * 64 * sizeof(double2);
inline size_t ribbon_tile_lds(int NW) { return (size_t)2 * (NW + 2) * kTileEdgeBytes; }
// depths of the passes of a step of M >= 2 orders over a W x L ribbon (W <= 48)
// and the step's estimated time; R of the plan: rows per wavefront
TilePlan plan_ribbon_tile(int64_t W, int64_t L, int edge, int M, int num_cus, double *us);
hipError_t launch_ribbon_tile(const Ctx &c, hipStream_t s, const TileArgs &A, double *partials, double *knorm);

}  // namespace chebtd
