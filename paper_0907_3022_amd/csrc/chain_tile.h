// Many-order passes over 1D chains (chain_tile.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "internal.h"

namespace chebtd {

struct TileOp {
    const double *V;
    double dsh, s2, off2;  // as OpChain
    int64_t n;
};

// Operands of one pass, orders k0+1 .. k0+D; roles, weights and acc's factor
// as PipeArgs (pipe.h), out1 / out2 null: not written
struct TileArgs {
    const double2 *vkm1, *vk;  // v_{k0-1} (null: step head, vk = psi), v_{k0}
    double2 *out1, *out2;      // v_{k0+D-1}, v_{k0+D}
    const double2 *acc_in;
    double2 *acc_out;
    double2 *ckpt;
    double2 fin;               // the step's last pass: e^{-ib dt}; else 1
    const double *r;           // r[j]: weight of order k0+j, readable to j = D + 8
    int32_t D, k0;
};

constexpr int kTilePad = 12;  // weights read past M

// chains: R sites per lane; orders per pass, in launch order; empty: no tiled
// passes
TilePlan plan_tile(const Ctx &c, int M);
int64_t tile_blocks(const Ctx &c, int R, int D);
hipError_t launch_tile(const Ctx &c, hipStream_t s, int R, const TileArgs &A, double *partials, double *knorm);

}  // namespace chebtd
