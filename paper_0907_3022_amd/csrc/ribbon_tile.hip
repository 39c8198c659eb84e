// Register-resident many-order passes over ribbons of up to 48 rows: kernel,
// plan and launcher (the walk: ribbon_tile_walk.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>

#include "device_ops.h"
#include "internal.h"
#include "pair.h"
#include "ribbon_tile.h"
#include "ribbon_tile_walk.h"

namespace chebtd {

static_assert(sizeof(TileEdges) == kTileEdgeBytes, "edge rows");

template <int EDGE, int RW>
__global__ __launch_bounds__(512) void k_ribbon_tile(PipeOp op, TileArgs A, double *partials, double *knorm)
{
    extern __shared__ double2 lds_raw[];
    __shared__ double red[2 * 8];
    double s0 = 0.0, s1 = 0.0, sk = 0.0, z = 0.0;
    ribbon_tile_block<EDGE, RW>(op, A, logical_block(1), (int)(blockDim.x >> 6),
                                reinterpret_cast<TileEdges *>(lds_raw), s0, s1, sk);
    if (partials && A.vkm1 == nullptr) {
        block_sum2(s0, s1, red);
        if (threadIdx.x == 0) {
            partials[2 * blockIdx.x] = s0;
            partials[2 * blockIdx.x + 1] = s1;
        }
        __syncthreads();
    }
    if (knorm) {
        block_sum2(sk, z, red);
        if (threadIdx.x == 0) knorm[blockIdx.x] = sk;
    }
}

TilePlan plan_ribbon_tile(int64_t W, int64_t L, int edge, int M, int num_cus, double *us)
{
    TilePlan best;
    *us = 1e300;
    if (W > kTileRows || M < 2 || !deep_offsets_fit(W, L) || std::getenv("CHEBTD_DEPTH")) return best;
    int fd = 0;
    if (const char *env = std::getenv("CHEBTD_TILE")) {
        fd = std::atoi(env);
        if (fd < 2) return best;
    }
    const int R = ribbon_tile_rows(W), NW = ribbon_tile_waves(W);
    // an order: the wavefronts of the busiest SIMD, then the rows' exchange
    const double ns = R * (edge == CHEBTD_ZIGZAG ? 28 : 24) * (NW <= 4 ? 2.3 : 1.95 * std::ceil(NW / 4.0)) + 80.0;
    const int most = fd ? std::min(fd, kTileDepth) : kTileDepth, fewest = (M + most - 1) / most;
    for (int p = fewest; p <= std::min(M, 4 * fewest + 4); ++p) {
        const int D = (M + p - 1) / p;
        const double wgs = (double)ribbon_tile_blocks(L, D);
        const double t = p * (4.0 + std::ceil(wgs / num_cus) * D * ns * 1e-3 + (p == 1 ? 40.0 : 90.0) * W * L / 5.0e6);
        if (t < *us) {
            *us = t;
            best.R = R;
            best.depths.assign((size_t)p, D);
            for (int q = 0, over = D * p - M; q < over; ++q) --best.depths[(size_t)(p - 1 - q)];
        }
    }
    return best;
}

hipError_t launch_ribbon_tile(const Ctx &c, hipStream_t s, const TileArgs &A, double *partials, double *knorm)
{
    const int R = ribbon_tile_rows(c.W), NW = ribbon_tile_waves(c.W);
    if (c.W > kTileRows || A.D < 1 || A.D > kTileDepth || !deep_offsets_fit(c.W, c.L) || (!A.vkm1 && A.k0 != 0))
        return hipErrorInvalidValue;
    PipeOp op{};
    op.onsite = c.eps;
    op.dshift = -c.b;
    op.s2 = 2.0 / c.a;
    op.off2 = -2.0 * c.t_hop / c.a;
    op.W = (int32_t)c.W;
    op.L = (int32_t)c.L;
    const int64_t nb = ribbon_tile_blocks(c.L, A.D);
    if (nb > INT32_MAX) return hipErrorInvalidValue;
    const size_t dyn = ribbon_tile_lds(NW);
    auto run = [&](auto *kernel) {
        if (dyn > 65536) {
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)nb), dim3(64 * NW), dyn, s, op, A, partials, knorm);
        return hipGetLastError();
    };
    const bool zig = c.edge == CHEBTD_ZIGZAG;
    switch (R) {
        case 2: return zig ? run(&k_ribbon_tile<CHEBTD_ZIGZAG, 2>) : run(&k_ribbon_tile<CHEBTD_ARMCHAIR, 2>);
        case 4: return zig ? run(&k_ribbon_tile<CHEBTD_ZIGZAG, 4>) : run(&k_ribbon_tile<CHEBTD_ARMCHAIR, 4>);
        default: return zig ? run(&k_ribbon_tile<CHEBTD_ZIGZAG, 6>) : run(&k_ribbon_tile<CHEBTD_ARMCHAIR, 6>);
    }
}

}  // namespace chebtd
