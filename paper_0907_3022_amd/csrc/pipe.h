// Pipelined many-order passes over honeycomb ribbons (pipe.hip): D = DW NW
// Chebyshev orders in one pass over memory, carried by a workgroup of NW
// wavefronts with DW orders each.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "internal.h"

namespace chebtd {

constexpr int kMaxPipe = 24;  // most orders one pipelined pass carries

// Columns a workgroup reads (two per lane), and those it owns: an order
// spoils one column per side, so D orders need ceil(D / 2) halo lanes.
constexpr int pipe_halo_lanes(int D) { return (D + 1) / 2; }
constexpr int pipe_strip_cols(int D) { return 128 - 4 * pipe_halo_lanes(D); }

struct PipeOp {
    const double *onsite;  // eps
    double dshift;         // -b
    double s2;             // 2/a
    double off2;           // -2t/a
    int32_t W, L;          // rows, columns
    int32_t nstrips, nchunks;
};

// First row of chunk c of n over W rows.  A workgroup's walk takes rows +
// halo above + D iterations; the top chunk has no halo above it, so it takes
// D - 1 rows more than the others.  Even, so that the parity of a row is that
// of the walk's iteration.
__host__ __device__ inline int32_t pipe_row(int32_t c, int32_t n, int32_t W, int D)
{
    if (c <= 0) return 0;
    if (c >= n) return W;
    return (int32_t)((D - 1 + (int64_t)c * (W - (D - 1)) / n) & ~(int64_t)1);
}

// Operands of one pass, orders k0+1 .. k0+D (D a multiple of four, so k0 is
// one).  The weights are the real factors r_k (J_0, 2 J_k) of gamma_k =
// e^{-ib dt} (-i)^k r_k.  acc holds e^{ib dt} times the usual partial sum, so
// that every order adds a real multiple; the step's last pass multiplies with
// `fin` = e^{-ib dt}.
struct PipeArgs {
    const double2 *vkm1, *vk;  // v_{k0-1} (null: step head, vk = psi), v_{k0}
    double2 *out1, *out2;      // v_{k0+D-1}, v_{k0+D} (null: last pass of the step)
    const double2 *acc_in;     // head: not read
    double2 *acc_out;
    double2 *ckpt;             // head: a copy of psi, or null
    double2 fin;               // the step's last pass: e^{-ib dt}; else 1
    const double *r;           // r[j]: weight of order k0+j (r[0]: the head's); 0 past M
};

// passes of a step of M orders (the last one padded, or exact), empty: not
// pipelined
std::vector<PipeShape> plan_pipe(const Ctx &c, int M, bool exact);
// their estimated time, us
double pipe_time(int64_t W, int64_t L, const std::vector<PipeShape> &passes, int num_cus);
// adds what one ribbon of many costs a pass of each shape, us
constexpr int kPipeShapes = 5;
void pipe_shape_costs(int64_t W, int64_t L, int num_cus, double *cost);
// the same without the chunks, for lattices of `sites` sites in all or by the cost
// of a pass of each shape
std::vector<PipeShape> plan_pipe_shapes(int64_t sites, int M, bool exact, const double *cost = nullptr);
// row chunks of a pass
int pipe_chunks(int64_t W, int64_t L, int DW, int NW, int num_cus);
// iterations of the longest walk when W rows are cut into n chunks
int32_t pipe_iterations(int DW, int NW, int32_t W, int32_t n);
int64_t pipe_blocks(const Ctx &c, const PipeShape &s);
// partials: (norm, energy) per block from the head, knorm: sum |acc|^2 per
// block from the last pass; either may be null
hipError_t launch_pipe(const Ctx &c, hipStream_t s, const PipeShape &sh, const PipeArgs &A, double *partials,
                       double *knorm);
// Sums of `count` steps' head partials (stride doubles apart) into
// norm_out/energy_out[first ..] (two steps, first read from and advanced in
// *counter, if that is given: no check then); check (host-visible, or null):
// check[0] = norm of step 0 when first_step, check[2] = sum of the nk doubles
// at knorm when given.
struct NeSteps {
    const double *partials;
    int64_t stride;
    int nparts, count;
    double a, b;
    double *norm_out, *energy_out;
    int64_t first;
    int64_t *counter;
    const double *knorm;
    int nk;
    double *check;
    int first_step;
};
hipError_t launch_ne_steps(hipStream_t s, const NeSteps &f);

}  // namespace chebtd
