// Pipelined reverse passes of the adjoint over ribbons (pipe_rev.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "internal.h"
#include "pipe.h"

namespace chebtd {

constexpr int kRevPipeDW = 2, kRevPipeNW = 4, kRevPipeDepth = kRevPipeDW * kRevPipeNW;

// Levels k .. k-7 (k - 7 >= 0) with the forward vectors run downwards; roles
// as RevPass (internal.h).
struct RevPipeArgs {
    const double2 *uk2, *uk1, *v1, *v0;
    double2 *out1, *out2, *vout1, *vout2;
    const double2 *gbar;
    double *grad;
    double2 fac;      // i^k e^{ib dt}: conj(g_{k-j}) = fac (-i)^j r_{k-j}
    const double *r;  // r[-j]: weight of order k - j
    double gf;        // 2/a
    double half;      // 1/2 when the last level is level 0, else 1
};

bool rev_pipe_fits(const Ctx &c);
// chunks: rev_pipe_chunks' choice, kept with the plan
int rev_pipe_chunks(const Ctx &c);
hipError_t launch_rev_pipe(const Ctx &c, hipStream_t s, int chunks, const RevPipeArgs &A);

}  // namespace chebtd
