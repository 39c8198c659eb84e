// Pipelined many-order passes for single ribbons: kernel, pass plan and
// launcher (the walk: pipe_walk.h), and the sums of the per-step norm and
// energy partials.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "device_ops.h"
#include "internal.h"
#include "pair.h"
#include "pipe.h"
#include "pipe_walk.h"

namespace chebtd {

template <int EDGE, int DW, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_pipe(PipeOp op, PipeArgs A, double *partials, double *knorm)
{
    __shared__ PipeSlot slots[NW - 1][2];
    // consecutive chunks of a strip on one XCD, whose L2 then holds the halo
    // rows that both read
    const int32_t wg = logical_block(1);
    const int32_t strip = wg / op.nchunks, chunk = wg - strip * op.nchunks;
    const int32_t ys = pipe_row(chunk, op.nchunks, op.W, DW * NW);
    const int32_t ye = pipe_row(chunk + 1, op.nchunks, op.W, DW * NW);
    double s0 = 0.0, s1 = 0.0;
    pipe_block<EDGE, DW, NW>(op, A, strip, ys, ye, slots, s0, s1);
    const int w = pipe_wave<NW>(), lane = threadIdx.x & 63;
    if (w == 0 && A.vkm1 == nullptr && partials) {
        s0 = wave_sum(s0);
        s1 = wave_sum(s1);
        if (lane == 0) {
            partials[2 * blockIdx.x] = s0;
            partials[2 * blockIdx.x + 1] = s1;
        }
    }
    if (w == NW - 1 && knorm) {
        s0 = wave_sum(s0);
        if (lane == 0) knorm[blockIdx.x] = s0;
    }
}

// Block b: step first + b's norm and energy; the last block also the final
// norm.  Fixed order, as finalize_ne_block.
__global__ __launch_bounds__(256) void k_ne_steps(NeSteps f)
{
    __shared__ double red[2 * 4];
    const int nblk = gridDim.x;
    for (int i = blockIdx.x; i < f.count; i += nblk) {
        const double *p = f.partials + (int64_t)i * f.stride;
        double s0 = 0.0, s1 = 0.0;
        for (int q = threadIdx.x; q < f.nparts; q += blockDim.x) {
            s0 += p[2 * q];
            s1 += p[2 * q + 1];
        }
        block_sum2(s0, s1, red);
        if (threadIdx.x == 0) {
            if (f.norm_out) f.norm_out[f.first + i] = s0;
            if (f.energy_out) f.energy_out[f.first + i] = f.a * s1 + f.b * s0;
            if (f.check && f.first_step && i == 0) f.check[0] = s0;
        }
        __syncthreads();
    }
    if (f.knorm && f.check && (int)blockIdx.x == nblk - 1) {
        double s0 = 0.0, z = 0.0;
        for (int q = threadIdx.x; q < f.nk; q += blockDim.x) s0 += f.knorm[q];
        block_sum2(s0, z, red);
        if (threadIdx.x == 0) f.check[2] = s0;
    }
}

// The same for the two steps of a graph, whose place is in *counter: a half of
// the block to each step.  One step after the other, behind the read of the
// counter, two replays of a 64 x 1000 ribbon with order 9 took 94.6 us, now 92.6;
// with order 6 and walked steps 68.1 and 63.7.
constexpr int kGraphSteps = 2;
__global__ __launch_bounds__(256 * kGraphSteps) void k_ne_graph(NeSteps f)
{
    __shared__ double red[kGraphSteps][2 * 4];
    const int i = threadIdx.x >> 8, t = threadIdx.x & 255, w = t >> 6;
    const int64_t first = *f.counter;
    const double *p = f.partials + (int64_t)i * f.stride;
    double s0 = 0.0, s1 = 0.0;
    for (int q = t; q < f.nparts; q += 256) {
        s0 += p[2 * q];
        s1 += p[2 * q + 1];
    }
    s0 = wave_sum(s0);
    s1 = wave_sum(s1);
    if ((t & 63) == 0) {
        red[i][2 * w] = s0;
        red[i][2 * w + 1] = s1;
    }
    __syncthreads();  // and every thread has read the counter
    if (t != 0) return;
    s0 = s1 = 0.0;
    for (int v = 0; v < 4; ++v) {
        s0 += red[i][2 * v];
        s1 += red[i][2 * v + 1];
    }
    if (f.norm_out) f.norm_out[first + i] = s0;
    if (f.energy_out) f.energy_out[first + i] = f.a * s1 + f.b * s0;
    if (i == 0) *f.counter = first + kGraphSteps;
}

hipError_t launch_ne_steps(hipStream_t s, const NeSteps &f)
{
    if (f.counter) {
        if (f.count != kGraphSteps || f.knorm || f.check) return hipErrorInvalidValue;
        hipLaunchKernelGGL(k_ne_graph, dim3(1), dim3(256 * kGraphSteps), 0, s, f);
    } else {
        hipLaunchKernelGGL(k_ne_steps, dim3((unsigned)std::max(1, f.count)), dim3(256), 0, s, f);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Iterations of the longest walk when W rows are cut into n chunks.
int32_t pipe_iterations(int DW, int NW, int32_t W, int32_t n)
{
    int32_t most = 0;
    for (int32_t c : {0, 1, n - 1}) {
        if (c < 0 || c >= n) continue;
        const int32_t ys = pipe_row(c, n, W, DW * NW), ye = pipe_row(c + 1, n, W, DW * NW);
        for (int w = 0; w < NW; ++w) {
            const pipedev::PipeSpan sp = pipedev::pipe_span(DW, NW, w, ys, ye, W);
            most = std::max(most, sp.t0 + sp.n);
        }
    }
    return most;
}

// Row chunks of a pass: the count with the least estimated time.  Taller
// chunks repeat fewer halo rows, more chunks fill the CUs.  A CU holds two
// workgroups of four wavefronts or one of eight; measured on MI355X an
// iteration of a four-wavefront workgroup takes 0.44 us alone on its CU and
// 0.74 us for two together (zigzag, five orders per wavefront: 128 x 8192 in
// 2 / 3 / 5 chunks 52.8 / 63.5 / 55.5 us a step, 1024 x 32768 in 1 / 2 / 4 / 8
// chunks 789 / 700 / 687 / 763 us).  CHEBTD_PIPE_CHUNKS overrides.
static double pipe_rounds(int64_t wgs, int NW, int num_cus)
{
    const int64_t slots = (int64_t)num_cus * (NW <= 4 ? 2 : 1), rest = wgs % slots;
    return (double)(wgs / slots) + (rest == 0 ? 0.0 : rest <= num_cus && NW <= 4 ? 0.6 : 1.0);
}

int pipe_chunks(int64_t W, int64_t L, int DW, int NW, int num_cus)
{
    const int D = DW * NW;
    const int64_t most = std::max<int64_t>(1, (W - (D - 1)) / 8);  // at least 8 rows each
    if (const char *env = std::getenv("CHEBTD_PIPE_CHUNKS"))
        return (int)std::max<int64_t>(1, std::min<int64_t>(most, std::atoi(env)));
    const int64_t strips = ceil_div(L, pipe_strip_cols(D));
    const int64_t slots = (int64_t)num_cus * (NW <= 4 ? 2 : 1);
    int64_t best = 1;
    double bt = 1e300;
    const int64_t limit = std::min(most, std::max<int64_t>(1, 4 * slots / strips));
    auto iterations = [&](int64_t n) { return pipe_iterations(DW, NW, (int32_t)W, (int32_t)n); };
    // counts of as many rounds at a time: the fewest of them whose walks are as
    // short as those of the most (a tall narrow ribbon has thousands of counts)
    int64_t first = 1;
    for (int64_t k = 0; first <= limit; ++k)
        for (int64_t wgs : {k * slots + num_cus, (k + 1) * slots}) {
            const int64_t end = std::min(limit, wgs / strips);
            if (end < first) continue;
            const int32_t it = iterations(end);
            const double t = pipe_rounds(strips * end, NW, num_cus) * it;
            if (t < bt) {
                int64_t lo = first, hi = end;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) / 2;
                    if (iterations(mid) <= it)
                        hi = mid;
                    else
                        lo = mid + 1;
                }
                bt = t;
                best = lo;
            }
            first = end + 1;
        }
    return (int)best;
}

// An iteration of two workgroups on a CU (one of eight wavefronts): 0.74 us
// at five orders per wavefront, less in proportion below.
double pipe_time(int64_t W, int64_t L, const std::vector<PipeShape> &passes, int num_cus)
{
    double us = 0.0;
    for (const PipeShape &p : passes)
        us += 3.0 + pipe_rounds(ceil_div(L, pipe_strip_cols(p.depth())) * p.chunks, p.NW, num_cus) *
                        pipe_iterations(p.DW, p.NW, (int32_t)W, p.chunks) * (p.NW <= 4 ? 0.14 + 0.12 * p.DW : 0.55);
    return us;
}

// Passes of a step of M orders, the last padded with orders of weight 0: the
// cheapest by each pass's measured time (us, MI355X) on lattices of 10^4, 10^6
// and 3.4 10^7 sites (10 x 1000 armchair, 128 x 8192 and 1024 x 32768 zigzag).
// Not pipelined: lattices past the 32-bit offsets (deep_offsets_fit), and a
// depth forced by CHEBTD_DEPTH.  CHEBTD_PIPE=DW,NW forces one shape, 0 none.
// exact: no padding (the passes' orders add up to M, or there are none).
std::vector<PipeShape> plan_pipe(const Ctx &c, int M, bool exact)
{
    if (c.kind != HKind::Honeycomb || !deep_offsets_fit(c.W, c.L)) return {};
    std::vector<PipeShape> out = plan_pipe_shapes(c.n, M, exact);
    for (size_t i = 0; i < out.size(); ++i)
        out[i].chunks = i > 0 && out[i].DW == out[i - 1].DW && out[i].NW == out[i - 1].NW
                            ? out[i - 1].chunks
                            : pipe_chunks(c.W, c.L, out[i].DW, out[i].NW, c.num_cus);
    return out;
}

struct PipeCand {
    int DW, NW;
    double tiny, small, large;
};
static const PipeCand kPipeCands[kPipeShapes] = {{2, 4, 10.9, 26.0, 640.0}, {3, 4, 12.9, 32.0, 570.0},
                                                 {4, 4, 15.4, 41.0, 645.0}, {5, 4, 18.8, 53.0, 700.0},
                                                 {3, 8, 21.1, 62.0, 1090.0}};

// Adds a ribbon's share of a pass over so many that every CU is full: the larger
// of its workgroups' iterations, two of four wavefronts or one of eight sharing a
// CU, and its bytes at 4.2 TB/s.
void pipe_shape_costs(int64_t W, int64_t L, int num_cus, double *cost)
{
    for (int q = 0; q < kPipeShapes; ++q) {
        const PipeCand &x = kPipeCands[q];
        const double strips = (double)ceil_div(L, pipe_strip_cols(x.DW * x.NW));
        const double it = pipe_iterations(x.DW, x.NW, (int32_t)W, 1);
        const double us = x.NW <= 4 ? 0.5 * (0.14 + 0.12 * x.DW) : 0.55;
        cost[q] += std::max(0.9 * strips * it * us / num_cus, 104.0 * (double)(W * L) / 4.2e6);
    }
}

// cost: of each shape (or null: by the number of sites)
std::vector<PipeShape> plan_pipe_shapes(int64_t sites, int M, bool exact, const double *cost)
{
    std::vector<PipeShape> out;
    if (M < 2 || std::getenv("CHEBTD_DEPTH")) return out;
    int fdw = 0, fnw = 0;
    if (const char *env = std::getenv("CHEBTD_PIPE"))
        if (std::sscanf(env, "%d,%d", &fdw, &fnw) != 2) return out;
    std::vector<double> best((size_t)M + 1, 1e300);
    std::vector<int> from((size_t)M + 1, -1);
    best[0] = 0.0;
    for (int m = 1; m <= M; ++m)
        for (int q = 0; q < kPipeShapes; ++q) {
            const PipeCand &x = kPipeCands[q];
            if ((fdw && (x.DW != fdw || x.NW != fnw)) || (exact && x.DW * x.NW > m)) continue;
            const double t = best[(size_t)std::max(0, m - x.DW * x.NW)] +
                             (cost                           ? cost[q]
                              : sites < (int64_t(1) << 17)   ? x.tiny
                              : sites < (int64_t(1) << 22)   ? x.small
                                                             : x.large);
            if (t < best[(size_t)m]) {
                best[(size_t)m] = t;
                from[(size_t)m] = q;
            }
        }
    for (int m = M; m > 0;) {
        if (from[(size_t)m] < 0) return {};
        const PipeCand &x = kPipeCands[from[(size_t)m]];
        out.push_back({x.DW, x.NW, 1});
        m -= x.DW * x.NW;
    }
    // full passes first, so that only the last is padded: the depths in
    // descending order hold M, and the last alone covers what is left
    std::sort(out.begin(), out.end(), [](const PipeShape &a, const PipeShape &b) { return a.depth() > b.depth(); });
    return out;
}

static PipeOp make_pipe_op(const Ctx &c, const PipeShape &sh)
{
    PipeOp op{};
    op.onsite = c.eps;
    op.dshift = -c.b;
    op.s2 = 2.0 / c.a;
    op.off2 = -2.0 * c.t_hop / c.a;
    op.W = (int32_t)c.W;
    op.L = (int32_t)c.L;
    op.nstrips = (int32_t)ceil_div(c.L, pipe_strip_cols(sh.depth()));
    op.nchunks = sh.chunks;
    return op;
}

int64_t pipe_blocks(const Ctx &c, const PipeShape &sh)
{
    const PipeOp op = make_pipe_op(c, sh);
    return (int64_t)op.nstrips * op.nchunks;
}

hipError_t launch_pipe(const Ctx &c, hipStream_t s, const PipeShape &sh, const PipeArgs &A, double *partials,
                       double *knorm)
{
    const PipeOp op = make_pipe_op(c, sh);
    const int64_t nb = (int64_t)op.nstrips * op.nchunks;
    if (nb <= 0 || nb > INT32_MAX || !deep_offsets_fit(op.W, op.L)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nb), block(64 * sh.NW);
    const bool zig = c.edge == CHEBTD_ZIGZAG;
#define CHEBTD_PIPE_SHAPE(dw, nw)                                                                          \
    if (sh.DW == dw && sh.NW == nw) {                                                                      \
        if (zig)                                                                                           \
            hipLaunchKernelGGL((k_pipe<CHEBTD_ZIGZAG, dw, nw>), grid, block, 0, s, op, A, partials, knorm); \
        else                                                                                               \
            hipLaunchKernelGGL((k_pipe<CHEBTD_ARMCHAIR, dw, nw>), grid, block, 0, s, op, A, partials, knorm); \
        return hipGetLastError();                                                                          \
    }
    CHEBTD_PIPE_SHAPE(2, 4)
    CHEBTD_PIPE_SHAPE(3, 4)
    CHEBTD_PIPE_SHAPE(4, 4)
    CHEBTD_PIPE_SHAPE(5, 4)
    CHEBTD_PIPE_SHAPE(3, 8)
#undef CHEBTD_PIPE_SHAPE
    return hipErrorInvalidValue;
}

}  // namespace chebtd
