// Eight levels of the adjoint's reverse recursion per pass over a ribbon, the
// forward vectors run downwards beside them (the recursions of deep_walk.h's
// kDeepRev), pipelined over the four wavefronts of a workgroup as in
// pipe_walk.h:
//   u_{k-j+1} = conj(g_{k-j+1}) gbar + 2 H~ u_{k-j+2} - u_{k-j+3},
//   v_{k-j}   = 2 H~ v_{k-j+1} - v_{k-j+2},
//   dL/dV    += (2/a) Re[conj(u_{k-j+2}) v_{k-j+1}],      j = 1 .. 8.
// Two levels per wavefront: the two recursions' windows, gbar, the partial
// dL/dV and the diagonal of the rows in flight fill the registers; a column
// hands on 96 B per row.  168 B per site and pass, as for the five levels of
// the single-wavefront walk.
//
// What bounds it: at 512 x 16384 HBM (168 B per site for eight levels at a large
// copy's rate); at 256 x 4096 a row of the slowest wavefront as in pipe_walk.h (21
// instructions and 8 lane shifts per site and level, 4 on armchair edges, 0.76
// wavefronts per SIMD, VALU busy 23%), with 4.65 TB/s counted beside it: a strip's halo of 8 columns per side and the refill of every
// chunk weigh less than the second pass over memory that they save.  Measured
// on MI355X, reverse run per step, single-wavefront passes of five levels ->
// these: 256 x 4096 (64 orders) 503 -> 353 us (44 us a pass, 4.0 TB/s),
// 512 x 16384 (40 orders) 2559 -> 1535 us (307 us a pass, 4.6 TB/s, a large
// copy's rate), 64 x 1000 253 -> 117 us, 8 x 64 159 -> 80 us.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "device_ops.h"
#include "internal.h"
#include "pair.h"
#include "pipe_rev.h"
#include "pipe_walk.h"

namespace chebtd {

namespace {

// One row handed on, 64 lanes of 16 B each: newest u of the lane's two
// columns, the one before; the same of v; gbar; diagonal; dL/dV.
struct RevSlot {
    double2 part[12][64];
};
using LdsBytes = __attribute__((address_space(3))) char;
using LdsD2 = double __attribute__((ext_vector_type(2)));

}  // namespace

namespace revdev {

using namespace deepdev;
using namespace pairdev;
using pipedev::arrived;
using pipedev::kUnroll;
using pipedev::PipeSpan;
using pipedev::pipe_span;
using pipedev::row_barrier;
using pipedev::turn;

constexpr int kFirst = 0, kMid = 1, kLast = 2;

struct RowSet {
    double2 a[2], k[2], va[2], vk[2], p[2];
    double e[2], g[2];
};
__device__ __forceinline__ void arrived(const RowSet &n)
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        arrived(n.a[c]);
        arrived(n.k[c]);
        arrived(n.va[c]);
        arrived(n.vk[c]);
        arrived(n.p[c]);
    }
    arrived(n.e);
    arrived(n.g);
}

// y += (-i)^n r x
template <int n>
__device__ __forceinline__ double2 add_turned(double r, double2 x, double2 y)
{
    pipedev::add_order(n, r, x, y);
    return y;
}

template <int EDGE, int ROLE>
__device__ __forceinline__ void wave(const PipeOp &op, const RevPipeArgs &A, int w, int32_t strip, int32_t ys,
                                     int32_t ye, int32_t tend, RevSlot (*slots)[2])
{
    constexpr int DW = kRevPipeDW, NW = kRevPipeNW;
    constexpr bool FIRST = ROLE == kFirst, LASTW = ROLE == kLast;
    constexpr int D = DW * NW, HL = pipe_halo_lanes(D), S = pipe_strip_cols(D);
    const int lane = threadIdx.x & 63;
    const int32_t W = op.W, L = op.L;
    const int32_t x = strip * S - 2 * HL + 2 * lane;
    const bool in0 = x >= 0 && x < L, in1 = x + 1 >= 0 && x + 1 < L;
    const bool own = lane >= HL && lane < 64 - HL;
    const uint32_t nb16 = (uint32_t)W * (uint32_t)L * 16u, row16 = (uint32_t)L * 16u, row8 = (uint32_t)L * 8u;
    const double2 zero = make_double2(0.0, 0.0);
    // range checks as in pipe_walk.h; a missing buffer reads zeros and drops
    // its stores
    auto ld2 = [&](const double2 *p, int32_t row, bool ok, uint32_t lanepart) {
        return bload2(rsrc(p ? p : A.uk1, p && ok ? nb16 : 0u), lanepart, ok ? (uint32_t)row * row16 : 0u);
    };
    auto st2 = [&](double2 *p, int32_t row, bool ok, uint32_t lanepart, double2 v) {
        bstore2(rsrc(p ? p : A.out2, p && ok ? nb16 : 0u), (ok ? (uint32_t)row * row16 : 0u) + lanepart, 0, v);
    };
    auto inside = [&](int32_t row) { return (uint32_t)row < (uint32_t)W; };
    auto mine = [&](int32_t q) { return q >= ys && q < ye; };
    const uint32_t c16[2] = {in0 ? (uint32_t)x * 16u : kOut, in1 ? (uint32_t)(x + 1) * 16u : kOut};
    const uint32_t c8[2] = {in0 ? (uint32_t)x * 8u : kOut, in1 ? (uint32_t)(x + 1) * 8u : kOut};
    const uint32_t s16[2] = {own ? c16[0] : kOut, own ? c16[1] : kOut};
    const uint32_t s8[2] = {own ? c8[0] : kOut, own ? c8[1] : kOut};
    const double off[2] = {in0 ? op.off2 : 0.0, in1 ? op.off2 : 0.0};

    const PipeSpan sp = pipe_span(DW, NW, w, ys, ye, W);
    double r[DW];  // of level l: order k - (w DW + l - 1)
#pragma unroll
    for (int l = 0; l < DW; ++l) r[l] = A.r[-(w * DW + l)];

    double2 lu[DW][3][2], lv[DW][3][2];  // windows of both recursions
    double2 P[kUnroll][2];               // gbar by row, turned by (-i)^(w DW)
    double G[kUnroll][2], dd[kUnroll][2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int j = 0; j < DW; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q) lu[j][q][c] = lv[j][q][c] = zero;
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            P[j][c] = zero;
            G[j][c] = dd[j][c] = 0.0;
        }
    }
    RowSet set[2];
    const double ds = op.s2 * op.dshift;
    auto load = [&](RowSet &n, int32_t row) {
        const bool ok = inside(row + 1), okm = mine(row + 1), okk = inside(row);
        const Rsrc re = rsrc(op.onsite, ok ? nb16 / 2 : 0u), rg = rsrc(A.grad, okm ? nb16 / 2 : 0u);
        const uint32_t o8 = ok ? (uint32_t)(row + 1) * row8 : 0u, g8 = okm ? (uint32_t)(row + 1) * row8 : 0u;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n.a[c] = ld2(A.uk1, row + 1, ok, c16[c]);
            n.k[c] = ld2(A.uk2, row, okk, c16[c]);
            n.va[c] = ld2(A.v0, row + 1, ok, c16[c]);
            n.vk[c] = ld2(A.v1, row, okk, c16[c]);
            n.p[c] = ld2(A.gbar, row + 1, ok, c16[c]);
            n.e[c] = bload1(re, c8[c], o8);
            n.g[c] = bload1(rg, s8[c], g8);
        }
    };
    // Slot of a workgroup iteration as in pipe_walk.h (t0 is even here).  All
    // words are counted from the slots read, through an address the compiler
    // does not see into: one register and an offset reach every word (it would
    // keep an address per word, and spill them).
    static_assert(DW % 2 == 0 && 4 * sizeof(RevSlot) <= 65536, "slot offsets");
    LdsBytes *lds = (LdsBytes *)(slots[FIRST ? 0 : w - 1]) + lane * 16;
    asm volatile("" : "+v"(lds));
    constexpr int kWr = FIRST ? 0 : 2 * (int)sizeof(RevSlot);
    auto get = [&](int at) {
        const LdsD2 v = *(const __attribute__((address_space(3))) LdsD2 *)(lds + at);
        return make_double2(v.x, v.y);
    };
    auto put = [&](int at, double2 v) {
        *(__attribute__((address_space(3))) LdsD2 *)(lds + at) = LdsD2{v.x, v.y};
    };
    auto fetch = [&](RowSet &n, int slot) {
        const int at = slot * (int)sizeof(RevSlot);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n.a[c] = get(at + (0 + c) * 1024);
            n.k[c] = get(at + (2 + c) * 1024);
            n.va[c] = get(at + (4 + c) * 1024);
            n.vk[c] = get(at + (6 + c) * 1024);
            n.p[c] = get(at + (8 + c) * 1024);
        }
        const double2 e = get(at + 10 * 1024), g = get(at + 11 * 1024);
        n.e[0] = e.x;
        n.e[1] = e.y;
        n.g[0] = g.x;
        n.g[1] = g.y;
    };
    if (FIRST) {
        load(set[0], sp.st);
    } else {
        for (int32_t t = 0; t + 1 < sp.t0; ++t) row_barrier();
        fetch(set[0], 0);
        arrived(set[0]);
        row_barrier();
    }

    int32_t base = sp.st;
    auto step = [&](auto phc) {
        constexpr int ph = decltype(phc)::value;
        constexpr int n0 = ph % 3, n1 = (ph + 2) % 3, n2 = (ph + 1) % 3;
        const int32_t row = base + ph;
        RowSet &cur = set[ph & 1];
        if constexpr (FIRST)
            load(set[(ph + 1) & 1], row + 1);
        else
            fetch(set[(ph + 1) & 1], (ph & 1) ^ 1);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int sn = (ph + 1) % kUnroll;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            lu[0][n0][c] = cur.a[c];
            lv[0][n0][c] = cur.va[c];
            G[sn][c] = cur.g[c];
            if constexpr (FIRST) {
                dd[sn][c] = fma(op.s2, cur.e[c], ds);
                const double2 b = cur.p[c];
                P[sn][c] = make_double2(fma(A.fac.x, b.x, -(A.fac.y * b.y)), fma(A.fac.x, b.y, A.fac.y * b.x));
            } else {
                dd[sn][c] = cur.e[c];
                P[sn][c] = cur.p[c];
            }
        }
        double2 u[2], v[2];
        auto level = [&](auto lc) {
            constexpr int l = decltype(lc)::value;
            constexpr int sq = (ph - (l - 1) + 4 * kUnroll) % kUnroll;
            const int32_t q = row - (l - 1);
            const double fv = __longlong_as_double(inside(q) ? 0x3FF0000000000000ll : 0ll);
            auto stencil = [&](const double2 (&win)[3][2], int c) {
                const double2 *ctr = win[n1], *up = win[n2], *dn = win[n0];
                const bool even = ((c + ph + l - 1) & 1) == 0;
                const double2 vert = EDGE == CHEBTD_ZIGZAG ? (even ? dn[c] : up[c]) : cadd(up[c], dn[c]);
                double2 h;
                if (EDGE == CHEBTD_ZIGZAG)
                    h = c == 0 ? cadd(from_left0(ctr[1]), ctr[1]) : cadd(ctr[0], from_right0(ctr[0]));
                else if (even)
                    h = c == 0 ? ctr[1] : from_right0(ctr[0]);
                else
                    h = c == 0 ? from_left0(ctr[1]) : ctr[0];
                return make_double2(fma(fv, vert.x, h.x), fma(fv, vert.y, h.y));
            };
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double d = dd[sq][c];
                const double2 uc = lu[l - 1][n1][c], vc = lv[l - 1][n1][c];
                const double2 su = stencil(lu[l - 1], c), sv = stencil(lv[l - 1], c);
                const double2 pu = l == 1 ? cur.k[c] : lu[l >= 2 ? l - 2 : 0][n2][c];
                const double2 pv = l == 1 ? cur.vk[c] : lv[l >= 2 ? l - 2 : 0][n2][c];
                double du = d, ou = off[c], gf = A.gf;
                if (LASTW && l == DW) {  // level 0: H~ u_1 in place of 2 H~
                    du *= A.half;
                    ou *= A.half;
                    gf *= A.half;
                }
                u[c] = add_turned<l - 1>(r[l - 1], P[sq][c],
                                         make_double2(fma(du, uc.x, fma(ou, su.x, -pu.x)),
                                                      fma(du, uc.y, fma(ou, su.y, -pu.y))));
                v[c] = make_double2(fma(d, vc.x, fma(off[c], sv.x, -pv.x)), fma(d, vc.y, fma(off[c], sv.y, -pv.y)));
                G[sq][c] = fma(gf, fma(uc.y, vc.y, uc.x * vc.x), G[sq][c]);
            }
            if constexpr (LASTW && l >= DW - 1) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    st2(l == DW ? A.out2 : A.out1, q, mine(q), s16[c], u[c]);
                    st2(l == DW ? A.vout2 : A.vout1, q, mine(q), s16[c], v[c]);
                }
            }
            if constexpr (l < DW) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    lu[l][n0][c] = u[c];
                    lv[l][n0][c] = v[c];
                }
            }
        };
        level(std::integral_constant<int, 1>{});
        level(std::integral_constant<int, 2>{});
        constexpr int sR = (ph - (DW - 1) + 4 * kUnroll) % kUnroll;
        if constexpr (LASTW) {
            const int32_t R = row - (DW - 1);
            const bool ok = mine(R);
            const Rsrc rg = rsrc(A.grad, ok ? nb16 / 2 : 0u);
#pragma unroll
            for (int c = 0; c < 2; ++c) bstore1(rg, (ok ? (uint32_t)R * row8 : 0u) + s8[c], 0, G[sR][c]);
        } else {
            constexpr int at = kWr + (ph & 1) * (int)sizeof(RevSlot);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                put(at + (0 + c) * 1024, u[c]);
                put(at + (2 + c) * 1024, lu[DW - 1][n2][c]);
                put(at + (4 + c) * 1024, v[c]);
                put(at + (6 + c) * 1024, lv[DW - 1][n2][c]);
                put(at + (8 + c) * 1024, turn<4 * DW - DW>(P[sR][c]));  // (-i)^DW
            }
            put(at + 10 * 1024, make_double2(dd[sR][0], dd[sR][1]));
            put(at + 11 * 1024, make_double2(G[sR][0], G[sR][1]));
        }
        if constexpr (!FIRST) arrived(set[(ph + 1) & 1]);
        row_barrier();
    };
    static_assert(kRevPipeDW == 2, "levels are written out");
    for (int32_t i = 0; i < sp.n; i += kUnroll, base += kUnroll) phases<0, kUnroll>(step);
    for (int32_t t = sp.t0 + sp.n; t < tend; ++t) row_barrier();
}

}  // namespace revdev

template <int EDGE>
__global__ __launch_bounds__(64 * kRevPipeNW, 2) void k_rev_pipe(PipeOp op, RevPipeArgs A)
{
    using namespace revdev;
    constexpr int DW = kRevPipeDW, NW = kRevPipeNW;
    __shared__ RevSlot slots[NW - 1][2];
    const int32_t wg = logical_block(1);
    const int32_t strip = wg / op.nchunks, chunk = wg - strip * op.nchunks;
    const int32_t ys = pipe_row(chunk, op.nchunks, op.W, DW * NW);
    const int32_t ye = pipe_row(chunk + 1, op.nchunks, op.W, DW * NW);
    const int w = pipe_wave<NW>();
    int32_t tend = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        const PipeSpan s = pipe_span(DW, NW, v, ys, ye, op.W);
        tend = max(tend, s.t0 + s.n);
    }
    if (w == 0)
        wave<EDGE, kFirst>(op, A, 0, strip, ys, ye, tend, slots);
    else if (w == NW - 1)
        wave<EDGE, kLast>(op, A, NW - 1, strip, ys, ye, tend, slots);
    else
        wave<EDGE, kMid>(op, A, w, strip, ys, ye, tend, slots);
}

// Every ribbon whose buffer offsets fit: at each size measured, from 8 x 64 to
// 512 x 16384, 1.4 to 2.2 times the rate of the single-wavefront passes (above).
// A forced depth of those (CHEBTD_REV_DEPTH) keeps them.
bool rev_pipe_fits(const Ctx &c)
{
    return c.kind == HKind::Honeycomb && deep_offsets_fit(c.W, c.L) && !std::getenv("CHEBTD_REV_DEPTH");
}

int rev_pipe_chunks(const Ctx &c)
{
    if (const char *env = std::getenv("CHEBTD_REV_CHUNKS")) {
        const int64_t most = std::max<int64_t>(1, (c.W - (kRevPipeDepth - 1)) / 8);
        return (int)std::max<int64_t>(1, std::min<int64_t>(most, std::atoi(env)));
    }
    return pipe_chunks(c.W, c.L, kRevPipeDW, kRevPipeNW, c.num_cus);
}

hipError_t launch_rev_pipe(const Ctx &c, hipStream_t s, int chunks, const RevPipeArgs &A)
{
    if (c.kind != HKind::Honeycomb || !deep_offsets_fit(c.W, c.L) || chunks < 1) return hipErrorInvalidValue;
    PipeOp op{};
    op.onsite = c.eps;
    op.dshift = -c.b;
    op.s2 = 2.0 / c.a;
    op.off2 = -2.0 * c.t_hop / c.a;
    op.W = (int32_t)c.W;
    op.L = (int32_t)c.L;
    op.nstrips = (int32_t)((c.L + pipe_strip_cols(kRevPipeDepth) - 1) / pipe_strip_cols(kRevPipeDepth));
    op.nchunks = chunks;
    const int64_t nb = (int64_t)op.nstrips * op.nchunks;
    if (nb > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nb), block(64 * kRevPipeNW);
    if (c.edge == CHEBTD_ZIGZAG)
        hipLaunchKernelGGL(k_rev_pipe<CHEBTD_ZIGZAG>, grid, block, 0, s, op, A);
    else
        hipLaunchKernelGGL(k_rev_pipe<CHEBTD_ARMCHAIR>, grid, block, 0, s, op, A);
    return hipGetLastError();
}

}  // namespace chebtd
