// Many Chebyshev orders in one pass over a narrow ribbon (Sect. 2.2
// recursion of arXiv:0907.3022), W <= 48: a workgroup holds a strip of 128 columns of
// all W rows in registers, RW rows by two columns per lane, and runs the D
// orders in place.  Between orders each wavefront passes its first and last
// row to its neighbours through LDS, one barrier per order.  An order spoils
// one column per side, so 128 - 4 ceil(D / 2) columns are the workgroup's own;
// there is no halo in the rows.
//
// What bounds it: the chain of orders, each a wavefront's issue (10 FP64
// instructions and 4 or 2 lane shifts per site) and a barrier, at which it waits
// as long (counted: issuing 36% of its life, waiting 38% at 10 x 1000), and for the
// few workgroups of a small ribbon the launch.  Against the pipelined passes (pipe_walk.h) it has
// no pipeline to fill and no rows to repeat, which is what a narrow ribbon
// spends its time on there.  Measured on MI355X, us per step of 20 orders,
// pipelined -> here: 6 x 200 17.6 -> 8.0, armchair 10 x 1000 19.9 -> 10.5 (69
// orders: 61 -> 29), 32 x 512 31.7 -> 15.9, 16 x 20000 23.5 -> 11.6, 45 x 6000
// 32 -> 23, 40 x 32768 51 -> 45.  Past 48 rows the registers end: eight rows
// per wavefront spill (64 x 1450: 32 -> 41 with the diagonal in LDS).
//
// A site's arithmetic is that of the pipelined passes, bit for bit; values that are
// not finite spread along the edge as there.
#pragma once

#include <hip/hip_runtime.h>

#include "pipe_walk.h"
#include "ribbon_tile.h"

namespace chebtd {

// first and last row of each wavefront (slots 1 .. NW; 0 and NW + 1 stay
// zero), by column of the lane's pair, for the order in flight and the next
struct TileEdges {
    double2 first[2][64], last[2][64];
};

namespace rtiledev {

using namespace deepdev;
using namespace pairdev;

// edges: [2][NW + 2].  Wavefront w of NW = ceil(W / RW).
template <int EDGE, int RW>
__device__ __forceinline__ void wave(const PipeOp &op, const TileArgs &A, int w, int NW, int32_t strip,
                                     TileEdges *edges, double &s0, double &s1, double &sk)
{
    const int lane = threadIdx.x & 63;
    const int D = A.D, HL = (D + 1) / 2, S = 128 - 4 * HL;
    const int32_t W = op.W, L = op.L, y0 = w * RW;
    const int32_t x = strip * S - 2 * HL + 2 * lane;
    const bool in[2] = {x >= 0 && x < L, x + 1 >= 0 && x + 1 < L};
    const bool mid = lane >= HL && lane < 64 - HL;
    const bool own[2] = {mid && in[0], mid && in[1]};
    const double off[2] = {in[0] ? op.off2 : 0.0, in[1] ? op.off2 : 0.0};
    const double2 zero = make_double2(0.0, 0.0);
    const bool head = A.vkm1 == nullptr;
    const uint32_t nb16 = (uint32_t)W * (uint32_t)L * 16u, row16 = (uint32_t)L * 16u, row8 = (uint32_t)L * 8u;
    // rows past the ribbon: a buffer of size 0; columns outside: kOut (see
    // pipe_walk.h)
    auto ld2 = [&](const double2 *p, int32_t row, bool ok, uint32_t lanepart) {
        return bload2(rsrc(p ? p : A.vk, p && ok ? nb16 : 0u), lanepart, ok ? (uint32_t)row * row16 : 0u);
    };
    auto st2 = [&](double2 *p, int32_t row, bool ok, uint32_t lanepart, double2 v) {
        bstore2(rsrc(p ? p : A.acc_out, p && ok ? nb16 : 0u), (ok ? (uint32_t)row * row16 : 0u) + lanepart, 0, v);
    };
    const uint32_t c16[2] = {in[0] ? (uint32_t)x * 16u : kOut, in[1] ? (uint32_t)(x + 1) * 16u : kOut};
    const uint32_t c8[2] = {in[0] ? (uint32_t)x * 8u : kOut, in[1] ? (uint32_t)(x + 1) * 8u : kOut};
    const uint32_t s16[2] = {mid ? c16[0] : kOut, mid ? c16[1] : kOut};

    double2 X[RW][2], Y[RW][2], P[RW][2];  // v_{k-1}, v_k, the partial sum
    double d[RW][2];
    const double ds = op.s2 * op.dshift;
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const bool ok = y0 + i < W;
        const Rsrc re = rsrc(op.onsite, ok ? nb16 / 2 : 0u);
        const uint32_t o8 = ok ? (uint32_t)(y0 + i) * row8 : 0u;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            Y[i][c] = ld2(A.vk, y0 + i, ok, c16[c]);
            X[i][c] = ld2(head ? nullptr : A.vkm1, y0 + i, ok, c16[c]);
            P[i][c] = ld2(head ? nullptr : A.acc_in, y0 + i, ok, s16[c]);
            d[i][c] = fma(op.s2, bload1(re, c8[c], o8), ds);
        }
    }
    int buf = 0;
    auto publish = [&](const double2 (&v)[RW][2]) {
        TileEdges &e = edges[buf * (NW + 2) + w + 1];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (EDGE == CHEBTD_ZIGZAG && c == 0) continue;  // see apply
            e.first[c][lane] = v[0][c];
            e.last[c][lane] = v[RW - 1][c];
        }
        pipedev::row_barrier();
    };
    // x <- 2 H~ y - x, y's outside rows from LDS.  RW is even, so a row's
    // parity is its index's; on zigzag edges only odd columns bond across the
    // wavefront's first and last row
    auto apply = [&](double2 (&v)[RW][2], const double2 (&y)[RW][2]) {
        const TileEdges *e = edges + buf * (NW + 2) + w;
        double2 up0[2], dnL[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (EDGE == CHEBTD_ZIGZAG && c == 0) {
                up0[c] = dnL[c] = zero;
                continue;
            }
            up0[c] = e[0].last[c][lane];
            dnL[c] = e[2].first[c][lane];
        }
        buf ^= 1;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            const double fv = __longlong_as_double(y0 + i < W ? 0x3FF0000000000000ll : 0ll);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const bool even = ((c + i) & 1) == 0;
                const double2 up = i > 0 ? y[i > 0 ? i - 1 : 0][c] : up0[c];
                const double2 dn = i + 1 < RW ? y[i + 1 < RW ? i + 1 : i][c] : dnL[c];
                const double2 vert = EDGE == CHEBTD_ZIGZAG ? (even ? dn : up) : cadd(up, dn);
                double2 h;
                if (EDGE == CHEBTD_ZIGZAG)
                    h = c == 0 ? cadd(from_left0(y[i][1]), y[i][1]) : cadd(y[i][0], from_right0(y[i][0]));
                else if (even)
                    h = c == 0 ? y[i][1] : from_right0(y[i][0]);
                else
                    h = c == 0 ? from_left0(y[i][1]) : y[i][0];
                const double2 s = make_double2(fma(fv, vert.x, h.x), fma(fv, vert.y, h.y));
                v[i][c] = make_double2(fma(d[i][c], y[i][c].x, fma(off[c], s.x, -v[i][c].x)),
                                       fma(d[i][c], y[i][c].y, fma(off[c], s.y, -v[i][c].y)));
            }
        }
    };
    auto add = [&](auto lc, double wt, const double2 (&v)[RW][2]) {
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) pipedev::add_order(decltype(lc)::value, wt, v[i][c], P[i][c]);
    };
    using std::integral_constant;
    // P's frame during the pass: i^k times the partial sum, k the orders
    // before the loop
    int k = A.k0, left = D;
    const double *wp = A.r + 1;
    publish(Y);
    if (head) {
        apply(X, Y);  // 2 H~ psi
        const double r0 = A.r[0], r1 = A.r[1];
#pragma unroll
        for (int i = 0; i < RW; ++i) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const double2 q = Y[i][c];
                X[i][c] = make_double2(0.5 * X[i][c].x, 0.5 * X[i][c].y);
                const double2 v = X[i][c];
                s0 += own[c] ? q.x * q.x + q.y * q.y : 0.0;
                s1 += own[c] ? q.x * v.x + q.y * v.y : 0.0;
                if (A.ckpt) st2(A.ckpt, y0 + i, y0 + i < W, s16[c], q);
                // i (r0 psi - i r1 v_1)
                P[i][c] = make_double2(fma(r1, v.x, -(r0 * q.y)), fma(r1, v.y, r0 * q.x));
                X[i][c] = q;
                Y[i][c] = v;
            }
        }
        k = 1;
        --left;
        ++wp;
        if (left) publish(Y);
    } else {
#pragma unroll
        for (int i = 0; i < RW; ++i)
#pragma unroll
            for (int c = 0; c < 2; ++c) P[i][c] = turn_by(k, P[i][c]);
    }
    // four orders an iteration, their weights read one iteration ahead
    double w0 = wp[0], w1 = wp[1], w2 = wp[2], w3 = wp[3];
    for (; left >= 4; left -= 4) {
        wp += 4;
        const double n0 = wp[0], n1 = wp[1], n2 = wp[2], n3 = wp[3];
        apply(X, Y);
        publish(X);
        add(integral_constant<int, 1>{}, w0, X);
        apply(Y, X);
        publish(Y);
        add(integral_constant<int, 2>{}, w1, Y);
        apply(X, Y);
        publish(X);
        add(integral_constant<int, 3>{}, w2, X);
        apply(Y, X);
        publish(Y);
        add(integral_constant<int, 0>{}, w3, Y);
        w0 = n0;
        w1 = n1;
        w2 = n2;
        w3 = n3;
    }
    if (left >= 1) {
        apply(X, Y);
        if (left >= 2) publish(X);
        add(integral_constant<int, 1>{}, w0, X);
    }
    if (left >= 2) {
        apply(Y, X);
        if (left >= 3) publish(Y);
        add(integral_constant<int, 2>{}, w1, Y);
    }
    if (left >= 3) {
        apply(X, Y);
        add(integral_constant<int, 3>{}, w2, X);
    }
    const bool swapped = left & 1;  // the newest order is in X
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        const bool ok = y0 + i < W;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const double2 p = turn_by(4 - (k & 3), P[i][c]);
            const double2 a = make_double2(fma(A.fin.x, p.x, -(A.fin.y * p.y)), fma(A.fin.x, p.y, A.fin.y * p.x));
            st2(A.acc_out, y0 + i, ok, s16[c], a);
            sk += ok && own[c] ? a.x * a.x + a.y * a.y : 0.0;
            if (A.out2) {
                st2(A.out1, y0 + i, ok, s16[c], csel(swapped, Y[i][c], X[i][c]));
                st2(A.out2, y0 + i, ok, s16[c], csel(swapped, X[i][c], Y[i][c]));
            }
        }
    }
}

}  // namespace rtiledev

// The workgroup's strip; edges: [2][NW + 2].
template <int EDGE, int RW>
__device__ __forceinline__ void ribbon_tile_block(const PipeOp &op, const TileArgs &A, int32_t strip, int NW,
                                                  TileEdges *edges, double &s0, double &s1, double &sk)
{
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    // the slots beside the first and last wavefront are read as zero rows
    if (w == 0) {
        const double2 zero = make_double2(0.0, 0.0);
        for (int b = 0; b < 2; ++b) {
            TileEdges &lo = edges[b * (NW + 2)], &hi = edges[b * (NW + 2) + NW + 1];
#pragma unroll
            for (int c = 0; c < 2; ++c) lo.last[c][lane] = hi.first[c][lane] = zero;
        }
    }
    rtiledev::wave<EDGE, RW>(op, A, w, NW, strip, edges, s0, s1, sk);
}

}  // namespace chebtd
