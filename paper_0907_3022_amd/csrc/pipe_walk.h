// D = DW NW Chebyshev orders in one pass over a honeycomb ribbon (Sect. 2.2
// recursion of arXiv:0907.3022), pipelined over the NW wavefronts of a
// workgroup.
//
// The workgroup walks down a strip of 128 columns (two per lane) row by row.
// Wavefront w carries orders w DW + 1 .. (w+1) DW: level l = 1 .. DW of it
// runs one row behind level l - 1, three rows of each level in registers as in
// deep_walk.h, and what leaves its last level goes through LDS to wavefront
// w + 1, two iterations later: the newest order at row R, the one before it
// at row R - 1, the partial sum and the diagonal term of row R (56 B per
// column).  Only the first wavefront reads memory and only the last one
// writes it: a whole step of D >= M orders reads psi and eps and writes the
// next psi, 40 B per site.
//
// What bounds it: a row of the workgroup's slowest wavefront, two thirds of it
// VALU issue, behind the barrier that ends every row (counted on MI355X: the
// chip's VALU busy 54% of a pass at 1024 x 32768, 28% at 128 x 8192 with 188
// workgroups on 256 CUs; a wavefront issues half of its life and waits a third
// of it; 2.0 and 0.8 TB/s).  Per site and order 10 FP64 instructions (the
// weights are real, see PipeArgs) and 4 lane shifts; two columns per lane
// make the sublattice of every register a constant (no selects) and halve the
// lane shifts, rows outside the lattice are cut off by a factor 0 on the
// vertical bond instead of selects, columns outside by a zero hopping.  The
// price is the halo, D columns per side and D - 1 rows above each chunk.  A value
// that is not finite passes those factors as NaN: such a state spreads along the
// lattice's edge and by the orders past M farther than the M bonds of a step.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "deep_walk.h"
#include "device_ops.h"
#include "pair_walk.h"
#include "pipe.h"

namespace chebtd {

// One row handed from a wavefront to the next, by column of the lane's pair.
struct PipeSlot {
    double2 a[2][64], k[2][64], p[2][64], d[64];
};

namespace pipedev {

using namespace deepdev;
using namespace pairdev;

constexpr int kUnroll = 6;  // window slots (3) times row parity (2)

// Wavefront w's part of a workgroup's walk over the rows [ys, ye): first row
// of level 1 (even; two rows early to fill the windows), the iteration of the
// workgroup at which it starts, and its iterations (whole unrolled bodies).
struct PipeSpan {
    int32_t st, t0, n;
};
__host__ __device__ inline PipeSpan pipe_span(int DW, int NW, int w, int32_t ys, int32_t ye, int32_t W)
{
    const int D = DW * NW;
    auto first = [&](int v) {
        const int32_t b = ys - (D - 1) + v * DW;
        return (b > 0 ? b & ~1 : 0) - 2;
    };
    PipeSpan s;
    s.st = first(w);
    s.t0 = s.st - first(0) + w * (DW + 2);
    const int32_t below = ye - 1 + (D - (w + 1) * DW);
    // last row of level DW handed on: the next wavefront keeps row W at zero,
    // whose v_{k-1} comes with row W + 1
    const int32_t e = below < W + 1 ? below : W + 1;
    s.n = (e + DW - 1 - s.st + 1 + kUnroll - 1) / kUnroll * kUnroll;
    return s;
}

// every lane's LDS traffic of this iteration done, then all wavefronts; loads
// in flight from memory are not waited for
__device__ __forceinline__ void row_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The loads of these values come before this point.  Without it the compiler
// moves LDS reads whose first use lies behind a branch past a row_barrier() in
// front of that branch, where the next wavefront's stores may overtake them.
// Every row read ahead passes here before the barrier, except in the loop of the
// batched kernel, which has no registers left (1049 -> 1202 us for four steps of
// 64 ribbons): there the built code's waits are what a test of it looks at.
__device__ __forceinline__ void arrived(const double2 &v) { asm volatile("" ::"v"(v.x), "v"(v.y)); }
__device__ __forceinline__ void arrived(const double (&v)[2]) { asm volatile("" ::"v"(v[0]), "v"(v[1])); }

constexpr int kHead = 0, kHeadKeep = 1, kFirst = 2, kMid = 3, kLast = 4, kFinal = 5;

struct RowSet {
    double2 a[2], k[2], p[2];
    double e[2];
};
__device__ __forceinline__ void arrived(const RowSet &n)
{
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        arrived(n.a[c]);
        arrived(n.k[c]);
        arrived(n.p[c]);
    }
    arrived(n.e);
}

// i^n (x + iy)
template <int n>
__device__ __forceinline__ double2 turn(double2 v)
{
    if constexpr ((n & 3) == 1) return make_double2(-v.y, v.x);
    if constexpr ((n & 3) == 2) return make_double2(-v.x, -v.y);
    if constexpr ((n & 3) == 3) return make_double2(v.y, -v.x);
    return v;
}
// P += (-i)^l r v
__device__ __forceinline__ void add_order(int l, double r, double2 v, double2 &P)
{
    switch (l & 3) {
        case 0: P.x = fma(r, v.x, P.x); P.y = fma(r, v.y, P.y); break;
        case 1: P.x = fma(r, v.y, P.x); P.y = fma(-r, v.x, P.y); break;
        case 2: P.x = fma(-r, v.x, P.x); P.y = fma(-r, v.y, P.y); break;
        default: P.x = fma(-r, v.y, P.x); P.y = fma(r, v.x, P.y); break;
    }
}

// Wavefront w of the workgroup.  ROLE: kHead (a step's first pass; kHeadKeep
// also copies psi) and kFirst read memory, kLast (acc and the last two orders)
// and kFinal (acc alone) write it, kMid does neither.
template <int EDGE, int DW, int NW, int ROLE, bool GUARD>
__device__ __forceinline__ void wave(const PipeOp &op, const PipeArgs &A, int w, int32_t strip, int32_t ys, int32_t ye,
                                     int32_t tend, PipeSlot (*slots)[2], double &s0, double &s1)
{
    constexpr bool FIRST = ROLE <= kFirst, HEAD = ROLE <= kHeadKeep, LASTW = ROLE >= kLast;
    constexpr int D = DW * NW, HL = pipe_halo_lanes(D), S = pipe_strip_cols(D);
    static_assert(DW >= 2 && DW <= 5 && NW >= 2 && D % 4 == 0 && D <= kMaxPipe, "depth");
    const int lane = threadIdx.x & 63;
    const int32_t W = op.W, L = op.L;
    const int32_t x = strip * S - 2 * HL + 2 * lane;
    const bool in0 = x >= 0 && x < L, in1 = x + 1 >= 0 && x + 1 < L;
    const bool own = lane >= HL && lane < 64 - HL;
    const uint32_t nb16 = (uint32_t)W * (uint32_t)L * 16u, row16 = (uint32_t)L * 16u, row8 = (uint32_t)L * 8u;
    const double2 zero = make_double2(0.0, 0.0);
    // Range checks: lanes outside the lattice's columns get offsets past the
    // buffer (kOut); rows outside the lattice, or not to be stored, a buffer
    // of size 0.  Loads carry the row in the scalar offset (the check does not
    // see it), stores in the lane's (see deep_walk.h).
    auto ld2 = [&](const double2 *p, int32_t row, bool ok, uint32_t lanepart) {
        return bload2(rsrc(p, ok ? nb16 : 0u), lanepart, ok ? (uint32_t)row * row16 : 0u);
    };
    auto st2 = [&](double2 *p, int32_t row, bool ok, uint32_t lanepart, double2 v) {
        bstore2(rsrc(p, ok ? nb16 : 0u), (ok ? (uint32_t)row * row16 : 0u) + lanepart, 0, v);
    };
    auto inside = [&](int32_t row) { return (uint32_t)row < (uint32_t)W; };
    // offsets of the lane's columns: loads, and stores / acc (own columns)
    const uint32_t c16[2] = {in0 ? (uint32_t)x * 16u : kOut, in1 ? (uint32_t)(x + 1) * 16u : kOut};
    const uint32_t c8[2] = {in0 ? (uint32_t)x * 8u : kOut, in1 ? (uint32_t)(x + 1) * 8u : kOut};
    const uint32_t s16[2] = {own ? c16[0] : kOut, own ? c16[1] : kOut};
    // hopping, zero on columns outside the lattice (their values stay zero)
    const double off[2] = {in0 ? op.off2 : 0.0, in1 ? op.off2 : 0.0};
    auto mine = [&](int32_t q) { return q >= ys && q < ye; };

    const PipeSpan sp = pipe_span(DW, NW, w, ys, ye, W);
    double r[DW + 1];
#pragma unroll
    for (int l = 0; l <= DW; ++l) r[l] = A.r[w * DW + l];

    double2 lv[DW][3][2];        // levels 0 .. DW-1, three rows
    double2 P[kUnroll][2];       // partial sums by row
    double dd[kUnroll][2];       // 2 (eps - b) / a by row
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int j = 0; j < DW; ++j) lv[j][0][c] = lv[j][1][c] = lv[j][2][c] = zero;
#pragma unroll
        for (int j = 0; j < kUnroll; ++j) {
            P[j][c] = zero;
            dd[j][c] = 0.0;
        }
    }
    // operands ahead: from memory two rows ahead at a step's head (12
    // registers a row), one elsewhere (28 a row); from LDS one
    constexpr int K = HEAD ? 3 : 2;
    RowSet set[K];
    const double ds = op.s2 * op.dshift;
    auto load = [&](RowSet &n, int32_t row) {  // for the iteration whose level 1 is at `row`
        const bool ok = inside(row + 1);
        const Rsrc re = rsrc(op.onsite, ok ? nb16 / 2 : 0u);
        const uint32_t o8 = ok ? (uint32_t)(row + 1) * row8 : 0u;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n.a[c] = ld2(A.vk, row + 1, ok, c16[c]);
            n.e[c] = bload1(re, c8[c], o8);
            if (!HEAD) {
                n.k[c] = ld2(A.vkm1, row, inside(row), c16[c]);
                n.p[c] = ld2(A.acc_in, row + 1, mine(row + 1), s16[c]);
            }
        }
    };
    auto fetch = [&](RowSet &n, const PipeSlot *q) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            n.a[c] = q->a[c][lane];
            n.k[c] = q->k[c][lane];
            n.p[c] = q->p[c][lane];
        }
        const double2 e = q->d[lane];
        n.e[0] = e.x;
        n.e[1] = e.y;
    };
    // workgroup iteration t writes slot t & 1 and reads what t - 1 wrote
    const int tb = sp.t0 & 1;
    PipeSlot *wr[2] = {nullptr, nullptr};
    const PipeSlot *rd[2] = {nullptr, nullptr};
    if (!LASTW) {
        wr[0] = &slots[w][tb];
        wr[1] = &slots[w][tb ^ 1];
    }
    if (!FIRST) {
        rd[0] = &slots[w - 1][tb ^ 1];
        rd[1] = &slots[w - 1][tb];
    }
    if (FIRST) {
#pragma unroll
        for (int j = 0; j + 1 < K; ++j) load(set[j], sp.st + j);
    } else {
        for (int32_t t = 0; t + 1 < sp.t0; ++t) row_barrier();
        fetch(set[0], rd[1]);
        arrived(set[0]);
        row_barrier();
    }

    int32_t base = sp.st;  // row of level 1 at the body's first iteration
    auto step = [&](auto phc) {
        constexpr int ph = decltype(phc)::value;
        constexpr int n0 = ph % 3, n1 = (ph + 2) % 3, n2 = (ph + 1) % 3;  // newest, centre, oldest row
        const int32_t row = base + ph;
        RowSet &cur = set[ph % K];
        if constexpr (FIRST)
            load(set[(ph + K - 1) % K], row + K - 1);
        else
            fetch(set[(ph + 1) % K], rd[ph & 1]);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int sn = (ph + 1) % kUnroll;  // slot of row + 1
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            lv[0][n0][c] = cur.a[c];
            if constexpr (FIRST)
                dd[sn][c] = fma(op.s2, cur.e[c], ds);
            else
                dd[sn][c] = cur.e[c];
            P[sn][c] = HEAD ? cscale(r[0], cur.a[c]) : cur.p[c];
            if constexpr (ROLE == kHeadKeep) st2(A.ckpt, row + 1, mine(row + 1), s16[c], cur.a[c]);
        }
        double2 v[2];
#pragma unroll
        for (int l = 1; l <= DW; ++l) {
            const int32_t q = row - (l - 1);
            constexpr int R6 = 4 * kUnroll;
            const int sq = (ph - (l - 1) + R6) % kUnroll;
            // 1 on the lattice's rows: a bond across its first or last row is none
            const double fv = __longlong_as_double((uint32_t)q < (uint32_t)W ? 0x3FF0000000000000ll : 0ll);
            const double2 *ctr = lv[l - 1][n1], *up = lv[l - 1][n2], *dn = lv[l - 1][n0];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const bool even = ((c + ph + l - 1) & 1) == 0;  // of column + row
                const double2 vert = EDGE == CHEBTD_ZIGZAG ? (even ? dn[c] : up[c]) : cadd(up[c], dn[c]);
                double2 h;
                if (EDGE == CHEBTD_ZIGZAG)
                    h = c == 0 ? cadd(from_left0(ctr[1]), ctr[1]) : cadd(ctr[0], from_right0(ctr[0]));
                else if (even)
                    h = c == 0 ? ctr[1] : from_right0(ctr[0]);
                else
                    h = c == 0 ? from_left0(ctr[1]) : ctr[0];
                const double2 s = make_double2(fma(fv, vert.x, h.x), fma(fv, vert.y, h.y));
                double d = dd[sq][c], o = off[c];
                if (HEAD && l == 1) {  // v_1 = H~ psi
                    d *= 0.5;
                    o *= 0.5;
                    v[c] = make_double2(fma(d, ctr[c].x, o * s.x), fma(d, ctr[c].y, o * s.y));
                    // rows of the chunk only; the lanes are sorted out after the walk
                    const double m = __longlong_as_double(mine(q) ? 0x3FF0000000000000ll : 0ll);
                    s0 = fma(m, fma(ctr[c].y, ctr[c].y, ctr[c].x * ctr[c].x), s0);
                    s1 = fma(m, fma(ctr[c].y, v[c].y, ctr[c].x * v[c].x), s1);
                } else {
                    const double2 pv = l == 1 ? cur.k[c] : lv[l >= 2 ? l - 2 : 0][n2][c];
                    v[c] = make_double2(fma(d, ctr[c].x, fma(o, s.x, -pv.x)), fma(d, ctr[c].y, fma(o, s.y, -pv.y)));
                }
                add_order(l, r[l], v[c], P[sq][c]);
            }
            if (ROLE == kLast && l >= DW - 1) {
#pragma unroll
                for (int c = 0; c < 2; ++c) st2(l == DW ? A.out2 : A.out1, q, mine(q), s16[c], v[c]);
            }
            if (l < DW) {
                lv[l][n0][0] = v[0];
                lv[l][n0][1] = v[1];
            }
        }
        // row R = row - (DW - 1) is through
        constexpr int sR = (ph - (DW - 1) + 4 * kUnroll) % kUnroll;
        if constexpr (LASTW) {
            const int32_t R = row - (DW - 1);
            const bool ok = mine(R);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                // the last wavefront's sum is turned by i^((NW - 1) DW)
                const double2 p = turn<4 * NW - (NW - 1) * DW + 4 * DW * NW>(P[sR][c]);
                const double2 o =
                    make_double2(fma(A.fin.x, p.x, -(A.fin.y * p.y)), fma(A.fin.x, p.y, A.fin.y * p.x));
                const double m = __longlong_as_double(ok ? 0x3FF0000000000000ll : 0ll);
                s0 = fma(m, fma(o.y, o.y, o.x * o.x), s0);
                st2(A.acc_out, R, ok, s16[c], o);
            }
        } else {
            PipeSlot *q = wr[ph & 1];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                q->a[c][lane] = v[c];
                q->k[c][lane] = lv[DW - 1][n2][c];
                q->p[c][lane] = turn<DW>(P[sR][c]);
            }
            q->d[lane] = make_double2(dd[sR][0], dd[sR][1]);
        }
        if constexpr (!FIRST && GUARD) arrived(set[(ph + 1) % K]);
        row_barrier();
    };
    for (int32_t i = 0; i < sp.n; i += kUnroll, base += kUnroll) phases<0, kUnroll>(step);
    for (int32_t t = sp.t0 + sp.n; t < tend; ++t) row_barrier();
    if (!own) s0 = s1 = 0.0;
}

}  // namespace pipedev

// This wavefront's place in the pipeline.  The first and last have more to do
// than the others; the second workgroup that a CU receives (256 workgroups on)
// numbers its wavefronts the other way round, so that the two firsts do not
// share a SIMD.
template <int NW>
__device__ __forceinline__ int pipe_wave()
{
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    return NW == 4 && (blockIdx.x >> 8 & 1) ? NW - 1 - w : w;
}

// The workgroup's share: strip `strip`, rows [ys, ye).  sums: <v0|v0> and
// <v0|H~ v0> of a head pass (wavefront 0's lanes), sum |acc|^2 (the last
// wavefront's).
template <int EDGE, int DW, int NW, bool GUARD = true>
__device__ __forceinline__ void pipe_block(const PipeOp &op, const PipeArgs &A, int32_t strip, int32_t ys, int32_t ye,
                                           PipeSlot (*slots)[2], double &s0, double &s1)
{
    using namespace pipedev;
    const int w = pipe_wave<NW>();
    int32_t tend = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        const PipeSpan s = pipe_span(DW, NW, v, ys, ye, op.W);
        tend = max(tend, s.t0 + s.n);
    }
    if (w == 0) {
        if (A.vkm1 == nullptr && A.ckpt == nullptr)
            wave<EDGE, DW, NW, kHead, GUARD>(op, A, 0, strip, ys, ye, tend, slots, s0, s1);
        else if (A.vkm1 == nullptr)
            wave<EDGE, DW, NW, kHeadKeep, GUARD>(op, A, 0, strip, ys, ye, tend, slots, s0, s1);
        else
            wave<EDGE, DW, NW, kFirst, GUARD>(op, A, 0, strip, ys, ye, tend, slots, s0, s1);
    } else if (w == NW - 1) {
        if (A.out2 == nullptr)
            wave<EDGE, DW, NW, kFinal, GUARD>(op, A, NW - 1, strip, ys, ye, tend, slots, s0, s1);
        else
            wave<EDGE, DW, NW, kLast, GUARD>(op, A, NW - 1, strip, ys, ye, tend, slots, s0, s1);
    } else {
        wave<EDGE, DW, NW, kMid, GUARD>(op, A, w, strip, ys, ye, tend, slots, s0, s1);
    }
}

}  // namespace chebtd
