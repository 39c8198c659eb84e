// Many Chebyshev orders per pass over a 1D chain longer than the whole-run
// kernels take (Sect. 3.1 Hamiltonian, Sect. 2.2 recursion of
// arXiv:0907.3022).
//
// A wavefront holds 64 R consecutive sites in registers, R per lane, of which
// the outer D on each side are halo: an order spoils one site per side, so
// after D orders exactly its own 64 R - 2 D are right.  A pass then reads
// v_{k-1}, v_k, V and acc once and writes acc (and the last two orders if
// another pass follows) for all D orders: 40 B per site where one pass takes
// the whole step.  No LDS, no barrier: wavefronts are independent.
//
// What bounds it: a wavefront's issue and its dependent chain (half of its life
// each, counted at 65536 sites), 8 FP64 instructions per site and order and 8
// lane shifts per R sites; below about 10^5 sites the launch and the chain of
// orders itself (0.10 us an order with four sites per lane).  Measured on
// MI355X, us per step of 64 orders, passes of two and three orders before:
// 142 -> 9.9 at 65536 sites, 670 -> 36 at 2^20, 2961 -> 115 at 4 million.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "chain_tile.h"
#include "device_ops.h"
#include "internal.h"
#include "pair.h"
#include "pair_walk.h"

namespace chebtd {

// INSIDE: every site of the wavefront lies on the chain
template <int R, bool INSIDE>
__device__ __forceinline__ void tile_wave(const TileOp &op, const TileArgs &A, int64_t base, double &s0, double &s1,
                                          double &sk)
{
    using namespace pairdev;
    const int lane = threadIdx.x & 63;
    const int D = A.D;
    const int32_t j0 = lane * R;
    const int64_t i0 = base + j0;
    const double2 zero = make_double2(0.0, 0.0);
    const bool head = A.vkm1 == nullptr;
    double d[R], o[INSIDE ? 1 : R];
    double2 X[R], Y[R], P[R];  // v_{k-1}, v_k and the partial sum
    bool own[R];
    o[0] = op.off2;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = i0 + r;
        const bool in = INSIDE || (i >= 0 && i < op.n);
        const bool mid = j0 + r >= D && j0 + r < 64 * R - D;
        own[r] = in && mid;
        d[r] = in ? op.s2 * (op.V[i] + op.dsh) : 0.0;
        if (!INSIDE) o[r] = in ? op.off2 : 0.0;  // sites off the chain stay zero
        Y[r] = in ? A.vk[i] : zero;
        X[r] = !head && in ? A.vkm1[i] : zero;
        P[r] = !head && own[r] ? A.acc_in[i] : zero;
    }
    auto off = [&](int r) { return o[INSIDE ? 0 : r]; };
    // X <- 2 H~ Y - X
    auto apply = [&](double2 (&x)[R], const double2 (&y)[R]) {
        const double2 l0 = from_left0(y[R - 1]), rR = from_right0(y[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double2 l = r == 0 ? l0 : y[r > 0 ? r - 1 : 0], g = r == R - 1 ? rR : y[r < R - 1 ? r + 1 : r];
            const double sx = l.x + g.x, sy = l.y + g.y;
            x[r] = make_double2(fma(d[r], y[r].x, fma(off(r), sx, -x[r].x)),
                                fma(d[r], y[r].y, fma(off(r), sy, -x[r].y)));
        }
    };
    // P += (-i)^l w v
    auto add = [&](auto lc, double w, const double2 (&v)[R]) {
        constexpr int l = decltype(lc)::value & 3;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double a = l & 1 ? v[r].y : v[r].x, b = l & 1 ? v[r].x : v[r].y;
            P[r].x = fma(l >= 2 ? -w : w, a, P[r].x);
            P[r].y = fma(l == 1 || l == 2 ? -w : w, b, P[r].y);
        }
    };
    // P's frame during the pass: i^k times the partial sum, k the orders
    // before the loop
    int k = A.k0, left = D;
    const double *w = A.r + 1;
    if (head) {
        // v_1 = H~ psi: half of 2 H~ psi
        apply(X, Y);
        const double r0 = A.r[0], r1 = A.r[1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            X[r] = make_double2(0.5 * X[r].x, 0.5 * X[r].y);
            s0 += own[r] ? Y[r].x * Y[r].x + Y[r].y * Y[r].y : 0.0;
            s1 += own[r] ? Y[r].x * X[r].x + Y[r].y * X[r].y : 0.0;
            if (A.ckpt && own[r]) A.ckpt[i0 + r] = Y[r];
            // i (r0 psi - i r1 v_1)
            P[r] = make_double2(fma(r1, X[r].x, -r0 * Y[r].y), fma(r1, X[r].y, r0 * Y[r].x));
            const double2 t = X[r];
            X[r] = Y[r];
            Y[r] = t;
        }
        k = 1;
        --left;
        ++w;
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) P[r] = turn_by(k, P[r]);
    }
    // four orders an iteration, their weights read one iteration ahead
    double w0 = w[0], w1 = w[1], w2 = w[2], w3 = w[3];
    for (; left >= 4; left -= 4) {
        w += 4;
        const double n0 = w[0], n1 = w[1], n2 = w[2], n3 = w[3];
        apply(X, Y);
        add(std::integral_constant<int, 1>{}, w0, X);
        apply(Y, X);
        add(std::integral_constant<int, 2>{}, w1, Y);
        apply(X, Y);
        add(std::integral_constant<int, 3>{}, w2, X);
        apply(Y, X);
        add(std::integral_constant<int, 0>{}, w3, Y);
        w0 = n0;
        w1 = n1;
        w2 = n2;
        w3 = n3;
    }
    if (left >= 1) {
        apply(X, Y);
        add(std::integral_constant<int, 1>{}, w0, X);
    }
    if (left >= 2) {
        apply(Y, X);
        add(std::integral_constant<int, 2>{}, w1, Y);
    }
    if (left >= 3) {
        apply(X, Y);
        add(std::integral_constant<int, 3>{}, w2, X);
    }
    const bool swapped = left & 1;  // the newest order is in X
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!own[r]) continue;
        const double2 p = turn_by(4 - (k & 3), P[r]);
        const double2 a = make_double2(fma(A.fin.x, p.x, -(A.fin.y * p.y)), fma(A.fin.x, p.y, A.fin.y * p.x));
        A.acc_out[i0 + r] = a;
        sk += a.x * a.x + a.y * a.y;
        if (A.out2) {
            A.out1[i0 + r] = csel(swapped, Y[r], X[r]);
            A.out2[i0 + r] = csel(swapped, X[r], Y[r]);
        }
    }
}

template <int R>
__global__ __launch_bounds__(256) void k_chain_tile(TileOp op, TileArgs A, double *partials, double *knorm)
{
    __shared__ double red[2 * 4];
    const int64_t S = 64 * R - 2 * A.D;
    const int64_t gw = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t base = gw * S - A.D;
    double s0 = 0.0, s1 = 0.0, sk = 0.0, z = 0.0;
    if (gw * S < op.n) {  // uniform per wavefront
        if (base >= 0 && base + 64 * R <= op.n)
            tile_wave<R, true>(op, A, base, s0, s1, sk);
        else
            tile_wave<R, false>(op, A, base, s0, s1, sk);
    }
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

int64_t tile_blocks(const Ctx &c, int R, int D)
{
    const int64_t S = 64 * R - 2 * D, waves = (c.n + S - 1) / S;
    return (waves + 3) / 4;
}

// Sites per lane and orders per pass.  An order costs a wavefront 8 R + 12
// instructions; a SIMD runs one wavefront's at 2.3 ns each and shares itself
// from there on (1.9 ns); a pass adds its launch (3 us) and its traffic.  More
// sites per lane spend less on halo, fewer fill the chip: 64 orders of a
// 65536-site chain take 10.9 / 9.9 / 14.8 us with 2 (two passes) / 4 / 8 sites
// per lane, of 2^20 sites 71 / 45 / 36 us.  Chains past the deep walk's 32-bit
// offsets keep two-order passes, as does a forced depth (CHEBTD_DEPTH).
// CHEBTD_TILE=R,D overrides, 0 turns tiled passes off.
TilePlan plan_tile(const Ctx &c, int M)
{
    TilePlan best;
    if (c.kind != HKind::Chain || M < 2 || !deep_offsets_fit(1, c.n) || std::getenv("CHEBTD_DEPTH")) return best;
    int fr = 0, fd = 0;
    if (const char *env = std::getenv("CHEBTD_TILE"))
        if (std::sscanf(env, "%d,%d", &fr, &fd) != 2 || fd < 2) return best;
    double bt = 1e300;
    for (int R : {2, 4, 8}) {
        if (fr && R != fr) continue;
        // from the fewest passes that leave 8 R own sites, or that a forced depth needs
        const int fewest = fd ? (M + fd - 1) / fd : (2 * M + 56 * R - 1) / (56 * R);
        for (int p = std::max(1, fewest); p <= std::min(M / 2, 4 * fewest + 8); ++p) {
            const int D = (M + p - 1) / p, S = 64 * R - 2 * D;
            if (S < 8 * R || (fd && D > fd)) continue;
            const double waves = (double)((c.n + S - 1) / S), simds = 4.0 * c.num_cus;
            const double share = std::max(1.0, 0.84 * std::ceil(waves / simds));
            const double t = p * (3.0 + D * (8 * R + 12) * 2.3e-3 * share + (p == 1 ? 40.0 : 90.0) * c.n / 5.0e6);
            if (t < bt) {
                bt = t;
                best.R = R;
                best.depths.assign((size_t)p, D);
                for (int q = 0, over = D * p - M; q < over; ++q) --best.depths[(size_t)(p - 1 - q)];
            }
        }
    }
    return best;
}

hipError_t launch_tile(const Ctx &c, hipStream_t s, int R, const TileArgs &A, double *partials, double *knorm)
{
    const int64_t nb = tile_blocks(c, R, A.D);
    if (A.D < 1 || 64 * R - 2 * A.D < 1 || nb < 1 || nb > INT32_MAX || (!A.vkm1 && A.k0 != 0))
        return hipErrorInvalidValue;
    TileOp op{c.V, 1.0 / (c.dx * c.dx) - c.b, 2.0 / c.a, 2.0 * (-0.5 / (c.dx * c.dx)) / c.a, c.n};
    const dim3 grid((unsigned)nb), block(256);
    if (R == 2)
        hipLaunchKernelGGL(k_chain_tile<2>, grid, block, 0, s, op, A, partials, knorm);
    else if (R == 4)
        hipLaunchKernelGGL(k_chain_tile<4>, grid, block, 0, s, op, A, partials, knorm);
    else if (R == 8)
        hipLaunchKernelGGL(k_chain_tile<8>, grid, block, 0, s, op, A, partials, knorm);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace chebtd
