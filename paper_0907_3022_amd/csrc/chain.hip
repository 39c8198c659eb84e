// Whole runs of a short 1D chain (Sect. 3.1 of arXiv:0907.3022, the double
// well on N <= 4096 grid points) in one launch: every step of the Chebyshev
// propagator (Sect. 2.2) with all vectors in registers, in one workgroup
// (k_chain_small) or, past 128 sites, spread over workgroups of one
// wavefront that exchange halo strips every few dozen orders (k_chain_multi).
//
// k_chain_small:
// T = 256 or 512 threads (one or two wavefronts per SIMD); thread t owns
// sites t*R .. t*R+R-1.
// One recursion order is
//   X <- 2 H~ Y - X        (v_{k+1} written over v_{k-1} in place)
//   acc += g_{k+1} X
// so two orders per loop iteration swap the roles of the two register
// arrays without copies.  Neighbours across lanes move by DPP wave shifts;
// the first and last site of each wavefront go through LDS (double
// buffered), one barrier per order, and the interior sites are computed
// while those LDS reads are in flight.  Sites past the end of the chain have
// zero coefficients, so they stay zero and act as the Dirichlet boundary.
// The step weights are read from LDS when they fit there.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "device_ops.h"
#include "internal.h"
#include "pair_walk.h"
#include "pipe.h"

namespace chebtd {

namespace {


template <int R>
struct ChainRegs {
    double d[R];  // 2 (H_ii - b) / a
    double o[R];  // 2 H_{i,i+-1} / a (0 past the end)
};

}  // namespace

// The real weights r_k of gamma_k = e^{-ib dt} (-i)^k r_k (J_0, 2 J_k) add to
// acc / e^{-ib dt}: P += (-i)^k r v.  With the sign of (-i)^k folded into the
// weight (w_k = r_k, negated for k mod 4 = 2, 3) an even order adds w v, an
// odd one -i w v.
__device__ __forceinline__ double signed_weight(const double *rw, int k) { return k & 2 ? -rw[k] : rw[k]; }
template <bool ODD, int R>
__device__ __forceinline__ void add_order(double w, const double2 (&v)[R], double2 (&P)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        P[r].x = fma(w, ODD ? v[r].y : v[r].x, P[r].x);
        P[r].y = fma(ODD ? -w : w, ODD ? v[r].x : v[r].y, P[r].y);
    }
}
// acc after the head's two orders, r0 psi - i r1 v_1, and the step's end
__device__ __forceinline__ double2 head_orders(double r0, double r1, double2 psi, double2 v1)
{
    return make_double2(fma(r1, v1.y, r0 * psi.x), fma(-r1, v1.x, r0 * psi.y));
}
__device__ __forceinline__ double2 with_phase(double2 f, double2 p)
{
    return make_double2(fma(f.x, p.x, -(f.y * p.y)), fma(f.x, p.y, f.y * p.x));
}

// G_LDS: the step weights r_0..r_M are copied to LDS first, so that reading
// them never waits behind a scalar-cache miss (scalar loads share a wait
// counter with LDS, and the per-order edge exchange waits on it).
template <int R, int T, bool G_LDS>
__global__ __launch_bounds__(T) void k_chain_small(OpChain op, const double2 *psi_in, double2 *psi_out,
                                                   const double *__restrict__ rw, double2 phase, int M, int64_t K,
                                                   double a, double b, double *norm_out, double *energy_out,
                                                   double2 *ckpt)
{
    using namespace pairdev;
    constexpr int NW = T / 64;
    __shared__ double2 edge_lo[2][NW], edge_hi[2][NW];  // first / last site of each wavefront
    __shared__ double red[2 * NW];
    extern __shared__ double g_lds[];  // r_0..r_M when G_LDS
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int64_t row0 = (int64_t)tid * R;
    const double2 zero = make_double2(0.0, 0.0);
    ChainRegs<R> c;
    double2 A[R], B[R], acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = row0 + r;
        const bool ok = i < op.n;
        c.d[r] = ok ? op.s2 * (op.V[i] + op.dsh) : 0.0;
        c.o[r] = ok ? op.off2 : 0.0;
        B[r] = ok ? psi_in[i] : zero;
        A[r] = zero;
    }
    const double *wt = rw;
    if (G_LDS) {
        for (int k = tid; k <= M; k += T) g_lds[k] = signed_weight(rw, k);
        wt = g_lds;  // the barrier in the first publish() orders these writes
    }
    int buf = 0;
    auto publish = [&](const double2 (&X)[R]) {
        if (lane == 0) edge_lo[buf][wave] = X[0];
        if (lane == 63) edge_hi[buf][wave] = X[R - 1];
        __syncthreads();
    };
    // X <- 2 H~ Y - X (REC) or X <- H~ Y (head), from Y's edges in edge_*[buf]
    auto apply = [&](double2 (&X)[R], const double2 (&Y)[R], bool head) {
        // every lane reads the neighbouring wavefronts' edges (one broadcast
        // address each); lanes 0 and 63 use them
        const double2 el = edge_hi[buf][wave > 0 ? wave - 1 : 0];
        const double2 er = edge_lo[buf][wave < NW - 1 ? wave + 1 : NW - 1];
        const double2 l0 = from_left0(Y[R - 1]);  // lane l-1's last site
        const double2 rR = from_right0(Y[0]);     // lane l+1's first site
        auto row = [&](int r, double2 l, double2 rr) {
            const double sx = l.x + rr.x, sy = l.y + rr.y;
            if (head)
                X[r] = make_double2(0.5 * fma(c.d[r], Y[r].x, c.o[r] * sx), 0.5 * fma(c.d[r], Y[r].y, c.o[r] * sy));
            else
                X[r] = make_double2(fma(c.d[r], Y[r].x, fma(c.o[r], sx, -X[r].x)),
                                    fma(c.d[r], Y[r].y, fma(c.o[r], sy, -X[r].y)));
        };
#pragma unroll
        for (int r = 1; r + 1 < R; ++r) row(r, Y[r - 1], Y[r + 1]);
        const double2 left = csel(lane == 0, wave > 0 ? el : zero, l0);
        const double2 right = csel(lane == 63, wave < NW - 1 ? er : zero, rR);
        if (R == 1) {
            row(0, left, right);
        } else {
            row(0, left, Y[1]);
            row(R - 1, Y[R - 2], right);
        }
    };
    auto w_at = [&](int k) -> double {
        k = k < M ? k : M;
        return G_LDS ? wt[k] : signed_weight(wt, k);
    };

    publish(B);
    for (int64_t s = 0; s < K; ++s) {
        // head: A = v_1 = H~ psi, acc = r_0 psi - i r_1 v_1, norm and energy
        apply(A, B, true);
        buf ^= 1;
        double nrm = 0.0, e = 0.0;
        const double r0 = wt[0], r1 = M >= 1 ? wt[1] : 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (ckpt && row0 + r < op.n) ckpt[(size_t)s * op.n + row0 + r] = B[r];
            nrm += B[r].x * B[r].x + B[r].y * B[r].y;
            e += B[r].x * A[r].x + B[r].y * A[r].y;
            acc[r] = head_orders(r0, r1, B[r], A[r]);
        }
        block_sum2(nrm, e, red);
        if (tid == 0) {
            if (norm_out) norm_out[s] = nrm;
            if (energy_out) energy_out[s] = a * e + b * nrm;
        }
        publish(A);
        // orders 2 .. M: B holds v_{k-1}, A holds v_k, alternately; the
        // weights are read one pair ahead
        int k = 1;
        double we = w_at(2), wo = w_at(3);
        for (; k + 2 <= M; k += 2) {
            const double xe = we, xo = wo;
            we = w_at(k + 3);
            wo = w_at(k + 4);
            apply(B, A, false);  // v_{k+1} over v_{k-1}
            buf ^= 1;
            add_order<false>(xe, B, acc);
            publish(B);
            apply(A, B, false);  // v_{k+2} over v_k
            buf ^= 1;
            add_order<true>(xo, A, acc);
            publish(A);
        }
        if (k + 1 <= M) {  // one order left: v_M over v_{M-2}
            apply(B, A, false);
            buf ^= 1;
            add_order<false>(we, B, acc);
        }
        // psi_{s+1}
#pragma unroll
        for (int r = 0; r < R; ++r) {
            B[r] = with_phase(phase, acc[r]);
            A[r] = zero;
        }
        publish(B);
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (row0 + r < op.n) psi_out[row0 + r] = B[r];
}

// The same run spread over P workgroups for chains longer than one
// workgroup's share.  Workgroup w owns the S sites [w S, w S + S) and keeps
// H more on each side (local site j is chain site w S - H + j), all in
// registers as above.  A site's value after an order depends on its
// neighbours' values before it, so the sites a workgroup holds correctly
// shrink by one per order from each end: after at most H orders exactly its
// own S sites are right.  Then it sends its first and last H own sites of
// both vectors to its two neighbours and receives theirs into its halo.
// Every site's arithmetic is that of the one-workgroup kernel.
//
// A message word is 8 bytes: 32 bits of a value and the 32-bit number of the
// exchange (from 1; the buffer is cleared before the run).  A receiver reads
// its words until each carries the number, so nothing orders one word against
// another and no fence writes back or invalidates a cache.  Each word is
// stored and loaded by one relaxed agent-scope atomic, neighbouring lanes'
// words adjacent.  Measured on MI355X an exchange costs 1.8 us (3 us with
// plain strips behind release / acquire flags; 2.8 us with each site's words
// together, a line per lane).
//
// xbuf holds two exchanges (even, odd): a workgroup sends exchange e + 2 only
// after it received e + 1 from both neighbours, which they send after reading
// its e.  psi may be read and written in place: each workgroup reads its
// sites and halo at the start and counts itself in; none writes psi_out
// before all have.  Every wait is bounded in wall-clock time: past the limit
// the workgroup records a timeout, stops, and writes NaN to its sites.
// A launch runs at most kChainRing steps; each step's norm and energy
// partials go to `part`, summed in workgroup order after the launch.
struct ChainXDev {
    uint64_t *xbuf;    // [2 exchanges][P][2 strips][R][8 words][ceil(H / R) lanes]
    int32_t *sync;     // setup arrivals, then the timeout flag
    double *part;      // [kChainRing][P][2] norm and energy partials, or null
    double *knorm;     // [P] norm partials of the last state, or null
    int32_t H, S, P;
    int64_t spin_limit;  // wall-clock ticks a wait may take
};

__global__ void k_chain_multi_clear(uint64_t *xbuf, int64_t words, int32_t *sync, int first)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) xbuf[i] = 0;
    if (i == 0) {
        sync[0] = 0;
        if (first) sync[1] = 0;
    }
}

template <int R, int T, bool G_LDS>
__global__ __launch_bounds__(T) void k_chain_multi(OpChain op, const double2 *psi_in, double2 *psi_out,
                                                   const double *__restrict__ rw, double2 phase, int M, int64_t K,
                                                   double2 *ckpt, ChainXDev x)
{
    using namespace pairdev;
    constexpr int NW = T / 64;
    __shared__ double2 edge_lo[2][NW], edge_hi[2][NW];
    __shared__ double red[2 * NW];
    __shared__ int32_t s_bad;
    extern __shared__ double g_lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int32_t w = blockIdx.x, P = x.P, H = x.H, S = x.S;
    const int64_t base = (int64_t)w * S - H;  // chain site of local site 0
    const int32_t j0 = tid * R;
    const double2 zero = make_double2(0.0, 0.0);
    int32_t *const arrive = x.sync, *const timeout = x.sync + 1;
    double d[R], o[R];
    double2 A[R], B[R], acc[R];
    bool own[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t g = base + j0 + r;
        const bool in = g >= 0 && g < op.n;
        d[r] = in ? op.s2 * (op.V[g] + op.dsh) : 0.0;
        o[r] = in ? op.off2 : 0.0;
        B[r] = in ? psi_in[g] : zero;
        A[r] = zero;
        acc[r] = zero;
        own[r] = in && j0 + r >= H && j0 + r < H + S;
    }
    const double *wt = rw;
    if (G_LDS) {
        for (int k = tid; k <= M; k += T) g_lds[k] = signed_weight(rw, k);
        wt = g_lds;
    }
    if (tid == 0) s_bad = 0;
    // psi_in has been read by every thread before the workgroup counts itself in
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(arrive, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);

    int buf = 0;
    // a one-wavefront workgroup needs no edge exchange (and no barrier) per order
    auto publish = [&](const double2 (&X)[R]) {
        if constexpr (NW > 1) {
            if (lane == 0) edge_lo[buf][wave] = X[0];
            if (lane == 63) edge_hi[buf][wave] = X[R - 1];
            __syncthreads();
        }
    };
    auto apply = [&](double2 (&X)[R], const double2 (&Y)[R], bool head) {
        double2 el = zero, er = zero;
        if constexpr (NW > 1) {
            el = edge_hi[buf][wave > 0 ? wave - 1 : 0];
            er = edge_lo[buf][wave < NW - 1 ? wave + 1 : NW - 1];
        }
        const double2 l0 = from_left0(Y[R - 1]);
        const double2 rR = from_right0(Y[0]);
        auto row = [&](int r, double2 l, double2 rr) {
            const double sx = l.x + rr.x, sy = l.y + rr.y;
            if (head)
                X[r] = make_double2(0.5 * fma(d[r], Y[r].x, o[r] * sx), 0.5 * fma(d[r], Y[r].y, o[r] * sy));
            else
                X[r] = make_double2(fma(d[r], Y[r].x, fma(o[r], sx, -X[r].x)),
                                    fma(d[r], Y[r].y, fma(o[r], sy, -X[r].y)));
        };
#pragma unroll
        for (int r = 1; r + 1 < R; ++r) row(r, Y[r - 1], Y[r + 1]);
        // one wavefront: lanes 0 and 63 already read 0 from the shifts
        const double2 left = NW > 1 ? csel(lane == 0, wave > 0 ? el : zero, l0) : l0;
        const double2 right = NW > 1 ? csel(lane == 63, wave < NW - 1 ? er : zero, rR) : rR;
        if (R == 1) {
            row(0, left, right);
        } else {
            row(0, left, Y[1]);
            row(R - 1, Y[R - 2], right);
        }
    };
    // the wait has run out at wall-clock t0 + limit, or another workgroup's
    // has; a limit of 0 gives up at once (set from the host to test the path)
    auto expired = [&](int64_t t0, int64_t spins) -> bool {
        if (x.spin_limit > 0 && wall_clock64() - t0 <= x.spin_limit &&
            ((spins & 255) != 255 || __hip_atomic_load(timeout, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0))
            return false;
        __hip_atomic_store(timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    };
    // first word of site j of strip `side` of workgroup wg in exchange e; the
    // others follow HR apart, so that neighbouring lanes' words are adjacent
    const int32_t HR = (H + R - 1) / R;
    auto words = [&](int32_t e, int32_t wg, int side, int32_t j) -> uint64_t * {
        return x.xbuf + (((size_t)(e & 1) * P + wg) * 2 + side) * (size_t)(8 * R * HR) + (size_t)(j % R) * 8 * HR +
               j / R;
    };
    auto send = [&](uint64_t *q, int32_t e, double2 b, double2 a) {
        const double v[4] = {b.x, b.y, a.x, a.y};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint64_t u = (uint64_t)__double_as_longlong(v[i]), tag = (uint64_t)(uint32_t)e << 32;
            __hip_atomic_store(q + 2 * i * HR, tag | (u & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(q + (2 * i + 1) * HR, tag | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // send this workgroup's strips of (B, A), receive the neighbours' into
    // the halo; false (uniformly) after a timeout
    int32_t ep = 0;
    auto exchange = [&]() __attribute__((always_inline)) -> bool {
        const int32_t e = ++ep;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t j = j0 + r;
            if (j >= H && j < 2 * H && w > 0) send(words(e, w, 0, j - H), e, B[r], A[r]);
            if (j >= S && j < S + H && w + 1 < P) send(words(e, w, 1, j - S), e, B[r], A[r]);
        }
        const uint64_t *src[R];
        bool mine[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t j = j0 + r;
            const bool lo = j < H && w > 0, hi = j >= H + S && w + 1 < P;
            mine[r] = lo || hi;
            src[r] = lo ? words(e, w - 1, 1, j) : words(e, hi ? w + 1 : w, 0, hi ? j - H - S : 0);
        }
        uint64_t u[R][8];
        bool late = true;
        const int64_t t0 = wall_clock64();
        bool bad = x.spin_limit <= 0 && P > 1;
        for (int64_t spins = 0; !bad; ++spins) {
            bool all = true;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (mine[r] && late) {
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        u[r][i] = __hip_atomic_load(src[r] + i * HR, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (mine[r] && late) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) all = all && (int32_t)(u[r][i] >> 32) == e;
                }
            late = late && !all;
            if (__ballot(late) == 0) break;
            bad = __ballot(expired(t0, spins)) != 0;
        }
        if (bad) __hip_atomic_store(timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (NW > 1) {
            __syncthreads();  // s_bad of the previous exchange has been read
            if (bad) s_bad = 1;
            __syncthreads();
            bad = __builtin_amdgcn_readfirstlane(s_bad) != 0;
        }
        if (bad) return false;
        auto val = [](uint64_t lo, uint64_t hi) {
            return __longlong_as_double((long long)((hi << 32) | (lo & 0xffffffffull)));
        };
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (mine[r]) {
                B[r] = make_double2(val(u[r][0], u[r][1]), val(u[r][2], u[r][3]));
                A[r] = make_double2(val(u[r][4], u[r][5]), val(u[r][6], u[r][7]));
            }
        return true;
    };
    auto w_at = [&](int k) -> double {
        k = k < M ? k : M;
        return G_LDS ? wt[k] : signed_weight(wt, k);
    };

    bool ok = true;
    publish(B);
    for (int64_t s = 0; s < K && ok; ++s) {
        if (ckpt) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (own[r]) ckpt[(size_t)s * op.n + base + j0 + r] = B[r];
        }
        // head: A = v_1 = H~ psi, acc = r_0 psi - i r_1 v_1, own sites' norm and energy
        apply(A, B, true);
        buf ^= 1;
        double nrm = 0.0, en = 0.0;
        const double r0 = wt[0], r1 = M >= 1 ? wt[1] : 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            nrm += own[r] ? B[r].x * B[r].x + B[r].y * B[r].y : 0.0;
            en += own[r] ? B[r].x * A[r].x + B[r].y * A[r].y : 0.0;
            acc[r] = head_orders(r0, r1, B[r], A[r]);
        }
        if (x.part) {
            block_sum2(nrm, en, red);
            if (tid == 0) {
                x.part[((size_t)s * P + w) * 2] = nrm;
                x.part[((size_t)s * P + w) * 2 + 1] = en;
            }
        }
        publish(A);
        // orders 2 .. M, at most H orders between exchanges (the head counts
        // as one); B holds v_{k-1}, A holds v_k at every exchange.  The weights
        // are read one pair ahead
        int k = 1, left = H - 1;
        double we = w_at(2), wo = w_at(3);
        for (;;) {
            const int n = min(left, M - k) >> 1;
            for (int p = 0; p < n; ++p) {
                const double xe = we, xo = wo;
                we = w_at(k + 3);
                wo = w_at(k + 4);
                apply(B, A, false);
                buf ^= 1;
                add_order<false>(xe, B, acc);
                publish(B);
                apply(A, B, false);
                buf ^= 1;
                add_order<true>(xo, A, acc);
                publish(A);
                k += 2;
            }
            left -= 2 * n;
            if (k >= M) break;
            if (k + 1 == M && left >= 1) {  // one order left: v_M over v_{M-2}
                apply(B, A, false);
                buf ^= 1;
                add_order<false>(we, B, acc);
                break;
            }
            if (!(ok = exchange())) break;
            publish(A);
            left = H;
        }
        if (!ok) break;
        // psi_{s+1}, right on the own sites; the halo comes from the neighbours
#pragma unroll
        for (int r = 0; r < R; ++r) {
            B[r] = with_phase(phase, acc[r]);
            A[r] = zero;
        }
        if (s + 1 < K && !(ok = exchange())) break;
        publish(B);
    }
    // every workgroup has read psi_in before any writes psi_out
    if (ok) {
        if (tid == 0) {
            const int64_t t0 = wall_clock64();
            bool bad = x.spin_limit <= 0;
            for (int64_t spins = 0;
                 !bad && __hip_atomic_load(arrive, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < P; ++spins)
                bad = expired(t0, spins);
            if (bad) __hip_atomic_store(timeout, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_bad = bad ? 1 : 0;
        }
        __syncthreads();
        ok = __builtin_amdgcn_readfirstlane(s_bad) == 0;
    }
    const double nan = __builtin_nan("");
    double kn = 0.0, z = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (own[r]) {
            const double2 p = ok ? B[r] : make_double2(nan, nan);
            psi_out[base + j0 + r] = p;
            kn += p.x * p.x + p.y * p.y;
        }
    if (x.knorm) {
        __syncthreads();
        block_sum2(kn, z, red);
        if (tid == 0) x.knorm[w] = kn;
    }
}

bool chain_small_fits(int64_t n) { return n >= 1 && n <= 4096; }

// Workgroups of one wavefront: an order then needs no barrier, only lane
// shifts, and the run pays an exchange every H orders instead.  Two sites per
// lane and the deepest halo that leaves S >= H, since an order costs 0.06 us
// with two sites and 0.10 us with four.  Measured on MI355X (double well,
// dt = 0.5), us per order with two sites and H = 42 / two and 32 / four and
// 84: 0.105 / 0.117 / 0.122 at n = 400, 0.106 / 0.118 / 0.122 at 1024, 0.105 /
// 0.118 / 0.122 at 4096 (0.19 there with the flags of before); the
// one-workgroup kernel takes 0.25, 0.25 and 0.40.  CHEBTD_CHAIN_MULTI =
// "R,T,H" overrides, "0" keeps one workgroup.
ChainMultiCfg chain_multi_config(int64_t n)
{
    ChainMultiCfg cfg;
    int R = 2, T = 64, H = 42;
    if (const char *env = std::getenv("CHEBTD_CHAIN_MULTI"))
        if (std::sscanf(env, "%d,%d,%d", &R, &T, &H) != 3) R = 0;
    const bool shape = (R == 1 && T == 512) || (R == 2 && T == 256) || (R == 2 && T == 512) || (R == 4 && T == 256) ||
                       (R == 2 && T == 64) || (R == 4 && T == 64) || (R == 8 && T == 64) || (R == 4 && T == 128);
    // from 129 sites (below that one workgroup holds the chain with one site per lane)
    if (!shape || H < 2 || (H & 1) || R * T < 3 * H || n <= 128 || !chain_small_fits(n)) return cfg;
    const int64_t S = (int64_t)R * T - 2 * H, P = (n + S - 1) / S;
    if (P < 2 || P > kChainMaxWG) return cfg;
    cfg.R = R;
    cfg.T = T;
    cfg.H = H;
    cfg.S = S;
    cfg.P = P;
    return cfg;
}

// Whether the workgroups of such a run may keep its weights (wbytes) in LDS.
// They wait on each other, so all P must be resident, also beside the runs of
// other streams: as many runs as the device's four hardware queues can start
// at once have to fit.  With 4096 sites (P = 94) two workgroups fill a CU's LDS
// from M = 6,700 on and one from 10,100 on, where three runs no longer fit the
// 256 CUs together and each may hold a part of them until its waits run out.
// Weights read from memory leave room for all of them; measured on MI355X an
// order then takes 0.123 us instead of 0.106 (n = 4096, M = 10,500 to 21,000).
constexpr int kChainRuns = 4;
bool chain_weights_in_lds(int64_t P, size_t wbytes, int64_t num_cus, size_t lds_per_cu)
{
    const size_t per_cu = lds_per_cu / (wbytes + 1024);  // beside a few hundred bytes of its own
    return num_cus * (int64_t)per_cu >= kChainRuns * P;
}

namespace {
constexpr size_t kChainIntBytes = 64;  // sync

size_t chain_part_bytes(const ChainMultiCfg &cfg) { return (size_t)(2 * kChainRing + 1) * cfg.P * sizeof(double); }
int64_t chain_x_words(const ChainMultiCfg &cfg) { return (int64_t)2 * cfg.P * 2 * 8 * cfg.R * ((cfg.H + cfg.R - 1) / cfg.R); }

ChainXDev chain_x_layout(const Ctx &c, const ChainMultiCfg &cfg, int64_t spin_limit)
{
    char *p = static_cast<char *>(c.chainx.p);
    ChainXDev x{};
    x.sync = reinterpret_cast<int32_t *>(p);
    x.part = reinterpret_cast<double *>(p + kChainIntBytes);
    x.knorm = x.part + (size_t)2 * kChainRing * cfg.P;
    x.xbuf = reinterpret_cast<uint64_t *>(p + kChainIntBytes + chain_part_bytes(cfg));
    x.H = cfg.H;
    x.S = (int32_t)cfg.S;
    x.P = (int32_t)cfg.P;
    x.spin_limit = spin_limit;
    return x;
}
}  // namespace

size_t chain_multi_scratch_bytes(const ChainMultiCfg &cfg)
{
    if (cfg.R == 0) return 0;
    return kChainIntBytes + chain_part_bytes(cfg) + (size_t)chain_x_words(cfg) * sizeof(uint64_t);
}

// the several-workgroup run's timeout flag when it runs for this context
int32_t *chain_multi_timeout(const Ctx &c)
{
    const ChainMultiCfg cfg = chain_multi_config(c.n);
    if (cfg.R == 0 || !c.chainx.p || c.chainx.bytes < chain_multi_scratch_bytes(cfg)) return nullptr;
    return chain_x_layout(c, cfg, 0).sync + 1;
}

namespace {

// dynamic LDS past 64 KiB has to be asked for
template <class K>
hipError_t allow_lds(K kernel, size_t dyn)
{
    if (dyn <= 65536) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)dyn);
}

template <int R, int T>
hipError_t launch_chain_rt(const Ctx &c, hipStream_t s, const OpChain &op, double2 *psi, double2 *out, int64_t K,
                           double *norm_out, double *energy_out, double2 *ckpt, size_t dyn)
{
    auto *kernel = dyn ? &k_chain_small<R, T, true> : &k_chain_small<R, T, false>;
    hipError_t e = allow_lds(kernel, dyn);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(T), dyn, s, op, psi, out, c.rweight_dev, c.phase, c.M, K, c.a, c.b,
                       norm_out, energy_out, ckpt);
    return hipGetLastError();
}

template <int R, int T>
hipError_t launch_chain_multi_rt(const Ctx &c, hipStream_t s, const OpChain &op, const ChainXDev &x, double2 *psi,
                                 double2 *out, int64_t K, double2 *ckpt, size_t dyn)
{
    auto *kernel = dyn ? &k_chain_multi<R, T, true> : &k_chain_multi<R, T, false>;
    hipError_t e = allow_lds(kernel, dyn);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3((unsigned)x.P), dim3(T), dyn, s, op, psi, out, c.rweight_dev, c.phase, c.M, K,
                       ckpt, x);
    return hipGetLastError();
}

hipError_t launch_chain_multi(const Ctx &c, hipStream_t s, const OpChain &op, const ChainMultiCfg &cfg,
                              const ChainXDev &x, double2 *psi, double2 *out, int64_t K, double2 *ckpt, size_t dyn)
{
    if (cfg.T == 64 && cfg.R == 2) return launch_chain_multi_rt<2, 64>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.T == 64 && cfg.R == 4) return launch_chain_multi_rt<4, 64>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.T == 64) return launch_chain_multi_rt<8, 64>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.T == 128) return launch_chain_multi_rt<4, 128>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.R == 1) return launch_chain_multi_rt<1, 512>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.R == 2 && cfg.T == 256) return launch_chain_multi_rt<2, 256>(c, s, op, x, psi, out, K, ckpt, dyn);
    if (cfg.R == 2) return launch_chain_multi_rt<2, 512>(c, s, op, x, psi, out, K, ckpt, dyn);
    return launch_chain_multi_rt<4, 256>(c, s, op, x, psi, out, K, ckpt, dyn);
}

}  // namespace

hipError_t launch_chain_small(const Ctx &c, hipStream_t s, double2 *psi, double2 *out, int64_t K, double *norm_out,
                              double *energy_out, double2 *ckpt, double *check, bool *checked)
{
    const OpChain op = make_chain(c);
    // weights in LDS when they fit beside the kernel's own few hundred bytes
    int max_lds = 0;
    if (hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, c.device) != hipSuccess)
        max_lds = 65536;
    const size_t gbytes = (size_t)(c.M + 1) * sizeof(double);
    const size_t dyn = gbytes + 1024 <= (size_t)max_lds ? gbytes : 0;
    const ChainMultiCfg cfg = chain_multi_config(c.n);
    *checked = false;
    if (cfg.R > 0 && c.chainx.p && c.chainx.bytes >= chain_multi_scratch_bytes(cfg)) {
        int khz = 0;
        if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, c.device) != hipSuccess || khz <= 0)
            khz = 100000;
        // two seconds per wait; CHEBTD_CHAIN_SPIN (wall-clock ticks) shortens it
        // (0: every wait gives up at once)
        int64_t limit = (int64_t)khz * 1000 * 2;
        if (const char *env = std::getenv("CHEBTD_CHAIN_SPIN")) limit = std::max<int64_t>(0, std::atoll(env));
        ChainXDev x = chain_x_layout(c, cfg, limit);
        double *const part = x.part, *const knorm = x.knorm;
        int cu_lds = 0;
        if (hipDeviceGetAttribute(&cu_lds, hipDeviceAttributeMaxSharedMemoryPerMultiprocessor, c.device) != hipSuccess)
            cu_lds = max_lds;
        const size_t wdyn = dyn && chain_weights_in_lds(cfg.P, dyn, c.num_cus, (size_t)cu_lds) ? dyn : 0;
        const int64_t words = chain_x_words(cfg);
        for (int64_t st = 0; st < K; st += kChainRing) {
            const int64_t k = std::min<int64_t>(kChainRing, K - st);
            const bool last = st + k == K;
            const bool sums = norm_out || energy_out || (check && (st == 0 || last));
            x.part = sums ? part : nullptr;
            x.knorm = check && last ? knorm : nullptr;
            hipLaunchKernelGGL(k_chain_multi_clear, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, x.xbuf,
                               words, x.sync, st == 0 ? 1 : 0);
            hipError_t e = launch_chain_multi(c, s, op, cfg, x, st == 0 ? psi : out, out, k,
                                              ckpt ? ckpt + (size_t)st * c.n : nullptr, wdyn);
            if (e == hipSuccess && sums)
                e = launch_ne_steps(s, {part, 2 * cfg.P, (int)cfg.P, (int)k, c.a, c.b, norm_out, energy_out, st,
                                        nullptr, x.knorm, (int)cfg.P, check, st == 0});
            if (e != hipSuccess) return e;
        }
        *checked = check != nullptr;
        return hipSuccess;
    }
    // two wavefronts per SIMD for the longer chains (one issues while the
    // other waits on the edge exchange; measured 15% faster at n = 4096),
    // one for the shorter ones
    const int64_t n = c.n;
    if (n <= 256) return launch_chain_rt<1, 256>(c, s, op, psi, out, K, norm_out, energy_out, ckpt, dyn);
    if (n <= 512) return launch_chain_rt<2, 256>(c, s, op, psi, out, K, norm_out, energy_out, ckpt, dyn);
    if (n <= 1024) return launch_chain_rt<4, 256>(c, s, op, psi, out, K, norm_out, energy_out, ckpt, dyn);
    if (n <= 2048) return launch_chain_rt<4, 512>(c, s, op, psi, out, K, norm_out, energy_out, ckpt, dyn);
    if (n <= 4096) return launch_chain_rt<8, 512>(c, s, op, psi, out, K, norm_out, energy_out, ckpt, dyn);
    return hipErrorInvalidValue;
}

}  // namespace chebtd
