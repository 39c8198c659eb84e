// Host-side check of the rules that choose a kernel or its launch shape.  Needs
// no GPU; linked with the library's objects.  Exit status 0: every check passed.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <string>

#include "batch_internal.h"
#include "chebtd.h"
#include "internal.h"
#include "pipe.h"

using namespace chebtd;

namespace chebtd {
int ensure(Ctx *c, DevBuf &b, size_t bytes, const char *what);  // api.cpp
}
struct chebtd_ctx : public Ctx {};

static int failures = 0;
#define CHECK(cond)                                                                \
    do {                                                                           \
        if (!(cond)) {                                                             \
            std::fprintf(stderr, "check failed: %s (line %d)\n", #cond, __LINE__); \
            ++failures;                                                            \
        }                                                                          \
    } while (0)

// Workgroups of the several-workgroup chain run wait on each other.  Counted
// here: four runs at once, one per hardware queue, find room for every
// workgroup on 256 CUs of 160 KiB LDS, whatever n and M.
static void chain_residency()
{
    const size_t lds = 160 * 1024;
    bool in_lds = false, in_memory = false;
    for (int64_t n = 129; n <= 4096; n += n < 600 ? 1 : 37) {
        const ChainMultiCfg cfg = chain_multi_config(n);
        for (int M = 1; M <= 40000; M += 61) {
            const size_t wbytes = (size_t)(M + 1) * sizeof(double);
            if (wbytes + 1024 > lds) continue;  // never in LDS
            const bool kept = chain_weights_in_lds(cfg.P, wbytes, 256, lds);
            const size_t per_wg = (kept ? wbytes : 0) + 1024;
            CHECK((int64_t)(lds / per_wg) * 256 >= 4 * cfg.P);
            (kept ? in_lds : in_memory) = true;
            if (failures > 20) return;
        }
    }
    CHECK(in_lds && in_memory);
    // the double well of 4096 points at dt = 0.5 (order 7256) keeps them in LDS
    CHECK(chain_weights_in_lds(chain_multi_config(4096).P, 7257 * sizeof(double), 256, lds));
}

// A matrix found complex is not copied again, but looked at now and then.
static void csr_copies()
{
    double pinned[16] = {};
    char room = 0;
    Ctx c;
    c.pinned = pinned;
    c.kind = HKind::Csr;
    c.n = 300000;
    c.nnz = 1200000;
    c.csr_buf.p = &room;  // never dereferenced here
    c.csr_buf.bytes = csr_copy_bytes(c.n, c.nnz);
    c.csr_orders = csr_copy_orders(c.n, c.nnz, 64 * 4 * ((c.n + 63) / 64), 4);
    CHECK(csr_copy_pays(c, 8) && csr_copy_pays(c, 8) && !csr_copy_pays(c, 7));
    *csr_seen(c) = 1;
    for (int call = 0; call < 40; ++call) CHECK(csr_copy_pays(c, 8));
    *csr_seen(c) = 2;
    int looked = 0;
    for (int call = 0; call < 160; ++call)
        if (csr_copy_pays(c, 8)) {
            ++looked;
            CHECK(c.csr_look);
        }
    CHECK(looked >= 5 && looked <= 16);
    c.csr_buf.p = nullptr;
    // even rows; lengths of 0 to 8; one long row in every 64, in all; long rows
    const int64_t n = 1 << 20, never = INT64_MAX;
    CHECK(csr_copy_orders(n, 4 * n, 4 * n, 4) == 8 && csr_copy_orders(n, 4 * n, 8 * n, 8) == 8);
    CHECK(csr_copy_orders(n, 5 * n, 64 * n, 64) == never);
    CHECK(csr_copy_orders(n, 3 * n, 3 * n + 64 * n, n) == never && csr_copy_orders(n, 5 * n, 6 * n, n) == never);
    CHECK(csr_copy_orders(2048, 2048 * 2048, 2048 * 2048, 2048) == 64);
    CHECK(csr_copy_orders(n, n, n, 1) == 64);
}

// An allocation that fails (there is no device here) gives the room of the
// matrix copy back, unless a call is reading the copy.
static void room_given_back()
{
    char room = 0;
    Ctx c;
    DevBuf b;
    c.csr_buf.p = &room;  // not an allocation: freeing it is refused
    c.csr_buf.bytes = 1;
    c.csr_copy = true;
    CHECK(ensure(&c, b, size_t(1) << 50, "test") == CHEBTD_E_OOM && c.csr_buf.p != nullptr);
    c.csr_copy = false;
    CHECK(ensure(&c, b, size_t(1) << 50, "test") == CHEBTD_E_OOM && c.csr_buf.p == nullptr && b.p == nullptr);
}

// Steps of few orders on ribbons: one walk, not a pipelined pass of eight
// orders; the benchmark's and the paper's steps stay where they are.
static void few_orders()
{
    for (int M = 2; M <= 5; ++M) CHECK(walk_takes_step(128, 8192, M, false) && walk_takes_step(64, 1000, M, false));
    CHECK(walk_takes_step(1024, 32768, 3, false) && walk_takes_step(1024, 32768, 6, false));
    CHECK(walk_takes_step(1500, 3495, 4, false) && walk_takes_step(777, 6748, 6, false));
    CHECK(walk_takes_step(1, 2000000, 2, true) && !walk_takes_step(1, 300000, 2, true));
    CHECK(!walk_takes_step(1024, 32768, 2, false) && !walk_takes_step(128, 8192, 6, false));
    CHECK(walk_takes_step(40, 500, 3, true) && !walk_takes_step(10, 1000, 3, true));
    for (int64_t W : {4, 16, 32, 48, 49, 128, 301, 1024, 30000})
        for (int64_t L : {64, 512, 5003, 32768})
            for (int M = 7; M <= 100; ++M) CHECK(!walk_takes_step(W, L, M, W <= 48));
}

// and chains that keep the step-end pairs: few orders of long chains
static void few_orders_kept()
{
    CHECK(walk_takes_kept_chain_step(1500000, 2) && walk_takes_kept_chain_step(1500000, 3));
    CHECK(!walk_takes_kept_chain_step(65536, 2) && !walk_takes_kept_chain_step(4000000, 4));
    for (int64_t n : {4097, 65536, 1048576, 4000000, 6000000})
        for (int M = 5; M <= 200; ++M) CHECK(!walk_takes_kept_chain_step(n, M));
}

// and in batches: the systems of the walk's depth, tall ribbons of few columns
static void few_orders_batched()
{
    CHECK(batch_walk_takes(100, 2000, 5, 5) && !batch_walk_takes(100, 2000, 6, 5));
    CHECK(batch_walk_takes(30000, 16, 10, 5) && batch_walk_takes(3000, 16, 10, 5));
    CHECK(!batch_walk_takes(2000, 16, 10, 5) && !batch_walk_takes(3000, 41, 10, 5));
    for (int M = 6; M <= 100; ++M) {
        int np = 0, ne = 0;
        batch_deep_split(M, 5, &np, &ne);
        CHECK(!batch_walk_takes(128, 8192, M, 5) && (!batch_walk_takes(30000, 16, M, 5) || 5 * np + ne == M));
    }
}

// Sites per thread of the Holstein walk, by configurations: enough of them and
// a thread walks all sites.
static void holstein_sites()
{
    auto spt = [](int L, int64_t nconf) {
        Ctx c;
        c.kind = HKind::Holstein;
        c.hol_L = L;
        c.n = nconf * L;
        return hol_sites_per_thread(c);
    };
    CHECK(spt(3, 302621) == 3 && spt(4, 211876) == 4 && spt(6, 177100) == 6 && spt(3, 91881) == 3);
    CHECK(spt(3, 39711) == 1 && spt(4, 135751) == 2 && spt(10, 92378) == 2 && spt(10, 43758) == 1);
    CHECK(spt(10, 184756) == 10 && spt(12, 1352078) == 12 && spt(1, 255) == 1 && spt(2, 32640) == 1);
}

// The row chunks of a pipelined pass: no count takes less time by the model, and
// a plan of the tallest ribbon does not try every one.
static void pipe_chunk_counts()
{
    const int shapes[][2] = {{2, 4}, {3, 4}, {4, 4}, {5, 4}, {3, 8}};
    for (int64_t W : {1, 7, 30, 50, 64, 97, 128, 301, 777, 1024, 4099, 30000})
        for (int64_t L : {2, 80, 200, 777, 1500, 5003, 8192, 32768})
            for (const auto &sh : shapes) {
                const int n = pipe_chunks(W, L, sh[0], sh[1], 256);
                const double t = pipe_time(W, L, {{sh[0], sh[1], n}}, 256);
                const int64_t most = (W - (sh[0] * sh[1] - 1)) / 8;
                CHECK(n >= 1 && (n == 1 || n <= most));
                const int64_t cols = pipe_strip_cols(sh[0] * sh[1]), strips = (L + cols - 1) / cols;
                const int64_t places = sh[1] <= 4 ? 512 : 256;  // on 256 CUs; up to four rounds of them are tried
                for (int64_t m = 1; m <= std::min(most, 4 * places / strips); ++m)
                    CHECK(t <= pipe_time(W, L, {{sh[0], sh[1], (int)m}}, 256) * (1.0 + 1e-12));
                if (failures > 20) return;
            }
    const auto t0 = std::chrono::steady_clock::now();
    for (int i = 0; i < 1000; ++i) pipe_chunks(30000, 2, 5, 4, 256);
    const double us = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count() * 1e3;
    std::printf("pipe_chunks at 30000 x 2: %.2f us\n", us);
    CHECK(us < 25.0);  // 87 us when every count is tried, 1.3 now
}

// The passes of a batch whose strips fill the chip: they hold every order, cost no
// more than those by the number of sites, and those of ribbons of one row, mostly
// filling and emptying where a pass holds many orders, hold twelve at most.
static void shapes_by_cost()
{
    const int shapes[][2] = {{2, 4}, {3, 4}, {4, 4}, {5, 4}, {3, 8}};
    for (int64_t W : {1, 2, 5, 16, 40, 100, 3000})
        for (int64_t L : {100000, 400000}) {
            double cost[kPipeShapes] = {};
            pipe_shape_costs(W, L, 256, cost);
            const auto sum = [&](const std::vector<PipeShape> &v, int &orders) {
                double t = 0.0;
                orders = 0;
                for (const PipeShape &p : v) {
                    orders += p.DW * p.NW;
                    for (int q = 0; q < kPipeShapes; ++q)
                        if (shapes[q][0] == p.DW && shapes[q][1] == p.NW) t += cost[q];
                }
                return t;
            };
            for (int M = 2; M < 140; ++M) {
                int here = 0, there = 0;
                const auto plan = plan_pipe_shapes(W * L, M, false, cost);
                const double t = sum(plan, here), by_sites = sum(plan_pipe_shapes(W * L, M, false), there);
                CHECK(here >= M && there >= M && t <= by_sites * (1.0 + 1e-12));
                for (const PipeShape &p : plan) CHECK(W > 1 || p.DW * p.NW <= 12);
                if (failures > 20) return;
            }
        }
}

// A plan whose allocations fail (there is no device here) leaves none behind:
// buffers of the one before may be gone.
static void failed_plan()
{
    chebtd_ctx c;
    c.kind = HKind::Honeycomb;
    c.W = 10;
    c.L = 100;
    c.n = 1000;
    c.num_cus = 256;
    c.a = 3.0;
    c.has_bounds = c.has_plan = true;
    CHECK(chebtd_plan_order(&c, 0.5, 12) != CHEBTD_OK && !c.has_plan);
    double d = 0.0;
    CHECK(chebtd_propagate(&c, &d, 1, nullptr, nullptr, 0) == CHEBTD_E_STATE);
}

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "chain") chain_residency();
    else if (what == "csr") csr_copies();
    else if (what == "room") room_given_back();
    else if (what == "walk") few_orders(), few_orders_kept(), few_orders_batched();
    else if (what == "holstein") holstein_sites();
    else if (what == "chunks") pipe_chunk_counts();
    else if (what == "shapes") shapes_by_cost();
    else if (what == "plan") failed_plan();
    else CHECK(!"known check");
    std::printf("dispatch_check %s: %d failures\n", what.c_str(), failures);
    return failures == 0 ? 0 : 1;
}
