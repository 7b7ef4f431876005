// Checks of the library's host code against the stand-in runtime, one per
// command-line name; exit status 0 when the check holds.
#include "fake_hip.h"

#include <functional>
#include <new>

#include "fcoo.h"
#include "fcoo_internal.h"

// host allocations of 256 bytes and more until one is refused (-1: none is)
static int refuse_in = -1;
void *operator new(size_t n)
{
    if (n >= 256 && refuse_in >= 0 && refuse_in-- == 0) throw std::bad_alloc();
    void *p = malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

#define CHECK(c)                                                                              \
    do {                                                                                      \
        if (!(c)) {                                                                           \
            fprintf(stderr, "%s:%d: %s (%s) %s\n", __FILE__, __LINE__, #c, fcoo_last_error(), \
                    fake::last_stale.c_str());                                                \
            exit(1);                                                                          \
        }                                                                                     \
    } while (0)

// Z nonzeros, one index of each mode after the other
static fcoo_tensor *tensor(std::vector<int64_t> dims, int64_t Z)
{
    std::vector<std::vector<int32_t>> idx(dims.size());
    std::vector<const int32_t *> p;
    for (size_t m = 0; m < dims.size(); ++m) {
        idx[m].resize(Z);
        for (int64_t e = 0; e < Z; ++e) idx[m][e] = (int32_t)((e * (m ? 7 : 1)) % dims[m]);
        p.push_back(idx[m].data());
    }
    std::vector<float> v(Z, 1.f);
    fcoo_tensor *t = nullptr;
    CHECK(fcoo_create((int)dims.size(), dims.data(), Z, p.data(), v.data(), &t) == FCOO_OK);
    return t;
}

static void *dev(size_t bytes)
{
    void *p = nullptr;
    CHECK(hipMalloc(&p, bytes) == hipSuccess);
    return p;
}

// CP-ALS from fresh factors on a new handle: no kernel is given scratch that the
// sweep has let go of, whichever mode's Gram takes the most of it.
static void cp_workspace(std::vector<int64_t> dims, int R, int dtype)
{
    fcoo_tensor *t = tensor(dims, 64);
    std::vector<void *> f;
    for (size_t m = 0; m < dims.size(); ++m) {
        CHECK(fcoo_build(t, (int)m, FCOO_OP_MTTKRP, nullptr, nullptr) == FCOO_OK);
        f.push_back(dev((size_t)dims[m] * R * 4));
    }
    double *lambda = (double *)dev(R * 8), *grams = (double *)dev(dims.size() * R * R * 8), fit;
    for (int sweep = 0; sweep < 2; ++sweep)
        CHECK(fcoo_cp_als_iter(t, f.data(), dtype, R, lambda, grams, sweep, &fit, nullptr, nullptr) == FCOO_OK);
    CHECK(fake::stale == 0);
    fcoo_destroy(t);
}

// A block goes back to the pool once nothing queued on its own device can still use
// it, whichever device is current when its build is released.
static void pool_device()
{
    using namespace fcoo;
    fcoo_tensor *t = tensor({4, 4}, 8);                  // (the pool keeps blocks while a handle lives)
    Built b;
    CHECK(pool_get((size_t)8 << 20, &b.arena) == FCOO_OK);
    CHECK(b.arena.dev == 0);
    fake::pending[0] = true;
    CHECK(hipSetDevice(1) == hipSuccess);
    b.free_device();
    CHECK(!fake::pending[0]);
    CHECK(fake::device == 1);
    fcoo_destroy(t);
}

// With no room left but what lies idle in the pool, whatever the library allocates
// gets it: nothing is refused for the sake of idle blocks.
static void pool_gives_way()
{
    using namespace fcoo;
    const size_t big = (size_t)64 << 20;
    fcoo_tensor *t = tensor({300, 200, 100}, 100000);
    PoolBlock b;
    auto fill = [&] {
        fake::limit = (size_t)1 << 40;
        CHECK(pool_get(big, &b) == FCOO_OK);
        pool_put(&b);
        fake::limit = fake::live_bytes + 64;
    };
    const int R = 256;
    void *f[3] = {dev(300 * R * 4), dev(200 * R * 4), dev(100 * R * 4)};
    float *out = (float *)dev(300 * R * 4), *g = (float *)dev(100000 * 4), best_ms;
    double *d = (double *)dev(3 * 64 * 64 * 8), fit;
    for (int m = 0; m < 3; ++m) {
        fill();
        CHECK(fcoo_build(t, m, FCOO_OP_MTTKRP, nullptr, nullptr) == FCOO_OK);
    }
    fill();
    CHECK(fcoo_spmttkrp(t, 0, f, FCOO_F32, R, out, nullptr) == FCOO_OK);             // carries
    fill();
    CHECK(fcoo_resid_spmttkrp(t, 0, f, FCOO_F32, 64, out, d, nullptr) == FCOO_OK);   // partial losses
    fill();
    CHECK(fcoo_gram(t, 0, f[0], FCOO_F32, R, d + 64, nullptr) == FCOO_OK);           // partial Grams
    fill();
    CHECK(fcoo_cp_als_iter(t, f, FCOO_F32, 64, d, d, 0, &fit, nullptr, nullptr) == FCOO_OK);
    fill();
    CHECK(fcoo_model_at_nnz(t, f, FCOO_F32, 8, g, nullptr) == FCOO_OK);              // coordinates
    fcoo_opts one{};
    one.single_pass = 1;
    fill();
    CHECK(fcoo_build(t, 1, FCOO_OP_MTTKRP, &one, nullptr) == FCOO_OK);
    fill();
    CHECK(fcoo_spmttkrp(t, 1, f, FCOO_F32, R, out, nullptr) == FCOO_OK);             // published partials
    const int tile = 4096;
    fcoo_opts best;
    fill();
    CHECK(fcoo_autotune(t, 2, FCOO_OP_MTTKRP, f, FCOO_F32, R, &tile, 1, 1, &best, &best_ms, nullptr) == FCOO_OK);
    fcoo_destroy(t);
}

// A build succeeds where the arrays it is made of fit, also with no room for the
// carries that the first operation will want.
static void build_without_carries(int single_pass)
{
    fcoo_opts o{};
    o.single_pass = single_pass;
    const size_t before = fake::live_bytes;
    fcoo_tensor *t = tensor({300, 200, 100}, 100000);
    CHECK(fcoo_build(t, 0, FCOO_OP_TTM, &o, nullptr) == FCOO_OK);
    const size_t all = fake::live_bytes - before;
    fcoo_destroy(t);
    t = tensor({300, 200, 100}, 100000);
    fake::limit = fake::live_bytes + all - 1;
    CHECK(fcoo_build(t, 0, FCOO_OP_TTM, &o, nullptr) == FCOO_OK);
    CHECK(std::string(fcoo_last_error()).empty());
    void *U = nullptr;
    fake::limit += (size_t)64 << 20;
    U = dev(300 * 16 * 4);
    CHECK(fcoo_spttm(t, 0, U, FCOO_F32, 16, (float *)dev((size_t)100000 * 16 * 4), nullptr) == FCOO_OK);
    fcoo_destroy(t);
    fake::limit = (size_t)1 << 40;
}

// Scratch goes by the widest rows that a build has worked on: once those have been
// through, no operation on rows as wide or narrower lets go of scratch (a captured
// graph may hold it) or asks for more (a stream may be being captured).
static void scratch_stays(int64_t Z, std::vector<int64_t> dims)
{
    fcoo_tensor *t = tensor(dims, Z);
    CHECK(fcoo_build(t, 0, FCOO_OP_MTTKRP, nullptr, nullptr) == FCOO_OK);
    const size_t W = 256;
    std::vector<void *> f;
    for (int64_t d : dims) f.push_back(dev((size_t)d * W * 4));
    float *out = (float *)dev((size_t)dims[0] * 2048 * 4), *g = (float *)dev((size_t)Z * 4);
    double *loss = (double *)dev(8);
    auto chain = [&](int a, int b) {
        std::vector<int> k(dims.size(), 1);
        k[1] = a;
        k[2] = b;
        CHECK(fcoo_spttmc(t, 0, f.data(), FCOO_F32, k.data(), out, nullptr) == FCOO_OK);
    };
    CHECK(fcoo_resid_spmttkrp(t, 0, f.data(), FCOO_F32, 64, out, loss, nullptr) == FCOO_OK);
    for (int widest : {64, 256, 2048}) {
        if (widest <= 256) CHECK(fcoo_spmttkrp(t, 0, f.data(), FCOO_F32, widest, out, nullptr) == FCOO_OK);
        else chain(64, 32);
        fake::capturing = true;
        const int frees = fake::frees, mallocs = fake::mallocs;
        for (int dtype : {FCOO_F32, FCOO_BF16})
            for (int R : {1, 3, 8, 16, 17, 31, 32, 33, 64, 128, 256}) {
                if (R > widest) break;
                CHECK(fcoo_spmttkrp(t, 0, f.data(), dtype, R, out, nullptr) == FCOO_OK);
                CHECK(fcoo_spmttkrp_values(t, 0, g, f.data(), dtype, R, out, nullptr) == FCOO_OK);
                if (R <= 64) CHECK(fcoo_resid_spmttkrp(t, 0, f.data(), dtype, R, out, loss, nullptr) == FCOO_OK);
            }
        for (int a = 1; a * 8 <= widest; a *= 2) chain(a, 8);
        CHECK(fake::frees == frees && fake::mallocs == mallocs);
        fake::capturing = false;
    }
    fcoo_destroy(t);
}

// ... and they hold the carries of each launch's tiles.
static void carries_hold(std::vector<int64_t> dims, int64_t Z, int tile)
{
    using namespace fcoo;
    fcoo_tensor *t = tensor(dims, Z);
    fcoo_opts o{};
    o.tile_nnz = tile;
    CHECK(fcoo_build(t, 0, FCOO_OP_MTTKRP, &o, nullptr) == FCOO_OK);
    const Built &b = t->b[FCOO_OP_MTTKRP][0];
    std::vector<void *> f;
    for (int64_t d : dims) f.push_back(dev((size_t)d * 4096 * 4));
    float *out = (float *)dev((size_t)dims[0] * 8192 * 4);
    const bool kron = dims.size() > 2;
    for (int w = 1; w <= (kron ? 4096 : 256); w += w < 70 ? 1 : w / 2) {
        std::vector<int> k(dims.size(), 1);
        k[1] = std::min(w, 256);
        if (kron) k[2] = w / k[1];
        const int W = k[1] * (kron ? k[2] : 1);
        if (w <= 256) CHECK(fcoo_spmttkrp(t, 0, f.data(), FCOO_BF16, w, out, nullptr) == FCOO_OK);
        CHECK(fcoo_spttmc(t, 0, f.data(), FCOO_F32, k.data(), out, nullptr) == FCOO_OK);
        for (int dtype : {FCOO_F32, FCOO_BF16})
            for (bool resid : {false, true})
                CHECK(w > 256 || 2 * pick_plan(b, dtype, w, resid, false).ntiles * w <= b.carry_cap);
        CHECK(2 * pick_plan(b, FCOO_F32, W, false, kron).ntiles * W <= b.carry_cap);
    }
    fcoo_destroy(t);
}

// Replaced values in stored order are as padded as the build's streams: a lane past
// the last nonzero reads 4 entries there.  They are copied where rows have several
// rank tiles, and where the values lie in the result's memory.
static void values_padded(int64_t Z, int R, bool inside)
{
    fcoo_tensor *t = tensor({3000, 200, 10}, Z);
    CHECK(fcoo_build(t, 0, FCOO_OP_MTTKRP, nullptr, nullptr) == FCOO_OK);
    std::vector<void *> f;
    for (int64_t d : {3000, 200, 10}) f.push_back(dev((size_t)d * R * 4));
    float *out = (float *)dev(((size_t)3000 * R + Z) * 4), *g = inside ? out : (float *)dev((size_t)Z * 4);
    const fcoo::Built &b = t->b[FCOO_OP_MTTKRP][0];
    for (int dtype : {FCOO_F32, FCOO_BF16}) {
        CHECK(fcoo_spmttkrp_values(t, 0, g, f.data(), dtype, R, out, nullptr) == FCOO_OK);
        CHECK(b.d_gperm && fake::find(b.d_gperm)->bytes >= (size_t)(Z + 4) * 4);
    }
    fcoo_destroy(t);
}

// With no room for the carries of the tiles that suit a call, it runs on the build's
// own tiles, whose carries fit.
static void carries_that_fit()
{
    fcoo_tensor *t = tensor({300, 200, 100}, 2000000);
    fcoo_opts o{};
    o.tile_nnz = 1 << 20;
    CHECK(fcoo_build(t, 0, FCOO_OP_MTTKRP, &o, nullptr) == FCOO_OK);
    void *f[3] = {nullptr, dev(200 * 32 * 4), dev(100 * 32 * 4)};
    const int k[3] = {1, 32, 32};
    float *out = (float *)dev(300 * 1024 * 4);
    fake::limit = fake::live_bytes + (size_t)4 * 1024 * 4;          // two tiles' carries
    CHECK(fcoo_spttmc(t, 0, f, FCOO_F32, k, out, nullptr) == FCOO_OK);
    fcoo_destroy(t);
}

// The launch after the tile kernel stays below 2^32 threads with the most and
// shortest tiles that a tensor can have, wide rows included.
static void finish_grid()
{
    using namespace fcoo;
    for (int R : {1, 64, 256, 1024, 16384}) {
        Built b;
        b.op = FCOO_OP_MTTKRP;
        b.nnz = INT32_MAX;
        b.pmodes = {1, 2};
        b.set_plans(256, true);
        Plan &pl = b.plan[0];
        pl.fix.resize((size_t)3 * pl.ntiles);
        pl.nshort = pl.ntiles;
        TileProblem p{};
        p.b = &b;
        p.plan = &pl;
        p.R = R;
        p.kron = R > 256;
        p.kr[0] = R / 64, p.kr[1] = 64;
        p.fac_rows[0] = p.fac_rows[1] = 10;
        CHECK(launch_segmented(p, nullptr, false) == FCOO_OK);
        CHECK((uint64_t)fake::grid.x * fake::block.x < (1ull << 32));
    }
}

// No host allocation that a build is refused leaves it by an exception: the C entry
// returns FCOO_ENOMEM, and the next build succeeds.
static void host_memory(int device, int single_pass)
{
    fcoo_tensor *t = tensor({300, 200, 100}, 5000);
    fcoo_opts o{};
    o.device = device;
    o.single_pass = single_pass;
    int rc = FCOO_ENOMEM;
    for (int k = 0; rc != FCOO_OK; ++k) {
        CHECK(k < 1000);
        refuse_in = k;
        rc = fcoo_build(t, 0, FCOO_OP_MTTKRP, &o, nullptr);
        const bool refused = refuse_in < 0;
        refuse_in = -1;
        CHECK(rc == (refused ? FCOO_ENOMEM : FCOO_OK));
    }
    fcoo_destroy(t);
}

// bfloat16 CP-ALS keeps one order of sums at every rank: a lane a column wherever the
// vector of 8 (of 4 with two product modes) does not divide it.
static void kept_order()
{
    using namespace fcoo;
    for (int np : {1, 2, 3, 4})
        for (int lane_cols : {0, 4, 8})
            for (int R = 1; R <= 64; ++R) {
                Built b;
                b.op = FCOO_OP_MTTKRP;
                b.pmodes.resize(np);
                b.lane_cols = lane_cols;
                const bool four = np <= 3 && (lane_cols == 4 || (lane_cols == 0 && np == 2));
                const int V = four && R % 4 == 0 ? 4 : 8;
                const LaneShape sh = lane_shape(b, FCOO_BF16, R, false, true);
                CHECK(R % V ? sh.vw == 1 && sh.lpn == 64 : sh.vw == V && sh.half == (V == 4));
            }
}

// The GPU builds of small tensors take little more memory than their arrays.
static void small_builds()
{
    fcoo_opts o{};
    o.device = 1;
    std::vector<fcoo_tensor *> ts(101);
    size_t before = 0;
    for (auto &t : ts) {
        t = tensor({200, 150, 100}, 1000);
        CHECK(fcoo_build(t, 0, FCOO_OP_MTTKRP, &o, nullptr) == FCOO_OK);
        if (t == ts[0]) before = fake::live_bytes;
    }
    CHECK(fake::live_bytes - before < (size_t)100 * 128 * 1024);
    for (auto t : ts) fcoo_destroy(t);
    CHECK(fake::live_bytes == 0);
}

int main(int argc, char **argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    const std::map<std::string, std::function<void()>> checks = {
        {"cp_workspace_f32", [] {
             cp_workspace({140000, 120000, 50}, 8, FCOO_F32);
             cp_workspace({131073, 131072, 5}, 16, FCOO_F32);
             cp_workspace({50, 131072, 131073, 262145}, 33, FCOO_F32);
         }},
        {"cp_workspace_bf16", [] {
             cp_workspace({524289, 524288, 50}, 16, FCOO_BF16);
             cp_workspace({600000, 500000, 50}, 8, FCOO_BF16);
         }},
        {"pool_device", [] { pool_device(); }},
        {"pool_gives_way", [] { pool_gives_way(); }},
        {"build_without_carries", [] { build_without_carries(0), build_without_carries(1); }},
        {"scratch_stays_small", [] { scratch_stays(5000, {30, 20, 10}), scratch_stays(300000, {300, 200, 10}); }},
        {"scratch_stays_large", [] { scratch_stays(1500000, {3000, 200, 10}); }},
        {"carries_hold", [] {
             for (int64_t Z : {1, 300, 5000, 250000, 450000, 1100000})
                 for (int tile : {0, 256, 1024, 65536}) carries_hold({30, 20}, Z, tile), carries_hold({30, 20, 10}, Z, tile);
         }},
        {"carries_that_fit", [] { carries_that_fit(); }},
        {"values_padded", [] {
             for (int64_t Z : {1, 4, 1024, 3072, 5001}) values_padded(Z, 200, false), values_padded(Z, 8, true);
         }},
        {"finish_grid", [] { finish_grid(); }},
        {"host_memory", [] { host_memory(0, 0), host_memory(0, 1), host_memory(1, 0), host_memory(1, 1); }},
        {"kept_order", [] { kept_order(); }},
        {"small_builds", [] { small_builds(); }},
    };
    const auto it = checks.find(name);
    if (it == checks.end()) {
        for (const auto &c : checks) printf("%s\n", c.first.c_str());
        return 2;
    }
    it->second();
    return 0;
}
