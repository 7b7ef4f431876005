// Host side of the F-COO library: the handle, the per-(op, mode) F-COO
// build (mode sort, bf / sf flags, per-segment and per-tile indexing, the
// carry fix-up list), the one-time upload, export, and argument checking of
// the C ABI.  F-COO itself is defined in Sec. IV-B; the build runs on the
// host once per mode and is uploaded once (Sec. IV-D, "complete tensor-based
// algorithms").
#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <thread>

#include "fcoo_internal.h"

namespace fcoo {

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string g_err;

int fail(int code, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

int hip_fail(hipError_t e, const char *what)
{
    if (e == hipErrorOutOfMemory) return fail(FCOO_ENOMEM, "%s: %s", what, hipGetErrorString(e));
    return fail(FCOO_EHIP, "%s: %s", what, hipGetErrorString(e));
}

void clear_error() { g_err.clear(); }

// ---------------------------------------------------------------------------
// small parallel helpers (std::thread; the host build is a one-time cost)
// ---------------------------------------------------------------------------
static int host_threads()
{
    const char *e = getenv("FCOO_HOST_THREADS");
    int n = e ? atoi(e) : (int)std::thread::hardware_concurrency();
    if (n < 1) n = 1;
    if (n > 32) n = 32;
    return n;
}

template <class F>
static void parallel_chunks(int64_t n, int T, F fn)
{
    if (T <= 1 || n < 65536) {
        fn(0, (int64_t)0, n);
        return;
    }
    std::vector<std::thread> th;
    th.reserve(T);
    for (int t = 0; t < T; ++t)
        th.emplace_back([=]() { fn(t, n * t / T, n * (t + 1) / T); });
    for (auto &x : th) x.join();
}

// Stable LSD radix sort of (key, id) pairs, 11-bit digits, `bits` significant
// key bits.  Ties keep their incoming order.
static void radix_sort(std::vector<uint64_t> &k, std::vector<uint32_t> &v, int bits, int T)
{
    const int64_t n = (int64_t)k.size();
    if (n < 2 || bits <= 0) return;
    constexpr int DB = 11, NB = 1 << DB;
    std::vector<uint64_t> k2(n);
    std::vector<uint32_t> v2(n);
    if (n < 65536) T = 1;
    std::vector<int64_t> hist((size_t)T * NB);
    for (int shift = 0; shift < bits; shift += DB) {
        std::fill(hist.begin(), hist.end(), 0);
        parallel_chunks(n, T, [&](int t, int64_t b, int64_t e) {
            int64_t *h = hist.data() + (size_t)t * NB;
            for (int64_t i = b; i < e; ++i) h[(k[i] >> shift) & (NB - 1)]++;
        });
        bool trivial = false;
        for (int d = 0; d < NB && !trivial; ++d) {
            int64_t c = 0;
            for (int t = 0; t < T; ++t) c += hist[(size_t)t * NB + d];
            if (c == n) trivial = true;
            else if (c) break;
        }
        if (trivial) continue;
        int64_t run = 0;
        for (int d = 0; d < NB; ++d)
            for (int t = 0; t < T; ++t) {
                int64_t c = hist[(size_t)t * NB + d];
                hist[(size_t)t * NB + d] = run;
                run += c;
            }
        parallel_chunks(n, T, [&](int t, int64_t b, int64_t e) {
            int64_t *h = hist.data() + (size_t)t * NB;
            for (int64_t i = b; i < e; ++i) {
                int64_t p = h[(k[i] >> shift) & (NB - 1)]++;
                k2[p] = k[i];
                v2[p] = v[i];
            }
        });
        k.swap(k2);
        v.swap(v2);
    }
}

static int bit_width(int64_t d)  // bits to hold 0..d-1
{
    int b = 0;
    while (b < 63 && ((int64_t)1 << b) < d) ++b;
    return b;
}

int64_t Built::format_bytes() const
{
    return 4 * nnz * (int64_t)pmodes.size() + 4 * nnz + (nnz + 7) / 8 + 4 * ((npart + 31) / 32);
}

namespace {
std::mutex g_pool_mu;
std::vector<PoolBlock> g_pool;               // idle blocks
size_t g_pool_bytes = 0;
int g_handles = 0;

// every idle block that `which` picks, back to the driver (g_pool_mu held)
template <class F>
void pool_trim(F which)
{
    for (size_t i = 0; i < g_pool.size();) {
        if (!which(g_pool[i])) { ++i; continue; }
        (void)hipFree(g_pool[i].p);
        g_pool_bytes -= g_pool[i].bytes;
        g_pool[i] = g_pool.back();
        g_pool.pop_back();
    }
}
}  // namespace

hipError_t device_malloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        pool_trim([&](const PoolBlock &x) { return x.dev == dev; });
    }
    return hipMalloc(p, bytes);
}

int pool_get(size_t bytes, PoolBlock *b)
{
    // (whole 2 MiB pages, but for blocks smaller than one)
    const size_t unit = bytes < ((size_t)2 << 20) ? 4096 : (size_t)2 << 20;
    bytes = (bytes + unit - 1) / unit * unit;
    int dev = 0;
    FCOO_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> lk(g_pool_mu);
        size_t best = g_pool.size();
        for (size_t i = 0; i < g_pool.size(); ++i)
            if (g_pool[i].dev == dev && g_pool[i].bytes >= bytes && g_pool[i].bytes <= bytes + bytes / 4 &&
                (best == g_pool.size() || g_pool[i].bytes < g_pool[best].bytes))
                best = i;
        if (best < g_pool.size()) {
            *b = g_pool[best];
            g_pool_bytes -= b->bytes;
            g_pool[best] = g_pool.back();
            g_pool.pop_back();
            return FCOO_OK;
        }
    }
    b->bytes = bytes;
    b->dev = dev;
    if (device_malloc(&b->p, bytes) == hipSuccess) return FCOO_OK;
    (void)hipGetLastError();
    b->p = nullptr;
    return fail(FCOO_ENOMEM, "device build (%lld bytes)", (long long)bytes);
}

void pool_free(PoolBlock *b)
{
    if (b->p) (void)hipFree(b->p);
    *b = PoolBlock();
}

void pool_put(PoolBlock *b)
{
    if (!b->p) return;
    std::lock_guard<std::mutex> lk(g_pool_mu);
    if (g_handles > 0 && g_pool_bytes + b->bytes <= kPoolKeep && g_pool.size() < kPoolBlocks) {
        try {
            g_pool.push_back(*b);
            g_pool_bytes += b->bytes;
            *b = PoolBlock();
            return;
        } catch (const std::bad_alloc &) {
        }
    }
    pool_free(b);
}

void pool_handles(int delta)
{
    std::lock_guard<std::mutex> lk(g_pool_mu);
    g_handles += delta;
    if (g_handles == 0) pool_trim([](const PoolBlock &) { return true; });
}

void Built::free_device()
{
    if (arena.p) {
        // work queued on any stream of the block's device (the current one may be
        // another) may still read the arrays, as before a hipFree, which waits;
        // where the wait is refused (a stream is being captured) the block goes to
        // the driver
        int cur = arena.dev;
        (void)hipGetDevice(&cur);
        bool idle = cur == arena.dev || hipSetDevice(arena.dev) == hipSuccess;
        idle = idle && hipDeviceSynchronize() == hipSuccess;
        if (!idle) (void)hipGetLastError();
        if (cur != arena.dev) (void)hipSetDevice(cur);
        if (idle) pool_put(&arena);
        else pool_free(&arena);
        for (auto &p : d_pidx) p = nullptr;
        d_val = nullptr; d_hr = nullptr; d_bf = nullptr; d_sf = nullptr; d_seg_row = nullptr;
        d_perm = nullptr; d_fix = nullptr; d_empty = nullptr;
    }
    for (auto &p : d_pidx) { if (p) (void)hipFree(p); p = nullptr; }
    void *ptrs[] = {d_val, d_hr, d_bf, d_sf, d_seg_row, d_perm, d_fix, d_empty, d_carry, d_bpart,
                    d_partial, d_gperm, d_sp_from, d_sp_words, d_sp_ticket, d_sp_err};
    for (void *p : ptrs) if (p) (void)hipFree(p);
    d_val = nullptr; d_hr = nullptr; d_bf = nullptr; d_sf = nullptr; d_seg_row = nullptr;
    d_perm = nullptr; d_fix = nullptr; d_empty = nullptr; d_carry = nullptr; d_bpart = nullptr;
    d_partial = nullptr; d_gperm = nullptr; d_sp_from = nullptr; d_sp_words = nullptr; d_sp_ticket = nullptr; d_sp_err = nullptr;
    carry_cap = 0; carry_width = 0; bpart_cap = 0; partial_cap = 0; gperm_cap = 0; device_bytes = 0;
    sp_words_cap = 0; sp_tickets = 0; sp_epoch = 0;
    on_device = false;
}

void Workspace::free_all()
{
    if (M) (void)hipFree(M);
    if (dbl) (void)hipFree(dbl);
    if (host_pinned) (void)hipHostFree(host_pinned);
    M = nullptr; dbl = nullptr; host_pinned = nullptr;
    M_cap = dbl_cap = 0;
}

// Grow a device scratch buffer.  The old buffer may still be read by work
// queued on `s`, so the stream is drained before it is released.
int ensure_device_floats(float **p, int64_t *cap, int64_t need, hipStream_t s)
{
    if (need <= *cap) return FCOO_OK;
    if (*p) {
        FCOO_HIP(hipStreamSynchronize(s));
        FCOO_HIP(hipFree(*p));
        *p = nullptr;
        *cap = 0;
    }
    FCOO_HIP(device_malloc((void **)p, (size_t)need * sizeof(float)));
    *cap = need;
    return FCOO_OK;
}

int ensure_device_doubles(double **p, int64_t *cap, int64_t need, hipStream_t s)
{
    if (need <= *cap) return FCOO_OK;
    if (*p) {
        FCOO_HIP(hipStreamSynchronize(s));
        FCOO_HIP(hipFree(*p));
        *p = nullptr;
        *cap = 0;
    }
    FCOO_HIP(device_malloc((void **)p, (size_t)need * sizeof(double)));
    *cap = need;
    return FCOO_OK;
}

template <class T>
static int upload(T **dst, const T *src, int64_t n, int64_t pad_elems, hipStream_t s, int64_t *acct)
{
    const size_t bytes = (size_t)(n + pad_elems) * sizeof(T);
    FCOO_HIP(device_malloc((void **)dst, bytes ? bytes : sizeof(T)));
    if (pad_elems) FCOO_HIP(hipMemsetAsync(*dst, 0, bytes, s));
    if (n) FCOO_HIP(hipMemcpyAsync(*dst, src, (size_t)n * sizeof(T), hipMemcpyHostToDevice, s));
    *acct += (int64_t)bytes;
    return FCOO_OK;
}

int upload_i32(int32_t **dst, const std::vector<int32_t> &v, int64_t pad, hipStream_t s, int64_t *acct)
{
    return upload(dst, v.data(), (int64_t)v.size(), pad, s, acct);
}

int upload_coo(fcoo_tensor *t, hipStream_t s)
{
    if (t->coo_on_device) return FCOO_OK;
    int64_t acct = 0;
    for (int m = 0; m < t->order; ++m) {
        int rc = upload(&t->d_coo[m], t->idx[m].data(), t->nnz, 0, s, &acct);
        if (rc) return rc;
    }
    int rc = upload(&t->d_coo_val, t->vals.data(), t->nnz, 0, s, &acct);
    if (rc) return rc;
    FCOO_HIP(hipStreamSynchronize(s));
    t->coo_on_device = true;
    return FCOO_OK;
}

int check_factors(const fcoo_tensor *t, int skip_mode, const void *const *factors, int dtype, int R)
{
    if (!factors) return fail(FCOO_EINVAL, "factors is NULL");
    if (dtype != FCOO_F32 && dtype != FCOO_BF16) return fail(FCOO_EUNSUPPORTED, "unknown dtype %d", dtype);
    if (R < 1 || R > kMaxR) return fail(FCOO_EUNSUPPORTED, "R = %d outside [1, %d]", R, kMaxR);
    for (int m = 0; m < t->order; ++m)
        if (m != skip_mode && !factors[m]) return fail(FCOO_EINVAL, "factors[%d] is NULL", m);
    return FCOO_OK;
}

// XCD blocks: the product mode with the most rows is split into nblk index
// ranges holding about Z / nblk nonzeros each; block b's nonzeros lead the
// sort order as a group, and its tiles are those that start inside it.
int setup_blocks(const fcoo_tensor *t, Built &b, int nblk, int xmode)
{
    b.nblk = 1;
    b.bmode = -1;
    b.blk_of.clear();
    b.rows = b.op == FCOO_OP_MTTKRP ? t->dims[b.mode] : 0;
    if (nblk <= 1) return FCOO_OK;
    if (nblk != kXcds) return fail(FCOO_EINVAL, "xcd_blocks must be 0, 1 or %d (got %d)", kXcds, nblk);
    if (b.op != FCOO_OP_MTTKRP) return fail(FCOO_EINVAL, "xcd_blocks applies to SpMTTKRP builds");
    if ((int64_t)nblk * t->dims[b.mode] > (int64_t)0x7fffffff)
        return fail(FCOO_EUNSUPPORTED, "xcd_blocks: %d x dims[mode] exceeds the int32 row range", nblk);
    int bm = -1;
    if (xmode >= 0) {
        for (int m : b.pmodes) if (m == xmode) bm = m;
        if (bm < 0) return fail(FCOO_EINVAL, "xcd_mode: mode %d is not a product mode of this build", xmode);
    } else {
        bm = b.pmodes[0];
        for (int m : b.pmodes) if (t->dims[m] > t->dims[bm]) bm = m;
    }
    const int64_t D = t->dims[bm], Z = t->nnz;
    std::vector<int64_t> cnt(D, 0);
    for (int64_t e = 0; e < Z; ++e) cnt[t->idx[bm][e]]++;
    b.blk_of.resize(D);
    std::vector<int64_t> zs(nblk + 1, 0);
    int64_t before = 0;
    for (int64_t i = 0; i < D; ++i) {
        int blk = Z > 0 ? (int)((before * nblk) / Z) : 0;
        if (blk >= nblk) blk = nblk - 1;
        b.blk_of[i] = blk;
        zs[blk + 1] += cnt[i];
        before += cnt[i];
    }
    for (int k = 0; k < nblk; ++k) zs[k + 1] += zs[k];
    for (Plan &pl : b.plan) {
        pl.blk_ts.assign(nblk + 1, 0);
        for (int k = 1; k < nblk; ++k) {
            const int64_t ts = std::min(zs[k] / pl.T, pl.ntiles);
            pl.blk_ts[k] = std::max(ts, pl.blk_ts[k - 1]);
        }
        pl.blk_ts[nblk] = pl.ntiles;
    }
    b.nblk = nblk;
    b.bmode = bm;
    return FCOO_OK;
}

int setup_single_pass(Built &b, hipStream_t s)
{
    if (b.nblk > 1) return fail(FCOO_EINVAL, "single_pass needs the plain layout (no xcd_blocks)");
    if (b.ntiles > (int64_t)0x7fffffff) return fail(FCOO_EUNSUPPORTED, "single_pass: too many tiles");
    const Plan &pl = b.plan[0];
    std::vector<int32_t> from(b.ntiles + 1, -1);
    b.sp_tail_from = -1;
    for (int64_t e = 0; e < pl.nfix(); ++e) {
        const int32_t tb = pl.fix[3 * e], ta = pl.fix[3 * e + 1];
        if (tb < b.ntiles) from[tb] = ta;
        else b.sp_tail_from = ta;
    }
    int64_t acct = 0;
    int rc = upload_i32(&b.d_sp_from, from, 0, s, &acct);
    if (rc) return rc;
    FCOO_HIP(device_malloc((void **)&b.d_sp_ticket, sizeof(unsigned long long)));
    FCOO_HIP(device_malloc((void **)&b.d_sp_err, sizeof(int)));
    FCOO_HIP(hipMemsetAsync(b.d_sp_ticket, 0, sizeof(unsigned long long), s));
    FCOO_HIP(hipMemsetAsync(b.d_sp_err, 0, sizeof(int), s));
    FCOO_HIP(hipStreamSynchronize(s));
    b.device_bytes += acct + (int64_t)sizeof(unsigned long long) + (int64_t)sizeof(int);
    b.sp_tickets = 0;
    b.sp_epoch = 0;
    b.sp = true;
    return FCOO_OK;
}

int prep_single_pass(Built *b, TileProblem &p, hipStream_t s)
{
    if (!b->sp || b->nnz == 0 || p.kron) return FCOO_OK;
    const int64_t need = 2 * b->ntiles * (int64_t)p.R;
    if (need > b->sp_words_cap) {
        // fresh words hold tag 0, which no launch uses
        if (b->d_sp_words) {
            FCOO_HIP(hipStreamSynchronize(s));
            FCOO_HIP(hipFree(b->d_sp_words));
            b->d_sp_words = nullptr;
            b->sp_words_cap = 0;
        }
        FCOO_HIP(device_malloc((void **)&b->d_sp_words, (size_t)need * sizeof(uint64_t)));
        FCOO_HIP(hipMemsetAsync(b->d_sp_words, 0, (size_t)need * sizeof(uint64_t), s));
        b->sp_words_cap = need;
    }
    if (++b->sp_epoch == 0) b->sp_epoch = 1;
    p.sp_words = b->d_sp_words;
    p.sp_epoch = b->sp_epoch;
    return FCOO_OK;
}

// The tile sizes a build can be launched with: the format's, and below it those
// that pick_plan chooses from (with a caller's own size for SpTTMc only).
void Built::set_plans(int fmt_tile, bool own)
{
    own_tile = own;
    plan.clear();
    plan.resize(1);
    plan[0].T = fmt_tile;
    for (int t : {2048, 1024, 512, 256, 128, 64}) {
        if (t >= plan.back().T || fmt_tile % t || (t < 256 && nnz >= 4000000)) continue;
        plan.emplace_back();
        plan.back().T = t;
    }
    for (Plan &pl : plan) pl.ntiles = (nnz + pl.T - 1) / pl.T;
}

// A tile costs a chain of dependent loads at its start and end whatever its
// length, so tiles are long where there are enough of them to fill 256 CUs
// several times over and short where there are not; a run stays a power of two
// long (runs that start inside a 128-byte line of the streams cost 10-20%), and
// with 4 lanes a row or fewer a lane group's stream vectors cover less than a
// line, so neighbouring runs should share it: 1024 nonzeros, one super-chunk a
// run.  Measured on Zipf(1.1) tensors, whole calls, 512 / 1024 / 2048 / 4096
// nonzeros a tile (us):
//   SpMTTKRP float32 R = 32 (8 lanes): 100k 13.6 / 13.7 / 16.3 / 24.9, 400k 17.1 /
//   13.5 / 16.9 / 26.0, 1.5M 40.5 / 26.1 / 26.1 / 33.6, 5M 113 / 67 / 67 / 77, 20M
//   412 / 226 / 216 / 219; R = 16 (4 lanes): 20M 326 / 187 / 196 / 205; R = 8: 289 /
//   169 / 177 / 242;
//   residual R = 64: 5M 209 / 133 / 139 / 168, 20M 792 / 470 / 444 / 438;
//   SpTTM R = 32: 400k 15.4 / 13.1 / 15.6 / 24.8, 5M 114 / 75 / 78 / 102, 20M 419 /
//   262 / 272 / 320; R = 8: 248 / 236 / 284 / 381.
// One lane a row or pieces of two columns take 2048: a lane's run is 4 nonzeros at
// 1024 (1024 / 2048 / 4096: SpMTTKRP of 8M, R = 4 62 / 43 / 69; 7M, order 2, bfloat16 R =
// 8 56 / 39 / 49; 1.6M, R = 3 24 / 18 / 22; but five modes, whose path has no vectors,
// 2.7M, R = 4 45 / 65 / 110).  Rows over several rank tiles have several workgroups a
// tile, so 1024 from 60k nonzeros on (512 / 1024: 100k, R = 200 31 / 19; 190k 44 / 26;
// 34k, R = 100 19 / 21).  Fibres of hardly more than one nonzero under 8-column
// bfloat16 lanes: 512 (512 / 1024 / 4096: 2.4M, R = 16 68 / 94 / 103, R = 80 237 / 319 /
// 316), but for wide rows in a few hundred tiles of 4096, each lane group of which
// writes its own long stretch (750k, R = 80 90 / 103 / 66; 150k 24 / 21 / 56).
// SpTTMc: a wave takes a tile, whatever tile a workgroup of the other operations was
// asked to take, and where segments are short it stores row after row, so tiles are
// as short as leaves each SIMD several waves (64 / 128 / 256 / 512 / 1024 / 4096
// nonzeros: 20k, ranks 8 x 8, rows of one nonzero 44 / 66 / 112 / 202 / 379 / 1428;
// 100k, 16 x 16, rows of 50 13 / 14 / 14 / 20 / 34 / 108; 600k, 8 x 8, rows of 3 38 / 36
// / 45 / 63 / 103 / 371; 1.6M Zipf, 16 x 16 100 / 77 / 80 / 103 / 167 / 587; 8M, 16 x 16,
// rows of 4000 (256) 102 / 97 / 97 / 106; 10M Zipf, rows in no order (512) 183 / 180), a
// size longer where wide, long rows make little work between carries (1.5M, 16 x 16,
// rows of 750 (256) 31 / 26) or a size shorter where they are few nonzeros long
// (1.4M Zipf over 129k rows, 1 x 8 (256) 52 / 39; 3M over 100k, 16 x 16 78 / 88), and
// unless their carries would pass kTtmcCarries.  Past 64M nonzeros short tiles gain
// nothing that their carries' scratch would be worth.
constexpr int64_t kTtmcCarries = (int64_t)64 << 20;      // floats

const Plan &pick_plan(const Built &b, int dtype, int R, bool resid, bool kron)
{
    const bool large = b.nnz > (int64_t)64000000;
    int want = b.plan[0].T;
    if (kron) {
        const bool short_rows = b.nnz < (R < 128 ? 40 : 8) * b.nseg, long_rows = R >= 128 && b.nnz > 300 * b.nseg;
        want = b.nnz < 150000 ? 64 : b.nnz < (short_rows ? 4000000 : 700000) ? 128
             : b.nnz < (long_rows ? 1200000 : 4000000) ? 256 : b.nnz < 8000000 ? 512 : large ? 2048 : 1024;
        for (size_t i = b.plan.size() - 1; i > 0; --i)
            if (b.plan[i].T >= want && 2 * b.plan[i].ntiles * (int64_t)R <= kTtmcCarries) return b.plan[i];
        return b.plan[0];
    }
    if (b.own_tile || large) return b.plan[0];
    const LaneShape sh = lane_shape(b, dtype, R, resid);
    const bool vectors = sh.vw > 1 && b.pmodes.size() <= 3;
    if (vectors && (sh.lpn == 1 || sh.vw == 2)) {
        want = 2048;
    } else {
        if (b.op == FCOO_OP_TTM && sh.vw == 8 && b.nnz < 2 * b.nseg) {
            if (R > 64 && b.nnz >= 500000 && b.nnz < 1600000) return b.plan[0];
            want = 512;
        } else if (b.op == FCOO_OP_TTM || sh.lpn <= 4) {
            want = 1024;
        } else {
            want = resid && b.nnz >= 10000000 ? 4096 : 2048;
        }
        if (b.nnz < 1000000) want = std::min(want, 1024);
    }
    if (b.nnz < (R > sh.lpn * sh.vw ? 60000 : 200000)) want = std::min(want, 512);
    for (const Plan &pl : b.plan)
        if (pl.T <= want) return pl;
    return b.plan.back();
}

// ---------------------------------------------------------------------------
// the F-COO build for one (op, mode)
// ---------------------------------------------------------------------------
static int build_host(fcoo_tensor *t, Built &b, int mode, int op, int threadlen, int tile_nnz, bool own_tile, int nblk,
                      int xmode)
{
    const int N = t->order;
    const int64_t Z = t->nnz;
    const int T = host_threads();
    b = Built();
    b.op = op; b.mode = mode; b.threadlen = threadlen; b.tile_nnz = tile_nnz; b.nnz = Z;
    b.set_plans(tile_nnz, own_tile);
    for (int m = 0; m < N; ++m) {
        if (m == mode) continue;
        if (op == FCOO_OP_MTTKRP) b.pmodes.push_back(m); else b.imodes.push_back(m);
    }
    if (op == FCOO_OP_MTTKRP) b.imodes.insert(b.imodes.begin(), mode); else b.pmodes.push_back(mode);
    int rc0 = setup_blocks(t, b, nblk, xmode);
    if (rc0) return rc0;
    const bool blocked = b.nblk > 1;
    const int bbits = blocked ? bit_width(b.nblk) : 0;

    // 1. stable lexicographic order of (block, index-mode tuple, product-mode tuple)
    std::vector<int> order_modes(b.imodes);
    order_modes.insert(order_modes.end(), b.pmodes.begin(), b.pmodes.end());
    int total_bits = bbits, pbits = 0;
    for (int m : b.imodes) total_bits += bit_width(t->dims[m]);
    for (int m : b.pmodes) { int w = bit_width(t->dims[m]); total_bits += w; pbits += w; }
    std::vector<uint32_t> perm(Z);
    std::vector<uint64_t> key;
    const bool packed = total_bits <= 64;
    if (packed) {
        key.resize(Z);
        parallel_chunks(Z, T, [&](int, int64_t lo, int64_t hi) {
            for (int64_t e = lo; e < hi; ++e) {
                uint64_t k = blocked ? (uint64_t)b.blk_of[t->idx[b.bmode][e]] : 0;
                for (int m : order_modes) k = (bit_width(t->dims[m]) ? (k << bit_width(t->dims[m])) : k) | (uint64_t)t->idx[m][e];
                key[e] = k;
                perm[e] = (uint32_t)e;
            }
        });
        radix_sort(key, perm, total_bits, T);
    } else {
        for (int64_t e = 0; e < Z; ++e) perm[e] = (uint32_t)e;
        std::stable_sort(perm.begin(), perm.end(), [&](uint32_t x, uint32_t y) {
            if (blocked) {
                const int bx = b.blk_of[t->idx[b.bmode][x]], by = b.blk_of[t->idx[b.bmode][y]];
                if (bx != by) return bx < by;
            }
            for (int m : order_modes) {
                int32_t a = t->idx[m][x], c = t->idx[m][y];
                if (a != c) return a < c;
            }
            return false;
        });
    }

    // 2. per-nonzero arrays in sorted order, and segment heads
    b.perm.resize(Z);
    b.val.resize(Z);
    b.pidx.assign(b.pmodes.size(), std::vector<int32_t>(Z));
    std::vector<uint8_t> head(Z);
    parallel_chunks(Z, T, [&](int, int64_t lo, int64_t hi) {
        for (int64_t s = lo; s < hi; ++s) {
            const uint32_t e = perm[s];
            b.perm[s] = (int32_t)e;
            b.val[s] = t->vals[e];
            for (size_t q = 0; q < b.pmodes.size(); ++q) b.pidx[q][s] = t->idx[b.pmodes[q]][e];
            bool h = (s == 0);
            if (!h) {
                if (packed) {
                    h = pbits < 64 && (key[s] >> pbits) != (key[s - 1] >> pbits);
                } else {
                    if (blocked) h = b.blk_of[t->idx[b.bmode][e]] != b.blk_of[t->idx[b.bmode][perm[s - 1]]];
                    for (int m : b.imodes)
                        if (!h && t->idx[m][e] != t->idx[m][perm[s - 1]]) { h = true; break; }
                }
            }
            head[s] = h;
        }
    });
    key.clear(); key.shrink_to_fit();

    // 3. bf (parity toggled at each head, starting at 1), sf, segments, tiles
    const int64_t P = (Z + threadlen - 1) / threadlen;
    const int64_t ntiles = (Z + tile_nnz - 1) / tile_nnz;
    b.npart = P; b.ntiles = ntiles;
    const Plan &fine = b.plan.back();
    const int wtile = fine.T;
    b.bf.assign((Z + 7) / 8, 0);
    b.sf.assign((P + 31) / 32, 0);
    b.tile_seg0.resize(ntiles);
    std::vector<int64_t> seg_start;  // position of each head
    std::vector<int64_t> heads_before_tile(fine.ntiles + 1, 0);
    int64_t cnt = 0;
    for (int64_t s = 0; s < Z; ++s) {
        const bool starts = s % wtile == 0;      // (a tile as launched; every format tile starts one)
        if (starts) heads_before_tile[s / wtile] = cnt;
        if (head[s]) {
            ++cnt;
            seg_start.push_back(s);
            b.sf[(s / threadlen) >> 5] |= 1u << ((s / threadlen) & 31);
        }
        if (cnt & 1) b.bf[s >> 3] |= (uint8_t)(1u << (s & 7));
        if (starts && s % tile_nnz == 0) b.tile_seg0[s / tile_nnz] = (int32_t)(cnt - 1);
    }
    heads_before_tile[fine.ntiles] = cnt;
    b.nseg = cnt;
    const int nim = (int)b.imodes.size();
    b.seg.resize((size_t)cnt * nim);
    for (int64_t g = 0; g < cnt; ++g) {
        const uint32_t e = perm[seg_start[g]];
        for (int q = 0; q < nim; ++q) b.seg[(size_t)g * nim + q] = t->idx[b.imodes[q]][e];
        if (blocked) b.seg[g] += b.blk_of[t->idx[b.bmode][e]] * (int32_t)t->dims[mode];
    }

    // 4. carry fix-up list and empty rows
    finish_tiles(t, b, mode, op, heads_before_tile);
    b.built = true;
    return FCOO_OK;
}

// Carry fix-up list: a segment that is still open at the end of a tile is
// finished by the first head of a later tile (or by the end of the tensor).
// Entry (b, a, row): tiles a+1 .. b-1 hold no head, tile a holds the segment's
// start.  The segment closed at tile b's first head is the last one that
// starts before tile b.  Then the output rows of MTTKRP that no nonzero
// touches (with XCD blocks: rows of the nblk x dims[mode] partial output).
void finish_tiles(const fcoo_tensor *t, Built &b, int mode, int op, const std::vector<int64_t> &hb)
{
    const int64_t cnt = b.nseg;
    auto out_row = [&](int64_t g) -> int32_t {
        return op == FCOO_OP_MTTKRP ? b.seg[(size_t)g] : (int32_t)g;
    };
    int64_t at = 0;
    for (Plan &pl : b.plan) {
        const int64_t ntiles = pl.ntiles, k = pl.T / b.plan.back().T, nfine = b.plan.back().ntiles;
        std::vector<int32_t> middle, shortest;
        pl.fix.clear();
        int64_t last = -1;
        auto add = [&](int64_t tb, int64_t g) {
            std::vector<int32_t> &to = tb - last > kLongChain ? pl.fix : tb - last > 2 ? middle : shortest;
            to.push_back((int32_t)tb);
            to.push_back((int32_t)last);
            to.push_back(out_row(g));
        };
        for (int64_t tb = 0; tb < ntiles; ++tb) {
            const int64_t h0 = hb[tb * k], h1 = hb[std::min((tb + 1) * k, nfine)];
            if (h1 == h0) continue;                  // no head in tile tb
            if (tb >= 1) add(tb, h0 - 1);
            last = tb;
        }
        if (b.nnz > 0) add(ntiles, cnt - 1);
        pl.nlong = pl.nfix();
        pl.nshort = (int64_t)shortest.size() / 3;
        pl.fix.insert(pl.fix.end(), middle.begin(), middle.end());
        pl.fix.insert(pl.fix.end(), shortest.begin(), shortest.end());
        pl.fix_at = at;
        at += pl.nfix();
    }
    b.empty_rows.clear();
    if (op == FCOO_OP_MTTKRP) {
        const int64_t rows = (int64_t)b.nblk * t->dims[mode];
        std::vector<uint8_t> present(rows, 0);
        for (int64_t g = 0; g < cnt; ++g) present[b.seg[g]] = 1;
        for (int64_t i = 0; i < rows; ++i)
            if (!present[i]) b.empty_rows.push_back((int32_t)i);
    }
}

std::vector<int32_t> all_fixes(const Built &b)
{
    std::vector<int32_t> all;
    for (const Plan &pl : b.plan) all.insert(all.end(), pl.fix.begin(), pl.fix.end());
    return all;
}

// the plans' fix-up lists, one after the other (the copy ends before it returns)
static int upload_plans(Built &b, hipStream_t s, int64_t *acct)
{
    const std::vector<int32_t> all = all_fixes(b);
    int rc = upload(&b.d_fix, all.data(), (int64_t)all.size(), 3, s, acct);
    if (!rc) FCOO_HIP(hipStreamSynchronize(s));
    return rc;
}

// Most tiles that an operation takes.
static int64_t most_tiles(const Built &b)
{
    const int64_t n = std::max(pick_plan(b, FCOO_F32, 16, false, false).ntiles, pick_plan(b, FCOO_BF16, 16, false, false).ntiles);
    return b.pmodes.size() > 1 ? std::max(n, pick_plan(b, FCOO_F32, 16, false, true).ntiles) : n;
}

// Carries that no operation on rows of `width` columns or fewer outgrows, whatever
// tiles it takes.  Scratch that is let go of may be in a captured graph, and none
// can be had while a stream is being captured: what a caller's widest rows have
// been through holds for all narrower ones.
static int64_t carry_need(const Built &b, int64_t width)
{
    return std::min(2 * most_tiles(b) * width, std::max(kTtmcCarries, 2 * b.plan[0].ntiles * width));
}

// Carries for rows of up to 64 columns (4 bytes for every 8 nonzeros), so that
// the first operation need not allocate them; wider rows grow them.  A build whose
// arrays leave no room for them is none the worse: that operation asks again.
static void first_carries(Built &b, hipStream_t s)
{
    if (b.nnz == 0) return;
    if (ensure_device_floats(&b.d_carry, &b.carry_cap, carry_need(b, 64), s) == FCOO_OK) {
        b.carry_width = 64;
    } else {
        (void)hipGetLastError();
        clear_error();
    }
}

static int build_device(Built &b, hipStream_t s)
{
    int64_t acct = 0;
    int rc;
    for (size_t q = 0; q < b.pidx.size(); ++q)
        if ((rc = upload(&b.d_pidx[q], b.pidx[q].data(), b.nnz, 4, s, &acct))) return rc;
    // 4 entries of zero padding: 16-byte stream vectors never read past the allocation
    if ((rc = upload(&b.d_val, b.val.data(), b.nnz, 4, s, &acct))) return rc;
    {   // the bf bits decoded for the kernels: per 32 nonzeros the heads (where bf
        // changes) and their running count, plus two zero pairs
        const int64_t words = (b.nnz + 31) / 32;
        std::vector<uint32_t> w(2 * words, 0);
        uint32_t last = 0, rank = 0;
        for (int64_t i = 0; i < words; ++i) {
            uint32_t x = 0;
            const int64_t left = (int64_t)b.bf.size() - 4 * i;
            memcpy(&x, b.bf.data() + 4 * i, (size_t)(left < 4 ? left : 4));
            uint32_t h = x ^ ((x << 1) | last);
            if (i == words - 1 && (b.nnz & 31)) h &= (1u << (b.nnz & 31)) - 1u;   // bf is 0 past Z
            w[2 * i] = h;
            w[2 * i + 1] = rank;
            rank += (uint32_t)__builtin_popcount(h);
            last = x >> 31;
        }
        if ((rc = upload(&b.d_hr, w.data(), 2 * words, 4, s, &acct))) return rc;
        FCOO_HIP(hipStreamSynchronize(s));
    }
    // bf itself and sf stay on the host (exported with the format)
    if (b.op == FCOO_OP_MTTKRP)
        if ((rc = upload(&b.d_seg_row, b.seg.data(), b.nseg, 2, s, &acct))) return rc;
    if ((rc = upload(&b.d_perm, b.perm.data(), b.nnz, 4, s, &acct))) return rc;
    if ((rc = upload_plans(b, s, &acct))) return rc;
    if ((rc = upload(&b.d_empty, b.empty_rows.data(), (int64_t)b.empty_rows.size(), 1, s, &acct)))
        return rc;
    FCOO_HIP(hipStreamSynchronize(s));
    b.device_bytes = acct;
    b.on_device = true;
    return FCOO_OK;
}

// The build of (op, mode), or NULL with *rc set: FCOO_EINVAL for a null
// handle, a mode outside [0, order) or an unknown op; FCOO_ENOTBUILT when
// that (op, mode) has no build (on the device, if need_device).
Built *get_built(fcoo_tensor *t, int mode, int op, bool need_device, int *rc)
{
    if (!t) { *rc = fail(FCOO_EINVAL, "null handle"); return nullptr; }
    if (mode < 0 || mode >= t->order) { *rc = fail(FCOO_EINVAL, "mode %d out of range", mode); return nullptr; }
    if (op != FCOO_OP_MTTKRP && op != FCOO_OP_TTM) { *rc = fail(FCOO_EINVAL, "unknown op %d", op); return nullptr; }
    Built &b = t->b[op][mode];
    if (!b.built || (need_device && !b.on_device)) {
        *rc = fail(FCOO_ENOTBUILT, "(op %d, mode %d) is not built%s", op, mode,
                   b.built ? " on the device" : "");
        return nullptr;
    }
    *rc = FCOO_OK;
    return &b;
}

}  // namespace fcoo

using namespace fcoo;

extern "C" {

int fcoo_version(void) { return 101; }

const char *fcoo_last_error(void) { return fcoo::g_err.c_str(); }

int fcoo_create(int order, const int64_t *dims, int64_t nnz, const int32_t *const *idx,
                const float *vals, fcoo_tensor **out)
{
    clear_error();
    if (!out) return fail(FCOO_EINVAL, "out is NULL");
    *out = nullptr;
    if (order < 2 || order > kMaxOrder) return fail(FCOO_EUNSUPPORTED, "order %d outside [2, 8]", order);
    if (!dims) return fail(FCOO_EINVAL, "dims is NULL");
    if (nnz < 0) return fail(FCOO_EINVAL, "nnz < 0");
    if (nnz > 0 && (!idx || !vals)) return fail(FCOO_EINVAL, "idx or vals is NULL");
    if (nnz > (int64_t)INT32_MAX) return fail(FCOO_ERANGE, "nnz %lld exceeds 2^31 - 1", (long long)nnz);
    for (int m = 0; m < order; ++m) {
        if (dims[m] < 1 || dims[m] > (int64_t)INT32_MAX)
            return fail(FCOO_ERANGE, "dims[%d] = %lld outside [1, 2^31 - 1]", m, (long long)dims[m]);
        if (nnz > 0 && !idx[m]) return fail(FCOO_EINVAL, "idx[%d] is NULL", m);
    }
    fcoo_tensor *t = new (std::nothrow) fcoo_tensor();
    if (!t) return fail(FCOO_ENOMEM, "handle");
    try {
        t->order = order;
        t->nnz = nnz;
        for (int m = 0; m < order; ++m) {
            t->dims[m] = dims[m];
            t->idx[m].assign(idx ? idx[m] : nullptr, idx ? idx[m] + nnz : nullptr);
        }
        t->vals.assign(vals, vals + nnz);
    } catch (const std::bad_alloc &) {
        delete t;
        return fail(FCOO_ENOMEM, "copying %lld nonzeros", (long long)nnz);
    }
    for (int m = 0; m < order; ++m) {
        const int32_t *c = t->idx[m].data();
        const int64_t d = dims[m];
        for (int64_t e = 0; e < nnz; ++e)
            if (c[e] < 0 || (int64_t)c[e] >= d) {
                int rc = fail(FCOO_ERANGE, "idx[%d][%lld] = %d outside [0, %lld)", m, (long long)e,
                              c[e], (long long)d);
                delete t;
                return rc;
            }
    }
    double s = 0.0;
    for (int64_t e = 0; e < nnz; ++e) s += (double)t->vals[e] * (double)t->vals[e];
    t->normX2 = s;
    pool_handles(1);
    *out = t;
    return FCOO_OK;
}

int fcoo_build(fcoo_tensor *t, int mode, int op, const fcoo_opts *opts, void *stream)
{
    clear_error();
    if (!t) return fail(FCOO_EINVAL, "null handle");
    if (mode < 0 || mode >= t->order) return fail(FCOO_EINVAL, "mode %d out of range", mode);
    if (op != FCOO_OP_MTTKRP && op != FCOO_OP_TTM) return fail(FCOO_EINVAL, "unknown op %d", op);
    int threadlen = opts && opts->threadlen ? opts->threadlen : 16;
    int tile_nnz = opts && opts->tile_nnz ? opts->tile_nnz : 4096;
    const bool host_only = opts && opts->host_only;
    const bool on_gpu = opts && opts->device;
    const int nblk = opts ? opts->xcd_blocks : 0;
    const int xmode = opts ? opts->xcd_mode - 1 : -1;
    const int lane_cols = opts ? opts->lane_cols : 0;
    const bool single_pass = opts && opts->single_pass;
    if (host_only && on_gpu) return fail(FCOO_EINVAL, "host_only and device are exclusive");
    if (lane_cols != 0 && lane_cols != 4 && lane_cols != 8)
        return fail(FCOO_EINVAL, "lane_cols %d not in {0, 4, 8}", lane_cols);
    if (threadlen != 8 && threadlen != 16 && threadlen != 32 && threadlen != 64)
        return fail(FCOO_EINVAL, "threadlen %d not in {8, 16, 32, 64}", threadlen);
    if (tile_nnz <= 0 || tile_nnz % 256 || tile_nnz % threadlen || tile_nnz > (1 << 20))
        return fail(FCOO_EINVAL, "tile_nnz %d must be a positive multiple of 256 and threadlen, <= 2^20",
                    tile_nnz);
    // a tile size that the caller chose is launched as it is, and so is the
    // single pass's (its chain table goes by the format's tiles)
    const bool own_tile = (opts && opts->tile_nnz) || single_pass;
    Built &b = t->b[op][mode];
    b.free_device();
    int rc;
    if (on_gpu) {
        try {
            rc = build_on_device(t, b, mode, op, threadlen, tile_nnz, own_tile, nblk, xmode, (hipStream_t)stream);
            if (!rc && single_pass) rc = setup_single_pass(b, (hipStream_t)stream);
        } catch (const std::bad_alloc &) {
            rc = fail(FCOO_ENOMEM, "device build (host side)");
        }
        if (!rc) first_carries(b, (hipStream_t)stream);
        if (rc) {
            b.free_device();
            b = Built();
        }
        b.lane_cols = lane_cols;
        return rc;
    }
    try {
        rc = build_host(t, b, mode, op, threadlen, tile_nnz, own_tile, nblk, xmode);
    } catch (const std::bad_alloc &) {
        b = Built();
        return fail(FCOO_ENOMEM, "host build");
    }
    if (rc) return rc;
    b.lane_cols = lane_cols;
    if (host_only) return FCOO_OK;
    try {
        rc = build_device(b, (hipStream_t)stream);
        if (!rc && single_pass) rc = setup_single_pass(b, (hipStream_t)stream);
    } catch (const std::bad_alloc &) {
        rc = fail(FCOO_ENOMEM, "device copies (host side)");
    }
    if (rc) { b.free_device(); return rc; }
    first_carries(b, (hipStream_t)stream);
    return FCOO_OK;
}

int fcoo_info(const fcoo_tensor *t, int mode, int op, fcoo_info_t *info)
{
    clear_error();
    if (!info) return fail(FCOO_EINVAL, "info is NULL");
    int rc;
    const Built *b = get_built(const_cast<fcoo_tensor *>(t), mode, op, false, &rc);
    if (!b) return rc;
    info->nnz = b->nnz;
    info->nseg = b->nseg;
    info->npart = b->npart;
    info->ntiles = b->ntiles;
    info->nfix = b->plan[0].nfix();
    info->nempty = (int64_t)b->empty_rows.size();
    info->bytes_format = b->format_bytes();
    info->bytes_device = b->device_bytes;
    info->threadlen = b->threadlen;
    info->tile_nnz = b->tile_nnz;
    info->order = t->order;
    info->on_device = b->on_device ? 1 : 0;
    info->xcd_blocks = b->nblk;
    info->block_mode = b->bmode;
    info->lane_cols = b->lane_cols;
    info->single_pass = b->sp ? 1 : 0;
    info->sp_gave_up = 0;
    if (b->sp && b->d_sp_err) {
        // reads the flag a bounded wait of the single-pass kernel sets (synchronous)
        int e = 0;
        FCOO_HIP(hipMemcpy(&e, b->d_sp_err, sizeof(int), hipMemcpyDeviceToHost));
        info->sp_gave_up = e != 0;
    }
    return FCOO_OK;
}

int fcoo_export(const fcoo_tensor *t, int mode, int op, int32_t *const *pidx, float *val,
                uint8_t *bf, uint32_t *sf, int32_t *seg, int32_t *tile_seg0, int32_t *perm)
{
    clear_error();
    int rc;
    const Built *b = get_built(const_cast<fcoo_tensor *>(t), mode, op, false, &rc);
    if (!b) return rc;
    if (!b->host_arrays) {
        // built on the GPU: the per-nonzero arrays live on the device only
        const int64_t Z = b->nnz;
        if (pidx)
            for (size_t q = 0; q < b->pmodes.size(); ++q)
                if (pidx[q]) FCOO_HIP(hipMemcpy(pidx[q], b->d_pidx[q], (size_t)Z * 4, hipMemcpyDeviceToHost));
        if (val) FCOO_HIP(hipMemcpy(val, b->d_val, (size_t)Z * 4, hipMemcpyDeviceToHost));
        if (bf) FCOO_HIP(hipMemcpy(bf, b->d_bf, (size_t)(Z + 7) / 8, hipMemcpyDeviceToHost));
        if (sf) FCOO_HIP(hipMemcpy(sf, b->d_sf, (size_t)((b->npart + 31) / 32) * 4, hipMemcpyDeviceToHost));
        if (perm) FCOO_HIP(hipMemcpy(perm, b->d_perm, (size_t)Z * 4, hipMemcpyDeviceToHost));
        if (seg) memcpy(seg, b->seg.data(), b->seg.size() * 4);
        if (tile_seg0) memcpy(tile_seg0, b->tile_seg0.data(), b->tile_seg0.size() * 4);
        return FCOO_OK;
    }
    if (pidx)
        for (size_t q = 0; q < b->pidx.size(); ++q)
            if (pidx[q]) memcpy(pidx[q], b->pidx[q].data(), b->pidx[q].size() * 4);
    if (val) memcpy(val, b->val.data(), b->val.size() * 4);
    if (bf) memcpy(bf, b->bf.data(), b->bf.size());
    if (sf) memcpy(sf, b->sf.data(), b->sf.size() * 4);
    if (seg) memcpy(seg, b->seg.data(), b->seg.size() * 4);
    if (tile_seg0) memcpy(tile_seg0, b->tile_seg0.data(), b->tile_seg0.size() * 4);
    if (perm) memcpy(perm, b->perm.data(), b->perm.size() * 4);
    return FCOO_OK;
}

void fcoo_destroy(fcoo_tensor *t)
{
    if (!t) return;
    for (auto &row : t->b)
        for (auto &b : row) b.free_device();
    for (auto &p : t->d_coo) if (p) (void)hipFree(p);
    if (t->d_coo_val) (void)hipFree(t->d_coo_val);
    t->ws.free_all();
    if (t->ev_dep) (void)hipEventDestroy(t->ev_dep);
    if (t->ev_solved) (void)hipEventDestroy(t->ev_solved);
    if (t->aux) (void)hipStreamDestroy(t->aux);
    delete t;
    pool_handles(-1);
}

// ---------------------------------------------------------------------------
// sparse operations: argument checks, then the HIP launchers
// ---------------------------------------------------------------------------

// Carries for the launch's tiles, p.plan.  They are those of the widest rows so far
// (carry_need), which no narrower launch replaces.
static int prep_carries(Built *b, TileProblem &p, hipStream_t s)
{
    const bool fits = 2 * p.plan->ntiles * (int64_t)p.R <= b->carry_cap;
    if (fits && p.R <= b->carry_width) return FCOO_OK;
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (fits && (hipStreamIsCapturing(s, &st) != hipSuccess || st != hipStreamCaptureStatusNone)) {
        (void)hipGetLastError();
        return FCOO_OK;
    }
    int rc = ensure_device_floats(&b->d_carry, &b->carry_cap, carry_need(*b, p.R), s);
    if (rc == FCOO_ENOMEM) {       // the format's tiles, which have the fewest carries
        (void)hipGetLastError();
        clear_error();
        p.plan = &b->plan[0];
        rc = ensure_device_floats(&b->d_carry, &b->carry_cap, 2 * p.plan->ntiles * (int64_t)p.R, s);
    }
    if (!rc) b->carry_width = std::max(b->carry_width, p.R);
    return rc;
}

// The tiles of a launch and its scratch: the carries, and with XCD blocks the
// partial output (nblk x rows x width floats) of the build.
static int prep_tiles(Built *b, TileProblem &p, bool resid, hipStream_t s)
{
    p.plan = p.keep_order ? &b->plan[0] : &pick_plan(*b, p.dtype, p.R, resid, p.kron);
    int rc = prep_carries(b, p, s);
    if (rc) return rc;
    p.carry = b->d_carry;
    if (b->nblk <= 1) return FCOO_OK;
    rc = ensure_device_floats(&b->d_bpart, &b->bpart_cap, (int64_t)b->nblk * b->rows * p.R, s);
    if (rc) return rc;
    p.bpart = b->d_bpart;
    return FCOO_OK;
}

int fcoo_spmttkrp(fcoo_tensor *t, int mode, const void *const *factors, int dtype, int R, float *M,
                  void *stream)
{
    clear_error();
    return spmttkrp(t, mode, factors, dtype, R, M, false, (hipStream_t)stream);
}

}  // extern "C"

int fcoo::spmttkrp(fcoo_tensor *t, int mode, const void *const *factors, int dtype, int R, float *M, bool keep_order,
                   hipStream_t s)
{
    int rc;
    Built *b = get_built(t, mode, FCOO_OP_MTTKRP, true, &rc);
    if (!b) return rc;
    rc = check_factors(t, mode, factors, dtype, R);
    if (rc) return rc;
    if (!M) return fail(FCOO_EINVAL, "M is NULL");
    TileProblem p{};
    p.b = b;
    for (size_t q = 0; q < b->pmodes.size(); ++q) p.fac[q] = factors[b->pmodes[q]];
    p.vals = b->d_val;
    p.dtype = dtype;
    p.R = R;
    p.out = M;
    p.keep_order = keep_order;
    if ((rc = prep_tiles(b, p, false, s))) return rc;
    if ((rc = prep_single_pass(b, p, s))) return rc;
    p.ev_before = t->ev_before;
    p.ev_after = t->ev_after;
    return launch_segmented(p, s, false);
}

extern "C" {

int fcoo_spttmc(fcoo_tensor *t, int mode, const void *const *factors, int dtype, const int *ranks,
                float *Y, void *stream)
{
    clear_error();
    int rc;
    Built *b = get_built(t, mode, FCOO_OP_MTTKRP, true, &rc);
    if (!b) return rc;
    if (!ranks) return fail(FCOO_EINVAL, "ranks is NULL");
    int64_t W = 1;
    for (int m = 0; m < t->order; ++m) {
        if (m == mode) continue;
        if (ranks[m] < 1 || ranks[m] > kMaxR)
            return fail(FCOO_EUNSUPPORTED, "ranks[%d] = %d outside [1, %d]", m, ranks[m], kMaxR);
        W *= ranks[m];
        if (W > kMaxKronWidth)
            return fail(FCOO_EUNSUPPORTED, "SpTTMc width (product of the ranks) above %d", kMaxKronWidth);
    }
    rc = check_factors(t, mode, factors, dtype, 1);
    if (rc) return rc;
    if (!Y) return fail(FCOO_EINVAL, "Y is NULL");
    hipStream_t s = (hipStream_t)stream;
    TileProblem p{};
    p.b = b;
    p.kron = b->pmodes.size() > 1;   // (a chain of one matrix is SpMTTKRP)
    for (size_t q = 0; q < b->pmodes.size(); ++q) {
        p.fac[q] = factors[b->pmodes[q]];
        p.kr[q] = ranks[b->pmodes[q]];
        p.fac_rows[q] = t->dims[b->pmodes[q]];
    }
    p.vals = b->d_val;
    p.dtype = dtype;
    p.R = (int)W;
    p.out = Y;
    if ((rc = prep_tiles(b, p, false, s))) return rc;
    if ((rc = prep_single_pass(b, p, s))) return rc;
    p.ev_before = t->ev_before;
    p.ev_after = t->ev_after;
    return launch_segmented(p, s, false);
}

int fcoo_spttm(fcoo_tensor *t, int mode, const void *U, int dtype, int R, float *Y, void *stream)
{
    clear_error();
    int rc;
    Built *b = get_built(t, mode, FCOO_OP_TTM, true, &rc);
    if (!b) return rc;
    if ((!U && b->nnz) || (!Y && b->nseg)) return fail(FCOO_EINVAL, "U or Y is NULL");
    if (dtype != FCOO_F32 && dtype != FCOO_BF16) return fail(FCOO_EUNSUPPORTED, "unknown dtype %d", dtype);
    if (R < 1 || R > kMaxR) return fail(FCOO_EUNSUPPORTED, "R = %d outside [1, %d]", R, kMaxR);
    hipStream_t s = (hipStream_t)stream;
    TileProblem p{};
    p.b = b;
    p.fac[0] = U;
    p.vals = b->d_val;
    p.dtype = dtype;
    p.R = R;
    p.out = Y;
    if ((rc = prep_tiles(b, p, false, s))) return rc;
    if ((rc = prep_single_pass(b, p, s))) return rc;
    p.ev_before = t->ev_before;
    p.ev_after = t->ev_after;
    return launch_segmented(p, s, false);
}

int fcoo_spmttkrp_values(fcoo_tensor *t, int mode, const float *g, const void *const *factors,
                         int dtype, int R, float *M, void *stream)
{
    clear_error();
    int rc;
    Built *b = get_built(t, mode, FCOO_OP_MTTKRP, true, &rc);
    if (!b) return rc;
    rc = check_factors(t, mode, factors, dtype, R);
    if (rc) return rc;
    if (!M || (!g && b->nnz)) return fail(FCOO_EINVAL, "M or g is NULL");
    hipStream_t s = (hipStream_t)stream;
    TileProblem p{};
    p.b = b;
    for (size_t q = 0; q < b->pmodes.size(); ++q) p.fac[q] = factors[b->pmodes[q]];
    p.vals = reinterpret_cast<const float *>(b->d_perm);
    p.gvals = g;
    // The tile kernel gathers the values with the rows.  A copy in stored order first
    // where it cannot, as they lie in the place of the result, and where rows have
    // several rank tiles, each of which would gather them again (1.6M nonzeros, order 2,
    // R = 200: 332 us, with the copy 264) -- unless there is no room for that one.
    const LaneShape sh = lane_shape(*b, dtype, R, false);
    const bool inside = g < M + t->dims[mode] * (int64_t)R && M < g + b->nnz;
    if (b->nnz && (inside || R > sh.lpn * sh.vw)) {
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        // (4 entries past the values, read but not used, as the build's streams have)
        const bool grows = b->gperm_cap < b->nnz + 4;
        if (grows && !inside && hipStreamIsCapturing(s, &st) != hipSuccess) st = hipStreamCaptureStatusActive;
        if (st == hipStreamCaptureStatusNone) rc = ensure_device_floats(&b->d_gperm, &b->gperm_cap, b->nnz + 4, s);
        if (st != hipStreamCaptureStatusNone || (rc == FCOO_ENOMEM && !inside)) {
            (void)hipGetLastError();
            clear_error();
        } else {
            if (rc || (rc = launch_permute_values(*b, g, b->d_gperm, s))) return rc;
            p.vals = b->d_gperm;
            p.gvals = nullptr;
        }
    }
    p.dtype = dtype;
    p.R = R;
    p.out = M;
    if ((rc = prep_tiles(b, p, false, s))) return rc;
    if ((rc = prep_single_pass(b, p, s))) return rc;
    p.ev_before = t->ev_before;
    p.ev_after = t->ev_after;
    return launch_segmented(p, s, false);
}

int fcoo_resid_spmttkrp(fcoo_tensor *t, int mode, const void *const *factors, int dtype, int R,
                        float *G, double *loss, void *stream)
{
    clear_error();
    int rc;
    Built *b = get_built(t, mode, FCOO_OP_MTTKRP, true, &rc);
    if (!b) return rc;
    rc = check_factors(t, -1, factors, dtype, R);
    if (rc) return rc;
    if (!G) return fail(FCOO_EINVAL, "G is NULL");
    hipStream_t s = (hipStream_t)stream;
    TileProblem p{};
    p.b = b;
    for (size_t q = 0; q < b->pmodes.size(); ++q) p.fac[q] = factors[b->pmodes[q]];
    p.vals = b->d_val;
    p.dtype = dtype;
    p.R = R;
    p.out = G;
    p.own = factors[mode];
    p.inv_nnz = b->nnz ? (float)(1.0 / (double)b->nnz) : 0.f;
    if ((rc = prep_tiles(b, p, true, s))) return rc;
    if ((rc = prep_single_pass(b, p, s))) return rc;
    if (loss) {
        // (for every rank's tiles, as the carries)
        if ((rc = ensure_device_doubles(&b->d_partial, &b->partial_cap, most_tiles(*b) + 1, s))) return rc;
        p.partial = b->d_partial;
        p.loss = loss;
        p.loss_scale = b->nnz ? 0.5 / (double)b->nnz : 0.0;
    }
    p.ev_before = t->ev_before;
    p.ev_after = t->ev_after;
    return launch_segmented(p, s, true);
}

int fcoo_set_tile_events(fcoo_tensor *t, void *before, void *after)
{
    clear_error();
    if (!t) return fail(FCOO_EINVAL, "null handle");
    if ((before == nullptr) != (after == nullptr)) return fail(FCOO_EINVAL, "give both events or neither");
    t->ev_before = (hipEvent_t)before;
    t->ev_after = (hipEvent_t)after;
    return FCOO_OK;
}

int fcoo_model_at_nnz(fcoo_tensor *t, const void *const *factors, int dtype, int R, float *xhat,
                      void *stream)
{
    clear_error();
    if (!t) return fail(FCOO_EINVAL, "null handle");
    int rc = check_factors(t, -1, factors, dtype, R);
    if (rc) return rc;
    if (!xhat && t->nnz) return fail(FCOO_EINVAL, "xhat is NULL");
    hipStream_t s = (hipStream_t)stream;
    if ((rc = upload_coo(t, s))) return rc;
    return launch_model(t, factors, dtype, R, xhat, s);
}

}  // extern "C"
