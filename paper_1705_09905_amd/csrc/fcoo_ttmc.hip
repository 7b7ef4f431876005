// SpTTMc (Eq. 4, Table I third row) on the matrix cores: row i of the result
// is the sum over slice i's nonzeros of the outer product of its product
// modes' factor rows, Y_i = A^T B with A the nonzeros x RA matrix of
// val * (Kronecker row of all product modes but the last) and B the nonzeros
// x RB matrix of the last mode's rows -- a contraction over the nonzeros.
//
// A wave owns a tile of T consecutive nonzeros and BA x BB blocks of 16 x 16
// output columns.  One 16x16x4 float32 step contracts 4 nonzeros: lane (g, m),
// g = lane / 16, holds element m of the A row (and of the B row) of the step's
// nonzero g, so a nonzero's rows are read once, one element per lane, and the
// block's 256 sums take 4 registers a lane.  (The form before this one held
// 16 columns a lane and read 2 x 16 bytes a lane for every nonzero, four times
// the bytes through the texture path, which bounded it: 10M nonzeros, Zipf(1.1),
// R = 16 a mode took 255 us.)
//
// Stream: 64 nonzeros a load, lane (g, m) taking nonzero 4 m + g, so step s of the
// 16 has nonzeros 4 s .. 4 s + 3, each in lane s of its row of 16: a row broadcast
// (DPP), folded into the address add.  The rows of the next sub-chunk are in flight while one is contracted.
// Nonzeros outside the segment at hand are zeroed in both operands (so that an
// infinity in one segment's row leaves the others alone).
//
// A segment closed inside the tile is written directly; the tile's first and
// last partials go to carry_a / carry_b, and finish_kernel sums the chains.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "fcoo_device.h"
#include "fcoo_internal.h"

namespace fcoo {
namespace dev {

typedef float floatx4 __attribute__((ext_vector_type(4)));

struct TtmcArgs {
    const int32_t *pidx[kMaxOrder];
    const void *fac[kMaxOrder];
    const float *vals;
    const uint2 *hr;                 // per 32 nonzeros: (segment heads, heads before), padded
    const int32_t *seg_row;
    float *out;                      // rows of W = RA * RB floats
    float *carry_a, *carry_b;        // ntiles x W
    int64_t ntiles;
    int64_t blk_ts[9];
    uint32_t nnz;
    int T;
    int np;                          // product modes (>= 2)
    int RA, RB;
    int kr[kMaxOrder];
    int nblk;
    int nyb;                         // column tiles along RB (blockIdx.y = ya * nyb + yb)
};

// lane SRC of each row of 16 lanes
template <int SRC>
__device__ __forceinline__ int row_bcast(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, 0x150 + SRC, 0xF, 0xF, true);   // ROW_NEWBCAST
}
template <int SRC>
__device__ __forceinline__ float row_bcast(float x)
{
    return __int_as_float(row_bcast<SRC>(__float_as_int(x)));
}

// scalar loads of what the whole wave shares (written by earlier launches only):
// they wait on a counter of their own, not behind the gathers in flight
template <typename T>
__device__ __forceinline__ T load_uniform(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

template <int N, int I = 0, class F>
__device__ __forceinline__ void unroll(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<N, I + 1>(f);
    }
}

// the register is loaded from here on: a use further down waits for nothing
__device__ __forceinline__ void loaded(float &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void loaded(uint32_t &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void loaded(float2 &x) { loaded(x.x), loaded(x.y); }
__device__ __forceinline__ void loaded(uint2 &x) { loaded(x.x), loaded(x.y); }
__device__ __forceinline__ void loaded(float4 &x) { loaded(x.x), loaded(x.y), loaded(x.z), loaded(x.w); }

// NA: product modes of the A side (1, 2 or 0: runtime, np - 1).  VB: columns of the B
// side that a lane holds next to each other, one of each of VB blocks (BB where it
// divides RB, else 1): its element of a row is one load and of a result row one
// store (RA = 5, RB = 40, bfloat16, 3.9M nonzeros, 194 us with four loads of one, now 165).
// WIDE: a factor of 4 GiB or more (64-bit row offsets instead of a 32-bit one on the base)
template <typename FT, int BA, int BB, int NA, int VB = 1, bool WIDE = false>
__global__ __launch_bounds__(256, (BA * BB > 1 ? 2 : 4)) void ttmc_kernel(TtmcArgs A)
{
    constexpr int NAM = NA > 0 ? NA : kMaxOrder - 1;
    constexpr int NS = BA + BB + (NAM - 1) * BA > 4 ? 4 : 8;   // steps per sub-chunk
    constexpr int SUB = 4 * NS;                                // nonzeros per sub-chunk
    constexpr int NH = 64 / SUB;                               // sub-chunks per 64 nonzeros
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = lane >> 4, m = lane & 15;
    int64_t tile = (int64_t)blockIdx.x * 4 + w, tend = A.ntiles;
    if (A.nblk > 1) {
        const int x = (int)(blockIdx.x % kXcds);
        tile = A.blk_ts[x] + (int64_t)(blockIdx.x / kXcds) * 4 + w;
        tend = A.blk_ts[x + 1];
    }
    if (tile >= tend) return;                                  // (no barriers below)
    const int na = NA > 0 ? NA : A.np - 1;
    const int ya = (int)blockIdx.y / A.nyb, yb = (int)blockIdx.y % A.nyb;
    const int W = A.RA * A.RB;

    // this lane's element of each A-side mode's row and of the last mode's row;
    // elements past the ranks read element 0 and are never stored
    int pa0[BA][NAM];
    constexpr int NVB = BB / VB;                               // column b of lane m: (b / VB, VB m + b % VB)
    int pb0[NVB];
#pragma unroll
    for (int a = 0; a < BA; ++a) {
        const int p = (ya * BA + a) * 16 + m;
        int rem = p < A.RA ? p : 0;
#pragma unroll
        for (int q = NAM - 1; q >= 0; --q) {
            if (q >= na) { pa0[a][q] = 0; continue; }
            pa0[a][q] = (NA == 1 ? rem : rem % A.kr[q]) * (int)sizeof(FT);
            if (NA != 1) rem /= A.kr[q];
        }
    }
#pragma unroll
    for (int b = 0; b < NVB; ++b) {
        const int p = (yb * BB + b) * 16 + m * VB;
        pb0[b] = (p < A.RB ? p : 0) * (int)sizeof(FT);
    }

    const uint32_t s0 = (uint32_t)tile * (uint32_t)A.T;
    const uint32_t s1 = A.nnz - s0 < (uint32_t)A.T ? A.nnz : s0 + (uint32_t)A.T;

    // the sums in two levels, acc over 64 nonzeros at most and tot over those, so
    // that no chain of roundings is longer than 64 + T / 64 (one level had 1.8
    // times the former kernel's error against float64; two have less than it)
    floatx4 acc[BA][BB], tot[BA][BB];
    auto clear = [](floatx4 (&x)[BA][BB]) {
#pragma unroll
        for (int a = 0; a < BA; ++a)
#pragma unroll
            for (int b = 0; b < BB; ++b) x[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    };
    auto add_up = [&]() {
#pragma unroll
        for (int a = 0; a < BA; ++a)
#pragma unroll
            for (int b = 0; b < BB; ++b) tot[a][b] += acc[a][b];
        clear(acc);
    };
    clear(acc);
    clear(tot);
    // register v of lane (g, m) holds column (16 a + 4 g + v, 16 b + m) of the block (VB = 1)
    auto store = [&](float *rowp) {
#pragma unroll
        for (int a = 0; a < BA; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int pa = (ya * BA + a) * 16 + 4 * g + v;
                if (pa >= A.RA) continue;
#pragma unroll
                for (int b = 0; b < NVB; ++b) {
                    const int pb = (yb * BB + b) * 16 + m * VB;
                    float x[VB];
#pragma unroll
                    for (int k = 0; k < VB; ++k) x[k] = tot[a][b * VB + k][v];
                    if (pb < A.RB) store_row<VB>(rowp + (pa * A.RB + pb), x);
                }
            }
    };

    // segment open at the tile's start; tiles start at multiples of 64
    int seg = (int)load_uniform(&A.hr[s0 >> 5].y) - 1;
    bool have = false;
    // the output row of the first segment that is closed here, then of the next one,
    // read a segment ahead
    int next_row = load_uniform(A.seg_row + (seg + 1));

    // 64 nonzeros of the stream: row indices (or byte offsets), values
    struct Stream {
        int ix[NAM + 1];
        float v;
    };
    const int lpos = 4 * m + g;
    auto load_stream = [&](uint32_t base, Stream &st) {
        const uint32_t e0 = base + (uint32_t)lpos;
        const uint32_t e = e0 < A.nnz ? e0 : A.nnz;            // the streams' padding past Z
#pragma unroll
        for (int q = 0; q < NAM; ++q)
            if (q < na) st.ix[q] = __builtin_nontemporal_load(A.pidx[q] + e);
        st.ix[NAM] = __builtin_nontemporal_load(A.pidx[na] + e);
        st.v = __builtin_nontemporal_load(A.vals + e);
    };
    // row indices to byte offsets
    auto to_offsets = [&](Stream &st) {
        if constexpr (WIDE) return;
#pragma unroll
        for (int q = 0; q < NAM; ++q)
            if (q < na) st.ix[q] = (int)((uint32_t)st.ix[q] * (uint32_t)(A.kr[q] * (int)sizeof(FT)));
        st.ix[NAM] = (int)((uint32_t)st.ix[NAM] * (uint32_t)(A.RB * (int)sizeof(FT)));
    };
    struct Rows {
        Raw<FT, 1> a[NS][BA][NAM];
        Raw<FT, VB> b[NS][NVB];
    };
    auto gather = [&](const Stream &st, auto hc, Rows &r) {
        constexpr int H = decltype(hc)::value;
        auto row = [&](int q, int x, int col) -> const FT * {
            const char *f = reinterpret_cast<const char *>(A.fac[q]);
            if constexpr (WIDE) f += (uint64_t)(uint32_t)x * (uint64_t)(uint32_t)(A.kr[q] * (int)sizeof(FT)) + (uint32_t)col;
            else f += (uint32_t)x + (uint32_t)col;
            return reinterpret_cast<const FT *>(f);
        };
        unroll<NS>([&](auto sc) {
            constexpr int S = decltype(sc)::value;
#pragma unroll
            for (int q = 0; q < NAM; ++q) {
                if (q >= na) continue;
                const int x = row_bcast<H * NS + S>(st.ix[q]);
#pragma unroll
                for (int a = 0; a < BA; ++a) load_raw<FT, 1>(row(q, x, pa0[a][q]), r.a[S][a][q]);
            }
            const int x = row_bcast<H * NS + S>(st.ix[NAM]);
#pragma unroll
            for (int b = 0; b < NVB; ++b) load_raw<FT, VB>(row(na, x, pb0[b]), r.b[S][b]);
        });
    };
    auto contract = [&](const Rows &r, int S, float v, bool act) {
        float av[BA], bv[BB];
#pragma unroll
        for (int a = 0; a < BA; ++a) {
            float x = v;
#pragma unroll
            for (int q = 0; q < NAM; ++q)
                if (q < na) {
                    float f[1];
                    to_float<FT, 1>(r.a[S][a][q], f);
                    x *= f[0];
                }
            av[a] = act ? x : 0.f;
        }
#pragma unroll
        for (int b = 0; b < NVB; ++b) {
            float f[VB];
            to_float<FT, VB>(r.b[S][b], f);
#pragma unroll
            for (int k = 0; k < VB; ++k) bv[b * VB + k] = act ? f[k] : 0.f;
        }
#pragma unroll
        for (int a = 0; a < BA; ++a)
#pragma unroll
            for (int b = 0; b < BB; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
    };
    // one sub-chunk: heads `hm` among its first n nonzeros
    auto consume = [&](Rows &r, auto hc, float vreg, uint32_t hm, int n) {
        constexpr int H = decltype(hc)::value;
        if (hm == 0u && n >= SUB) {
            unroll<NS>([&](auto sc) {
                constexpr int S = decltype(sc)::value;
                contract(r, S, row_bcast<H * NS + S>(vreg), true);
            });
            return;
        }
        if constexpr (NA > 0) {
            // the sub-chunk's rows are waited for here: inside the loop that wait would
            // be for the stores of the segments before, too (a counter has both in order)
#pragma unroll
            for (int S = 0; S < NS; ++S) {
#pragma unroll
                for (int a = 0; a < BA; ++a)
#pragma unroll
                    for (int q = 0; q < NAM; ++q) loaded(r.a[S][a][q].v);
#pragma unroll
                for (int b = 0; b < NVB; ++b) loaded(r.b[S][b].v);
            }
        }
        // step by step, and in a step segment by segment: rows of a few nonzeros meet a
        // head every other step, and looking for the steps of each segment among the
        // sub-chunk's cost more than its products
        unroll<NS>([&](auto sc) {
            constexpr int S = decltype(sc)::value;
            if (n <= 4 * S) return;
            const uint32_t live = n - 4 * S >= 4 ? 15u : (1u << (n - 4 * S)) - 1u;
            const float v = row_bcast<H * NS + S>(vreg);
            uint32_t heads = (hm >> (4 * S)) & live;
            uint32_t mask = live & ((heads & (0u - heads)) - 1u);     // up to the first head (all, with none)
            if (mask) contract(r, S, v, (mask >> g) & 1u);
            while (heads) {
                // a segment starts: the one before it is complete, or is the tile's first partial
                add_up();
                store(have ? A.out + (int64_t)next_row * W : A.carry_a + tile * W);
                if (have) next_row = load_uniform(A.seg_row + seg + 1);
                have = true;
                ++seg;
                clear(tot);
                const uint32_t rest = heads & (heads - 1u);
                mask = live & ((rest & (0u - rest)) - 1u) & ~((heads & (0u - heads)) - 1u);
                contract(r, S, v, (mask >> g) & 1u);
                heads = rest;
            }
        });
    };

    Stream cur, nxt;
    Rows buf[2];
    load_stream(s0, cur);
    to_offsets(cur);
    gather(cur, std::integral_constant<int, 0>{}, buf[0]);
    for (uint32_t base = s0; base < s1; base += 64) {
        const uint64_t hm = (uint64_t)load_uniform(&A.hr[base >> 5].x) |
                            ((uint64_t)load_uniform(&A.hr[(base >> 5) + 1].x) << 32);
        const int n = (int)(s1 - base);
        const bool more = base + 64 < s1;
        if (more) load_stream(base + 64, nxt);
        const float v = cur.v;
        unroll<NH>([&](auto hc) {
            constexpr int H = decltype(hc)::value;
            if constexpr (H + 1 < NH) {
                gather(cur, std::integral_constant<int, H + 1>{}, buf[(H + 1) & 1]);
            } else if (more) {
                cur = nxt;
                to_offsets(cur);
                gather(cur, std::integral_constant<int, 0>{}, buf[0]);
            }
            if (n > H * SUB)
                consume(buf[H & 1], hc, v, (uint32_t)((hm >> (H * SUB)) & ((SUB >= 32) ? 0xFFFFFFFFull : ((1ull << SUB) - 1ull))),
                        n - H * SUB);
        });
        add_up();
    }
    // the tile's carries: (sum before its first head, sum from its last one on)
    store(A.carry_b + tile * W);
    if (!have) store(A.carry_a + tile * W);
}

}  // namespace dev

namespace {

template <typename FT, int BA, int BB, int VB>
void ttmc_na(const dev::TtmcArgs &a, dim3 grid, hipStream_t s)
{
    if (a.np == 2) hipLaunchKernelGGL((dev::ttmc_kernel<FT, BA, BB, 1, VB>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((dev::ttmc_kernel<FT, BA, BB, 2, VB>), grid, dim3(256), 0, s, a);
}

template <typename FT, int BA, int BB>
void ttmc_vb(const dev::TtmcArgs &a, dim3 grid, hipStream_t s)
{
    if (a.RB % BB == 0) ttmc_na<FT, BA, BB, BB>(a, grid, s);
    else ttmc_na<FT, BA, BB, 1>(a, grid, s);
}

template <typename FT>
void ttmc_shape(const dev::TtmcArgs &a, bool wide, int ba, int bb, dim3 grid, hipStream_t s)
{
    if (wide) hipLaunchKernelGGL((dev::ttmc_kernel<FT, 1, 1, 0, 1, true>), grid, dim3(256), 0, s, a);
    else if (a.np > 3) hipLaunchKernelGGL((dev::ttmc_kernel<FT, 1, 1, 0>), grid, dim3(256), 0, s, a);
    else if (ba == 1 && bb == 1) ttmc_na<FT, 1, 1, 1>(a, grid, s);
    else if (ba == 1 && bb == 2) ttmc_vb<FT, 1, 2>(a, grid, s);
    else if (ba == 2 && bb == 1) ttmc_na<FT, 2, 1, 1>(a, grid, s);
    else if (ba == 2 && bb == 2) ttmc_vb<FT, 2, 2>(a, grid, s);
    else ttmc_vb<FT, 1, 4>(a, grid, s);
}

}  // namespace

// The tile kernel of SpTTMc: out and carries as the other tile kernels' (rows of
// p.R = W floats), two product modes or more.
int launch_ttmc(const TileProblem &p, float *out, hipStream_t s)
{
    const Built &b = *p.b;
    const Plan &pl = *p.plan;
    const int np = (int)b.pmodes.size();
    dev::TtmcArgs a{};
    int RA = 1;
    bool wide = false;
    for (int q = 0; q < np; ++q) {
        a.pidx[q] = b.d_pidx[q];
        a.fac[q] = p.fac[q];
        a.kr[q] = p.kr[q];
        if (q + 1 < np) RA *= p.kr[q];
        wide |= p.fac_rows[q] * p.kr[q] * (p.dtype == FCOO_F32 ? 4 : 2) >= ((int64_t)1 << 32);
    }
    a.vals = p.vals;
    a.hr = reinterpret_cast<const uint2 *>(b.d_hr);
    a.seg_row = b.d_seg_row;
    a.out = out;
    a.carry_a = p.carry;
    a.carry_b = p.carry + pl.ntiles * (int64_t)p.R;
    a.ntiles = pl.ntiles;
    a.nnz = (uint32_t)b.nnz;
    a.T = pl.T;
    a.np = np;
    a.RA = RA;
    a.RB = p.kr[np - 1];
    a.nblk = b.nblk;
    // blocks of 16 x 16 columns per wave: all of a small result, else 2 x 2 (a row
    // element then feeds two products; 4 x 4 blocks spill) or 1 x 4; one with
    // four product modes or more, whose row products hold the registers
    const int nA = (RA + 15) / 16, nB = (a.RB + 15) / 16;
    int ba = nA == 1 ? 1 : 2, bb = nB == 1 ? 1 : nB == 2 || ba == 2 ? 2 : 4;
    if (wide || np > 3) ba = bb = 1;
    a.nyb = (nB + bb - 1) / bb;
    int64_t gx = (pl.ntiles + 3) / 4;
    if (b.nblk > 1) {
        int64_t most = 0;
        for (int k = 0; k <= b.nblk; ++k) a.blk_ts[k] = pl.blk_ts[k];
        for (int k = 0; k < b.nblk; ++k) most = std::max(most, pl.blk_ts[k + 1] - pl.blk_ts[k]);
        gx = (int64_t)kXcds * ((most + 3) / 4);
        if (gx < 1) gx = 1;
    }
    const dim3 grid((unsigned)gx, (unsigned)(((nA + ba - 1) / ba) * a.nyb), 1);
    if (p.dtype == FCOO_F32) ttmc_shape<float>(a, wide, ba, bb, grid, s);
    else ttmc_shape<dev::bf16raw>(a, wide, ba, bb, grid, s);
    FCOO_HIP(hipGetLastError());
    return FCOO_OK;
}

}  // namespace fcoo
