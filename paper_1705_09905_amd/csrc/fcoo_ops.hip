// Launch plans of the segmented F-COO operations; what follows their tile
// kernel (carry fix-up, empty rows, the residual's loss); the order of replaced
// values; the CP model at the nonzeros.
#include <algorithm>

#include "fcoo_internal.h"
#include "fcoo_seg_dispatch.h"

namespace fcoo {

namespace dev {

// What is left after the tile kernel, in one launch whose workgroups take one
// of four parts (each was a kernel of its own; one launch costs 3-5 us on the
// stream whatever it does, as much as a small tensor's tile kernel):
//   the first fblk   carry fix-up: entry (b, a, row) finishes the segment that
//                    tile a starts (its last open partial) and tile b closes
//                    (its first partial; b = ntiles is the end of the tensor),
//                    with tiles a+1 .. b-1 wholly inside it.  The nlong chains
//                    of more than kLongChain tiles come first, a workgroup
//                    each; of the others four share one.  (With 256 threads for
//                    every chain a slice of 1.3M nonzeros over 1300 tiles took
//                    40 us at R = 256: one thread a column);
//   the next sblk    the nshort chains with at most one tile between (nearly all
//                    where segments are short): a thread a column, about kFlat
//                    elements a workgroup.  (Four such chains a workgroup of
//                    1024: SpTTM, R = 16, 20M Zipf nonzeros, 19.5k chains, 26.5
//                    us; now 7);
//   the next zblk    rows of an MTTKRP result that no nonzero touches: 0;
//   the last one     the residual form's loss: fixed-order strided sums of the
//                    tiles' partials, then a tree; bitwise repeatable.
struct FinishArgs {
    const int32_t *fix;
    const float *ca, *cb;
    int64_t ntiles;
    const int32_t *empty;
    int64_t nempty;
    float *out;
    const double *partial;
    int64_t npartial;
    double scale;
    double *loss;
    int nfix, nlong, nshort, fblk, sblk, zblk, R;
    int per;                         // short chains per workgroup
    bool in_turn;                    // chains on 256 threads, 8 tiles' carries in turn (TileProblem::keep_order)
};

constexpr int kFinish = 1024;        // threads per workgroup
constexpr int kFlat = 1024;          // elements per workgroup of the short chains
constexpr int kZeroPer = 4096;       // elements per workgroup of the zero rows
constexpr int kChain = 16;           // carries in flight per thread along a chain

__global__ __launch_bounds__(kFinish) void finish_kernel(FinishArgs A)
{
    const int R = A.R;
    if ((int)blockIdx.x < A.fblk) {
        __shared__ float red_s[kFinish];
        const bool is_long = (int)blockIdx.x < A.nlong;
        const int n = is_long && !A.in_turn ? kFinish : 256;         // threads of a chain (those past n add nothing)
        const int part = is_long ? 0 : (int)threadIdx.x / 256, tid = (int)threadIdx.x - part * 256;
        const int e = is_long ? (int)blockIdx.x : A.nlong + ((int)blockIdx.x - A.nlong) * 4 + part;
        float *red = red_s + part * 256;
        const bool on = e < A.nfix - A.nshort;
        int tb = 0, ta = 0, row = 0;
        if (on) { tb = A.fix[3 * e]; ta = A.fix[3 * e + 1]; row = A.fix[3 * e + 2]; }
        // columns cw at a time (SpTTMc's rows may be wider than the threads)
        const int cw = R < n ? R : n;
        const int slots = n / cw, slot = tid / cw, c0 = tid - slot * cw;
        for (int cb = 0; cb < R; cb += cw) {
            const int c = cb + c0;
            float s = 0.f;
            if (on && slot < slots && c < R) {
                // long chains (a slice over hundreds of tiles): kChain loads in flight
                for (int t = ta + 1 + slot; t < tb; t += kChain * slots) {
                    float x[kChain];
#pragma unroll
                    for (int u = 0; u < kChain; ++u) {               // (past the chain's end its last: no load behind a branch)
                        const int tt = t + u * slots;
                        x[u] = A.ca[(int64_t)(tt < tb ? tt : tb - 1) * R + c];
                    }
#pragma unroll
                    for (int u = 0; u < kChain; ++u) x[u] = t + u * slots < tb ? x[u] : 0.f;
                    if (A.in_turn) {
#pragma unroll
                        for (int u = 0; u < kChain; ++u) s += x[u];
                        continue;
                    }
                    // (in pairs: a wide row has one slot, and a chain of a thousand
                    // tiles would be as many roundings in a row)
#pragma unroll
                    for (int o = kChain / 2; o >= 1; o >>= 1)
#pragma unroll
                        for (int u = 0; u < o; ++u) x[u] += x[u + o];
                    s += x[0];
                }
            }
            if (slots > 1) {
                red[tid] = s;
                __syncthreads();                                     // (R decides: the same in every part)
            }
            if (on && tid < cw && c < R) {
                float v = A.cb[(int64_t)ta * R + c];
                const int used = tb - ta - 1 < slots ? tb - ta - 1 : slots;   // the other slots' sums are 0
                if (slots > 1) {
                    if (is_long && !A.in_turn) {
                        // up to 1024 slots: eight sums (64 in a row, R = 16, had twice the error)
                        float x[8] = {};
                        for (int k = 0; k < used; k += 8)
#pragma unroll
                            for (int u = 0; u < 8; ++u) x[u] += k + u < used ? red[(k + u) * cw + tid] : 0.f;
                        v += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
                    } else {
                        for (int k = 0; k < used; ++k) v += red[k * cw + tid];
                    }
                } else {
                    v += s;
                }
                if (tb < A.ntiles) v += A.ca[(int64_t)tb * R + c];
                A.out[(int64_t)row * R + c] = v;
            }
        }
        return;
    }
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < A.fblk + A.sblk) {
        const int e0 = A.nfix - A.nshort + ((int)blockIdx.x - A.fblk) * A.per;
        const int n = (A.nfix - e0 < A.per ? A.nfix - e0 : A.per) * R;
#pragma unroll 4
        for (int i = tid; i < n; i += kFinish) {
            const int e = e0 + i / R, c = i % R;
            const int tb = A.fix[3 * e], ta = A.fix[3 * e + 1], row = A.fix[3 * e + 2];
            float v = A.cb[(int64_t)ta * R + c];
            if (tb - ta > 1) v += A.ca[(int64_t)(ta + 1) * R + c];
            if (tb < A.ntiles) v += A.ca[(int64_t)tb * R + c];
            A.out[(int64_t)row * R + c] = v;
        }
        return;
    }
    if ((int)blockIdx.x < A.fblk + A.sblk + A.zblk) {
        const int64_t n = A.nempty * R;
        for (int64_t i0 = ((int64_t)blockIdx.x - A.fblk - A.sblk) * kZeroPer; i0 < n; i0 += (int64_t)A.zblk * kZeroPer) {
#pragma unroll
            for (int u = 0; u < kZeroPer / kFinish; ++u) {
                const int64_t i = i0 + u * kFinish + tid;
                if (i < n) {
                    const int64_t r = i / R;
                    A.out[(int64_t)A.empty[r] * R + (i - r * R)] = 0.f;
                }
            }
        }
        return;
    }
    __shared__ double sh[kFinish];
    double s = 0.0;
    for (int64_t i = tid; i < A.npartial; i += kFinish * 8) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = i + u * kFinish < A.npartial ? A.partial[i + u * kFinish] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) s += x[u];
    }
    sh[tid] = s;
    __syncthreads();
    for (int o = kFinish / 2; o >= 1; o >>= 1) {
        if (tid < o) sh[tid] += sh[tid + o];
        __syncthreads();
    }
    if (tid == 0) A.loss[0] = sh[0] * A.scale;
}

__global__ __launch_bounds__(256) void permute_kernel(const int32_t *__restrict__ perm, const float *__restrict__ g,
                                                      int64_t n, float *__restrict__ out)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) out[i] = g[perm[i]];
}

// XCD blocks: out[i][c] = sum over blocks b of part[b][i][c], in block order.
__global__ __launch_bounds__(256) void reduce_blocks_kernel(const float *__restrict__ part, int nblk,
                                                            int64_t n, float *__restrict__ out)
{
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < n; e += (int64_t)gridDim.x * 256) {
        float v = part[e];
        for (int k = 1; k < nblk; ++k) v += part[(int64_t)k * n + e];
        out[e] = v;
    }
}

struct ModelArgs {
    const int32_t *idx[kMaxOrder];
    const void *fac[kMaxOrder];
    float *xhat;
    int64_t nnz;
    int order;
    int R;
    int per;                         // nonzeros a lane group takes in turn
};

// gathered nonzeros in flight per lane group, by the registers their rows take; half
// as many over more than one rank tile, whose gathers wait on each other (more waves
// then: 0.9M nonzeros, order 3, bfloat16, R = 200 149 us, now 143)
template <typename FT, int VW, int LPN, int NM, bool TILES>
constexpr int model_batch()
{
    constexpr int regs = (NM > 0 ? NM : kMaxOrder) * (int)(sizeof(Raw<FT, VW>) / 4), all = TILES ? 24 : 48;
    constexpr int fit = pow2_floor(all / regs > 0 ? all / regs : 1);
    return fit < LPN ? fit : LPN;
}

// xhat[e] = sum_r prod_m A_m[i_m(e), r]: a lane group of LPN lanes takes `per`
// consecutive nonzeros (LPN at most), one index a lane and mode (the next ones in
// flight meanwhile), each lane VW columns of a row (the last piece moved down to
// end at column R, rank tiles looped inside), the gathers of a batch of nonzeros
// back to back; lane j keeps the sum of the group's j-th.
// (One nonzero a group at a time, and one column a lane at ranks that are no
// multiple of the vector: 20M Zipf nonzeros, float32, R = 16 368 us, R = 10 3556;
// now 316 and 371.  The gathers of random rows bound it.)
template <typename FT, int VW, int LPN, int NM, bool TILES>
__global__ __launch_bounds__(256) void model_kernel(ModelArgs A)
{
    constexpr int NMM = NM > 0 ? NM : kMaxOrder;
    constexpr int BS = model_batch<FT, VW, LPN, NM, TILES>();         // nonzeros per batch
    constexpr uint32_t G = 256 / LPN;                          // lane groups of the workgroup
    const int lane = threadIdx.x & 63;
    const int j = lane % LPN;
    const int nm = NM > 0 ? NM : A.order, per = LPN == BS ? BS : A.per;
    const uint32_t nnz = (uint32_t)A.nnz, stride = gridDim.x * G * (uint32_t)per;
    const uint32_t wave0 = (blockIdx.x * G + (threadIdx.x & ~63u) / LPN) * (uint32_t)per;   // this wave's first nonzero
    int cur[NMM], nxt[NMM];
    auto load = [&](uint32_t e, int (&ix)[NMM]) {
        const uint32_t ec = e < nnz ? e : nnz - 1;
#pragma unroll
        for (int m = 0; m < NMM; ++m)
            if (m < nm) ix[m] = __builtin_nontemporal_load(A.idx[m] + ec);
    };
    const uint32_t off = (uint32_t)(lane / LPN * per + j);     // (lanes past `per` hold the next group's)
    load(wave0 + off, cur);
    for (uint32_t e0 = wave0; e0 < nnz; e0 += stride) {
        const uint32_t e = e0 + off;
        load(e + stride, nxt);
        float mine = 0.f;
        static_for<LPN / BS>([&](auto bc) {
            constexpr int B0 = decltype(bc)::value * BS;
            if (B0 >= per) return;
            float s[BS];
#pragma unroll
            for (int b = 0; b < BS; ++b) s[b] = 0.f;
            for (int t0 = 0; t0 < A.R; t0 += LPN * VW) {
                const int c0 = t0 + j * VW;
                const bool cval = c0 < A.R;
                const int c1 = c0 + VW <= A.R ? c0 : A.R - VW;
                const int col = c1, dup = cval ? c0 - c1 : VW;          // columns the lane before sums
                Raw<FT, VW> raw[BS][NMM];
                int ix[BS][NMM];
                static_for<BS>([&](auto sc) {
                    constexpr int S = decltype(sc)::value;
#pragma unroll
                    for (int m = 0; m < NMM; ++m)
                        if (m < nm) ix[S][m] = bcast_imm<LPN, B0 + S>(cur[m]);
                });
                if (cval) {                                             // (lanes past R read nothing and sum nothing)
#pragma unroll
                    for (int b = 0; b < BS; ++b)
#pragma unroll
                        for (int m = 0; m < NMM; ++m)
                            if (m < nm)
                                load_raw<FT, VW>(reinterpret_cast<const FT *>(A.fac[m]) + (int64_t)ix[b][m] * A.R + col, raw[b][m]);
                }
#pragma unroll
                for (int b = 0; b < BS; ++b) {
                    float p[VW];
                    to_float<FT, VW>(raw[b][0], p);
#pragma unroll
                    for (int m = 1; m < NMM; ++m) {
                        if (m >= nm) continue;
                        float x[VW];
                        to_float<FT, VW>(raw[b][m], x);
#pragma unroll
                        for (int k = 0; k < VW; ++k) p[k] *= x[k];
                    }
#pragma unroll
                    for (int k = 0; k < VW; ++k) s[b] += k >= dup ? p[k] : 0.f;
                }
            }
#pragma unroll
            for (int b = 0; b < BS; ++b) {
                const float x = group_sum<LPN>(s[b]);
                mine = j == B0 + b ? x : mine;
            }
        });
        if (j < per && e < nnz) A.xhat[e] = mine;
#pragma unroll
        for (int m = 0; m < NMM; ++m) cur[m] = nxt[m];
    }
}

}  // namespace dev

static int next_pow2(int x)
{
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

static int grid_for(int64_t work, int64_t per_block, int cap = 65535 * 8)
{
    int64_t g = (work + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

LaneShape lane_shape(const Built &b, int dtype, int R, bool resid, bool keep_order)
{
    // bfloat16 in 4-column (8-byte) lane chunks: twice the rows per gather
    // batch at 4 waves per SIMD, against 8-column chunks at 3 waves.  The
    // build's lane_cols picks (fcoo_autotune times both); by default 4
    // columns for SpMTTKRP with exactly two product modes (with three, the
    // batch per mode gets short and 8-column chunks won on the order-4 Zipf
    // tensor), and for SpTTM, whose 32 bytes of output per 8 columns would
    // leave in two halves (8 / 4 columns, 20M nonzeros, Zipf, us: R = 8 266 /
    // 185, 24 411 / 368, 64 509 / 449, uniform 1848 / 1102), but for rows of 16
    // (236 / 253, uniform 508 / 603) or 32 (301 / 320, uniform 730 / 681), and past
    // 64 columns only for whole rank tiles of 64 (128 1205 / 854, 256 2414 / 1704; 96
    // 703 / 815), and but for few tiles of the caller's size, whose waves are too few
    // to have half the nonzeros at a time (237k in tiles of 16384, R = 64 110 / 139)
    const int np = (int)b.pmodes.size();
    const bool half_ok = dtype == FCOO_BF16 && !resid && np <= 3 && R >= 4 &&
                         (R <= 64 || (b.op == FCOO_OP_TTM && R % 64 == 0));
    const bool few = b.own_tile && b.plan[0].ntiles < 128;
    LaneShape sh;
    if (keep_order) {
        // ranks no multiple of the vector (8, or 4 by what lane_cols and the modes say)
        // have their sums' order from a time of one column a lane
        const bool half = half_ok && R % 4 == 0 && (b.lane_cols == 4 || (b.lane_cols == 0 && np == 2));
        if (R % (half ? 4 : 8)) return LaneShape{1, 64, false};
    }
    sh.half = half_ok && (b.lane_cols == 4 || R < 8 ||
                          (b.lane_cols == 0 && (b.op == FCOO_OP_TTM ? R != 16 && R != 32 && !few : np == 2)));
    // columns per lane: the type's vector, or the widest piece a shorter row
    // holds.  A row need not be a multiple of it: its last piece ends at
    // column R and overlaps the one before.  (Such rows once ran one column
    // per lane, 64 lanes a nonzero: SpMTTKRP of 4M nonzeros, order 4, R = 25
    // took 323 us and takes 100; SpTTM of 300k, bfloat16 R = 10, 321 and 16)
    sh.vw = (dtype == FCOO_F32 || sh.half) ? 4 : 8;
    while (sh.vw > R) sh.vw >>= 1;
    sh.lpn = next_pow2((R + sh.vw - 1) / sh.vw);
    if (sh.lpn > 16) sh.lpn = 16;
    return sh;
}

int launch_segmented(const TileProblem &p, hipStream_t s, bool resid)
{
    const Built &b = *p.b;
    const Plan &pl = *p.plan;
    const int R = p.R;
    if (b.nnz > 0 && p.kron) {
        if (p.ev_before) FCOO_HIP(hipEventRecord(p.ev_before, s));
        const int rc = launch_ttmc(p, b.nblk > 1 ? p.bpart : p.out, s);
        if (rc) return rc;
        if (p.ev_after) FCOO_HIP(hipEventRecord(p.ev_after, s));
    } else if (b.nnz > 0) {
        SegLaunch L{};
        dev::SegArgs &a = L.args;
        const int np = (int)b.pmodes.size();
        for (int q = 0; q < np; ++q) {
            a.pidx[q] = b.d_pidx[q];
            a.fac[q] = p.fac[q];
        }
        a.vals = p.vals;
        a.gvals = p.gvals;
        a.hr = reinterpret_cast<const uint2 *>(b.d_hr);
        a.seg_row = b.op == FCOO_OP_MTTKRP ? b.d_seg_row : nullptr;
        a.out = b.nblk > 1 ? p.bpart : p.out;
        a.carry_a = p.carry;
        a.carry_b = p.carry + pl.ntiles * (int64_t)R;
        a.own = p.own;
        a.partial = p.partial;
        a.nnz = b.nnz;
        a.ntiles = pl.ntiles;
        a.R = R;
        a.np = np;
        a.tile_nnz = pl.T;
        a.nseg = (int)b.nseg;
        a.inv_nnz = p.inv_nnz;
        const LaneShape sh = lane_shape(b, p.dtype, R, resid, p.keep_order);
        L.vw = sh.vw;
        L.half = sh.half;
        L.lpn = sh.lpn;
        const int rt = sh.lpn * sh.vw;
        const int nrt = (R + rt - 1) / rt;
        const int most = p.dtype == FCOO_BF16 && R % 8 == 0 ? 128 : 64;
        if (resid && R > most)
            return fail(FCOO_EUNSUPPORTED, "fused residual needs R <= %d for this dtype (R = %d)", most, R);
        L.npt = np <= 3 ? np : 0;
        L.out = b.op == FCOO_OP_MTTKRP ? dev::kOutMap
              : R % 16 == 0 || R > sh.lpn * sh.vw ? dev::kOutStream : dev::kOutPlain;
        a.nblk = b.nblk;
        a.rows_own = (int)b.rows;
        if (p.sp_words) {
            a.sp_words = p.sp_words;
            a.sp_from = b.d_sp_from;
            a.sp_ticket = b.d_sp_ticket;
            a.sp_err = b.d_sp_err;
            a.sp_base = b.sp_tickets;
            a.sp_epoch = p.sp_epoch;
            a.sp_tail_from = b.sp_tail_from;
        }
        int64_t gx = pl.ntiles;
        if (b.nblk > 1) {
            int64_t most_tiles = 1;
            for (int k = 0; k <= b.nblk; ++k) a.blk_ts[k] = pl.blk_ts[k];
            for (int k = 0; k < b.nblk; ++k) most_tiles = std::max(most_tiles, pl.blk_ts[k + 1] - pl.blk_ts[k]);
            gx = (int64_t)kXcds * most_tiles;            // workgroup w: XCD w % 8, its block's tiles
        }
        L.grid = dim3((unsigned)gx, (unsigned)nrt, 1);
        hipError_t e;
        if (p.ev_before) FCOO_HIP(hipEventRecord(p.ev_before, s));
        const bool narrow = !L.half && sh.vw < (p.dtype == FCOO_F32 ? 4 : 8);
        if (narrow) e = p.dtype == FCOO_F32 ? seg_launch_f32_narrow(L, resid, s) : seg_launch_bf16_narrow(L, resid, s);
        else if (resid && R % sh.vw) e = p.dtype == FCOO_F32 ? seg_launch_f32_resid_ragged(L, s) : seg_launch_bf16_resid_ragged(L, s);
        else if (p.dtype == FCOO_F32) e = resid ? seg_launch_f32_resid(L, s) : seg_launch_f32(L, s);
        else if (L.half) e = seg_launch_bf16_half(L, s);
        else e = resid ? seg_launch_bf16_resid(L, s) : seg_launch_bf16(L, s);
        if (e != hipSuccess) return hip_fail(e, "tile kernel launch");
        if (p.sp_words)   // every workgroup of the launch takes one ticket
            const_cast<Built &>(b).sp_tickets += (unsigned long long)L.grid.x * L.grid.y;
        if (p.ev_after) FCOO_HIP(hipEventRecord(p.ev_after, s));
    }
    dev::FinishArgs f{};
    f.nfix = b.nnz > 0 && !p.sp_words ? (int)pl.nfix() : 0;
    f.nempty = (int64_t)b.empty_rows.size();
    f.nlong = f.nfix > 0 ? (int)pl.nlong : 0;
    f.nshort = f.nfix > 0 ? (int)pl.nshort : 0;
    f.fblk = f.nlong + (f.nfix - f.nlong - f.nshort + 3) / 4;
    // (2^20 workgroups at most, as of the zero rows: a grid has less than 2^32 threads)
    f.per = std::max(R < dev::kFlat ? dev::kFlat / R : 1, (f.nshort >> 20) + 1);
    f.sblk = f.nshort > 0 ? grid_for(f.nshort, f.per, INT32_MAX) : 0;
    f.zblk = f.nempty > 0 ? grid_for(f.nempty * R, dev::kZeroPer, 1 << 20) : 0;
    if (f.nfix + f.zblk > 0 || p.loss) {
        f.fix = b.d_fix + 3 * pl.fix_at;
        f.ca = p.carry;
        f.cb = p.carry + pl.ntiles * (int64_t)R;
        f.ntiles = pl.ntiles;
        f.empty = b.d_empty;
        f.out = b.nblk > 1 ? p.bpart : p.out;
        f.partial = p.partial;
        f.npartial = b.nnz > 0 ? pl.ntiles : 0;
        f.scale = p.loss_scale;
        f.loss = p.loss;
        f.R = R;
        f.in_turn = p.keep_order;
        hipLaunchKernelGGL(dev::finish_kernel, dim3((unsigned)(f.fblk + f.sblk + f.zblk + (p.loss ? 1 : 0))), dim3(dev::kFinish), 0,
                           s, f);
        FCOO_HIP(hipGetLastError());
    }
    if (b.nblk > 1) {
        const int64_t n = b.rows * (int64_t)R;
        hipLaunchKernelGGL(dev::reduce_blocks_kernel, dim3(grid_for(n, 256 * 4)), dim3(256), 0, s, p.bpart,
                           b.nblk, n, p.out);
        FCOO_HIP(hipGetLastError());
    }
    return FCOO_OK;
}

int launch_permute_values(const Built &b, const float *g, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(dev::permute_kernel, dim3(grid_for(b.nnz, 256 * 8)), dim3(256), 0, s, b.d_perm, g, b.nnz, out);
    FCOO_HIP(hipGetLastError());
    return FCOO_OK;
}

template <typename FT, int VW, int LPN, bool TILES = false>
static void model_nm(const dev::ModelArgs &a, hipStream_t s)
{
    // a lane group takes a batch of nonzeros, or several up to its lanes where that
    // leaves the chip 32k waves and more: with LPN each, few nonzeros or wide rows had
    // few waves in flight (13k nonzeros, order 5, R = 256 46 us, now 13)
    auto go = [&](auto nm) {
        constexpr int NM = decltype(nm)::value;
        dev::ModelArgs x = a;
        x.per = dev::model_batch<FT, VW, LPN, NM, TILES>();
        while (x.per < LPN && a.nnz / (x.per * (64 / LPN)) > 32768) x.per *= 2;
        hipLaunchKernelGGL((dev::model_kernel<FT, VW, LPN, NM, TILES>), dim3(grid_for(a.nnz, x.per * (256 / LPN), 256 * 32)),
                           dim3(256), 0, s, x);
    };
    switch (a.order) {
        case 2: go(std::integral_constant<int, 2>{}); break;
        case 3: go(std::integral_constant<int, 3>{}); break;
        case 4: go(std::integral_constant<int, 4>{}); break;
        case 5: go(std::integral_constant<int, 5>{}); break;
        default: go(std::integral_constant<int, 0>{}); break;
    }
}

template <typename FT>
static hipError_t model_go(const dev::ModelArgs &a, int vw, int lpn, hipStream_t s)
{
    constexpr int V = dev::Elem<FT>::VEC;
    if (vw == 1) model_nm<FT, 1, 1>(a, s);
    else if (vw == 2) lpn == 1 ? model_nm<FT, 2, 1>(a, s) : model_nm<FT, 2, 2>(a, s);
    else if (vw < V) lpn == 1 ? model_nm<FT, 4, 1>(a, s) : model_nm<FT, 4, 2>(a, s);
    else switch (lpn) {
        case 1: model_nm<FT, V, 1>(a, s); break;
        case 2: model_nm<FT, V, 2>(a, s); break;
        case 4: model_nm<FT, V, 4>(a, s); break;
        case 8: model_nm<FT, V, 8>(a, s); break;
        default: a.R > 16 * V ? model_nm<FT, V, 16, true>(a, s) : model_nm<FT, V, 16>(a, s); break;
    }
    return hipGetLastError();
}

int launch_model(const fcoo_tensor *t, const void *const *factors, int dtype, int R, float *xhat,
                 hipStream_t s)
{
    if (t->nnz == 0) return FCOO_OK;
    dev::ModelArgs a{};
    for (int m = 0; m < t->order; ++m) {
        a.idx[m] = t->d_coo[m];
        a.fac[m] = factors[m];
    }
    a.xhat = xhat;
    a.nnz = t->nnz;
    a.order = t->order;
    a.R = R;
    int vw = dtype == FCOO_F32 ? 4 : 8;
    while (vw > R) vw >>= 1;
    int lpn = next_pow2((R + vw - 1) / vw);
    if (lpn > 16) lpn = 16;
    hipError_t e = dtype == FCOO_F32 ? model_go<float>(a, vw, lpn, s) : model_go<dev::bf16raw>(a, vw, lpn, s);
    if (e != hipSuccess) return hip_fail(e, "model kernel launch");
    return FCOO_OK;
}

}  // namespace fcoo
