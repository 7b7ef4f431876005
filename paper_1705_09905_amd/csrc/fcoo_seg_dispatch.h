// Picks the tile-kernel instantiation for a (storage type, lane layout,
// number of product modes) and launches it.  Included by the instantiation
// units (seg_*.hip), which are compiled separately to keep build times short.
#pragma once

#include "fcoo_segscan.h"

namespace fcoo {

struct SegLaunch {
    dev::SegArgs args;
    int vw;          // columns per lane: 8 (bfloat16), 4, 2 or 1
    int lpn;         // lanes per nonzero: 1, 2, 4, 8 or 16 (64: one column each)
    int npt;         // product modes as a template value: 1, 2, 3, or 0 (runtime count)
    int out;         // dev::kOutMap (SpMTTKRP), kOutStream or kOutPlain (SpTTM)
    bool half;       // bfloat16 in 4-column (8-byte) lane chunks
    dim3 grid;
};

template <typename FT, int VW, int LPN, int NP, bool RESID, int OUT, bool RAGGED = false>
static hipError_t seg_go(const SegLaunch &L, hipStream_t s)
{
    hipLaunchKernelGGL((dev::seg_tile_kernel<FT, VW, LPN, NP, RESID, OUT, RAGGED>), L.grid, dim3(256), 0, s,
                       L.args);
    return hipGetLastError();
}

// SpTTM has one product mode and identity row map; SpMTTKRP maps rows.
template <typename FT, int VW, int LPN, int NP>
static hipError_t seg_ttm(const SegLaunch &L, hipStream_t s)
{
    if (L.out == dev::kOutStream) return seg_go<FT, VW, LPN, NP, false, dev::kOutStream>(L, s);
    return seg_go<FT, VW, LPN, NP, false, dev::kOutPlain>(L, s);
}

template <typename FT, int VW, int LPN, bool RESID, bool RAGGED = false>
static hipError_t seg_np(const SegLaunch &L, hipStream_t s)
{
    if constexpr (!RESID) {
        if (L.out != dev::kOutMap) return seg_ttm<FT, VW, LPN, 1>(L, s);
    }
    switch (L.npt) {
        case 1: return seg_go<FT, VW, LPN, 1, RESID, dev::kOutMap, RAGGED>(L, s);
        case 2: return seg_go<FT, VW, LPN, 2, RESID, dev::kOutMap, RAGGED>(L, s);
        case 3: return seg_go<FT, VW, LPN, 3, RESID, dev::kOutMap, RAGGED>(L, s);
        default: return seg_go<FT, VW, LPN, 0, RESID, dev::kOutMap, RAGGED>(L, s);
    }
}

template <typename FT, bool RESID, bool RAGGED = false>
static hipError_t seg_dispatch(const SegLaunch &L, hipStream_t s)
{
    constexpr int V = dev::Elem<FT>::VEC;
    switch (L.lpn) {
        case 1:
            if constexpr (!RAGGED) return seg_np<FT, V, 1, RESID>(L, s);   // (one lane a row: R is its vector)
            else return hipErrorInvalidValue;
        case 2: return seg_np<FT, V, 2, RESID, RAGGED>(L, s);
        case 4: return seg_np<FT, V, 4, RESID, RAGGED>(L, s);
        case 8: return seg_np<FT, V, 8, RESID, RAGGED>(L, s);
        default: return seg_np<FT, V, 16, RESID, RAGGED>(L, s);
    }
}

// Rows shorter than the vector of their type: pieces of 4 (bfloat16, R < 8),
// 2 (R = 2, 3) or 1 column (R = 1, the generic path with a runtime mode count).
template <typename FT, bool RESID>
static hipError_t seg_dispatch_narrow(const SegLaunch &L, hipStream_t s)
{
    if constexpr (sizeof(FT) == 2 && !RESID) {
        if (L.lpn == 64) {           // a wave per nonzero, one column a lane (SpMTTKRP, kept order of sums)
            if (L.npt == 2) return seg_go<FT, 1, 64, 2, false, dev::kOutMap>(L, s);
            if (L.npt == 3) return seg_go<FT, 1, 64, 3, false, dev::kOutMap>(L, s);
            return seg_go<FT, 1, 64, 0, false, dev::kOutMap>(L, s);
        }
    }
    if (L.vw == 1) {
        if constexpr (!RESID) {
            if (L.out != dev::kOutMap) return seg_ttm<FT, 1, 1, 0>(L, s);
        }
        return seg_go<FT, 1, 1, 0, RESID, dev::kOutMap>(L, s);
    }
    if (L.vw == 2) return L.lpn == 1 ? seg_np<FT, 2, 1, RESID>(L, s) : seg_np<FT, 2, 2, RESID, RESID>(L, s);
    if constexpr (sizeof(FT) == 2 && RESID) return L.lpn == 1 ? seg_np<FT, 4, 1, true>(L, s) : seg_np<FT, 4, 2, true, true>(L, s);
    // (with up to three product modes, and in SpTTM, such rows are seg_launch_bf16_half's)
    if constexpr (sizeof(FT) == 2 && !RESID)
        return L.lpn == 1 ? seg_go<FT, 4, 1, 0, false, dev::kOutMap>(L, s) : seg_go<FT, 4, 2, 0, false, dev::kOutMap>(L, s);
    return hipErrorInvalidValue;
}

// bfloat16 in 4-column lane chunks (SpMTTKRP with 1-3 product modes, or
// SpTTM): half the row bytes per lane, so twice the rows per gather batch.
template <typename FT, int LPN>
static hipError_t seg_np_half(const SegLaunch &L, hipStream_t s)
{
    if (L.out != dev::kOutMap) return seg_ttm<FT, 4, LPN, 1>(L, s);
    switch (L.npt) {
        case 1: return seg_go<FT, 4, LPN, 1, false, dev::kOutMap>(L, s);
        case 2: return seg_go<FT, 4, LPN, 2, false, dev::kOutMap>(L, s);
        default: return seg_go<FT, 4, LPN, 3, false, dev::kOutMap>(L, s);
    }
}

template <typename FT>
static hipError_t seg_dispatch_half(const SegLaunch &L, hipStream_t s)
{
    switch (L.lpn) {
        case 1: return seg_np_half<FT, 1>(L, s);
        case 2: return seg_np_half<FT, 2>(L, s);
        case 4: return seg_np_half<FT, 4>(L, s);
        case 8: return seg_np_half<FT, 8>(L, s);
        default: return seg_np_half<FT, 16>(L, s);
    }
}

hipError_t seg_launch_f32(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_bf16(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_bf16_half(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_f32_resid(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_bf16_resid(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_f32_resid_ragged(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_bf16_resid_ragged(const SegLaunch &L, hipStream_t s);
hipError_t seg_launch_f32_narrow(const SegLaunch &L, bool resid, hipStream_t s);
hipError_t seg_launch_bf16_narrow(const SegLaunch &L, bool resid, hipStream_t s);

}  // namespace fcoo
