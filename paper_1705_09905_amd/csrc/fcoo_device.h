// Device-side building blocks for gfx950 (CDNA4, wave64): segment-head
// decoding, cross-lane moves inside a lane group, row loads of float32 /
// bfloat16 factor matrices.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fcoo {
namespace dev {

// ----- segment heads --------------------------------------------------------
// The kernels read the bf bits (Sec. IV-B) decoded: per 32 nonzeros one pair
// (.x: bit i set iff nonzero 32 w + i starts a segment, .y: heads before
// nonzero 32 w), with two zero pairs of padding, so the words of any 64
// nonzeros that start below Z can be read.  A run's first segment ordinal then
// takes one load and a popcount where it is wanted, not a count over the tile.

// Heads of the nonzeros from bit `sh` of the first word on (the third word only
// counts past 32 - sh + 32), of which the first n <= 64 are kept.
__device__ __forceinline__ uint64_t head_bits(uint32_t h0, uint32_t h1, uint32_t h2, int sh, int n)
{
    const uint64_t lo = (uint64_t)h0 | ((uint64_t)h1 << 32);
    const uint64_t hm = sh ? ((lo >> sh) | ((uint64_t)h2 << (64 - sh))) : lo;
    return n >= 64 ? hm : (hm & ((1ull << n) - 1ull));
}

// Heads before nonzero 32 w + sh, from its pair.
__device__ __forceinline__ int heads_before(uint32_t h0, uint32_t rank, int sh)
{
    return (int)rank + __popc(h0 & ((1u << sh) - 1u));
}

// ----- lane-group moves -------------------------------------------------------
// A lane group is LPN consecutive lanes (LPN a power of two) working on one
// nonzero.  Within a row of 16 lanes data moves by DPP, a modifier of an
// ordinary vector instruction; ds_swizzle, which did it before, goes through the
// LDS queue and its wait (the float32 residual, R = 64, six to seven moves a step:
// 300k nonzeros 26.3 -> 21.3 us, 5M 138 -> 122, 20M 439 -> 422).

template <int CTRL, int BANKS = 0xF>
__device__ __forceinline__ int dpp(int old, int x)
{
    return __builtin_amdgcn_update_dpp(old, x, CTRL, 0xF, BANKS, false);
}

// Broadcast with a compile-time source lane of the group (LDSQ: by ds_swizzle).
template <int LPN, int SRC, bool LDSQ = false>
__device__ __forceinline__ int bcast_imm(int x)
{
    if constexpr (LPN == 1) {
        return x;
    } else if constexpr (LDSQ && LPN <= 16) {
        return __builtin_amdgcn_ds_swizzle(x, (0x1F & ~(LPN - 1)) | (SRC << 5));
    } else if constexpr (LPN == 2) {
        return dpp<SRC | SRC << 2 | (2 + SRC) << 4 | (2 + SRC) << 6>(x, x);      // quad_perm
    } else if constexpr (LPN == 4) {
        return dpp<SRC * 0x55>(x, x);                                            // quad_perm
    } else if constexpr (LPN == 8) {
        return dpp<0x158 + SRC, 0xC>(dpp<0x150 + SRC>(x, x), x);                 // row_newbcast, upper half its own
    } else if constexpr (LPN == 16) {
        return dpp<0x150 + SRC>(x, x);                                           // row_newbcast
    } else {
        static_assert(LPN == 64, "lanes of a group");
        return __builtin_amdgcn_readlane(x, SRC);
    }
}

template <int LPN, int SRC, bool LDSQ = false>
__device__ __forceinline__ float bcast_imm_f(float x)
{
    return __int_as_float(bcast_imm<LPN, SRC, LDSQ>(__float_as_int(x)));
}

template <int CTRL>
__device__ __forceinline__ float add_dpp(float v)
{
    return v + __int_as_float(dpp<CTRL>(__float_as_int(v), __float_as_int(v)));
}

// Butterfly sum over the LPN lanes of a group (16 at most).
template <int LPN>
__device__ __forceinline__ float group_sum(float v)
{
    if constexpr (LPN >= 2) v = add_dpp<0xB1>(v);                                // quad_perm: lane ^ 1
    if constexpr (LPN >= 4) v = add_dpp<0x4E>(v);                                // quad_perm: lane ^ 2
    if constexpr (LPN >= 8) v = add_dpp<0x141>(v);                               // row_half_mirror: the other quad
    if constexpr (LPN >= 16) v = add_dpp<0x140>(v);                              // row_mirror: the other half
    static_assert(LPN <= 16, "a row of lanes");
    return v;
}

// ----- factor rows ------------------------------------------------------------
// Factor storage: float32, or bfloat16 kept as its raw 16 bits (the upper
// half of a float32).  VW elements per lane, one load each.  A row starts at
// any multiple of its element's size (R is not rounded up to VW), so the
// vector types are declared with the element's alignment: global loads and
// stores take it as it is, in one instruction.

struct bf16raw { uint16_t x; };

template <typename FT> struct Elem;
template <> struct Elem<float> { static constexpr int VEC = 4; };
template <> struct Elem<bf16raw> { static constexpr int VEC = 8; };

__device__ __forceinline__ float bf16_to_f32(uint32_t bits16) { return __uint_as_float(bits16 << 16); }

typedef float float4e __attribute__((ext_vector_type(4), aligned(4)));
typedef float float2e __attribute__((ext_vector_type(2), aligned(4)));
typedef uint32_t uint4e __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t uint2e __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t uint1e __attribute__((aligned(2)));

// A row chunk as loaded (raw registers), converted to float32 when used.
template <typename FT, int VW> struct Raw;
template <> struct Raw<float, 4> { float4 v; };
template <> struct Raw<bf16raw, 8> { uint4 v; };
template <> struct Raw<float, 2> { float2 v; };
template <> struct Raw<float, 1> { float v; };
template <> struct Raw<bf16raw, 1> { uint32_t v; };
template <> struct Raw<bf16raw, 2> { uint32_t v; };   // two consecutive bfloat16
template <> struct Raw<bf16raw, 4> { uint2 v; };      // four consecutive bfloat16 (8-byte loads)

template <typename FT, int VW>
__device__ __forceinline__ void load_raw(const FT *__restrict__ p, Raw<FT, VW> &r)
{
    if constexpr (sizeof(FT) == 4 && VW == 4) {
        const float4e x = *reinterpret_cast<const float4e *>(p);
        r.v = make_float4(x.x, x.y, x.z, x.w);
    } else if constexpr (sizeof(FT) == 4 && VW == 2) {
        const float2e x = *reinterpret_cast<const float2e *>(p);
        r.v = make_float2(x.x, x.y);
    } else if constexpr (sizeof(FT) == 2 && VW == 8) {
        const uint4e x = *reinterpret_cast<const uint4e *>(p);
        r.v = make_uint4(x.x, x.y, x.z, x.w);
    } else if constexpr (sizeof(FT) == 2 && VW == 4) {
        const uint2e x = *reinterpret_cast<const uint2e *>(p);
        r.v = make_uint2(x.x, x.y);
    } else if constexpr (sizeof(FT) == 2 && VW == 2) {
        r.v = *reinterpret_cast<const uint1e *>(p);
    } else if constexpr (sizeof(FT) == 4 && VW == 1) {
        r.v = *reinterpret_cast<const float *>(p);
    } else {
        r.v = (uint32_t)(*reinterpret_cast<const uint16_t *>(p));
    }
}

template <typename FT, int VW>
__device__ __forceinline__ void set_one(Raw<FT, VW> &r)
{
    if constexpr (sizeof(FT) == 4 && VW == 4) r.v = make_float4(1.f, 1.f, 1.f, 1.f);
    else if constexpr (sizeof(FT) == 2 && VW == 8) r.v = make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u);
    else if constexpr (sizeof(FT) == 4 && VW == 2) r.v = make_float2(1.f, 1.f);
    else if constexpr (sizeof(FT) == 4 && VW == 1) r.v = 1.f;
    else if constexpr (sizeof(FT) == 2 && VW == 2) r.v = 0x3F803F80u;
    else if constexpr (sizeof(FT) == 2 && VW == 4) r.v = make_uint2(0x3F803F80u, 0x3F803F80u);
    else r.v = 0x3F80u;
}

template <typename FT, int VW>
__device__ __forceinline__ void to_float(const Raw<FT, VW> &r, float (&out)[VW])
{
    if constexpr (sizeof(FT) == 4 && VW == 4) {
        out[0] = r.v.x; out[1] = r.v.y; out[2] = r.v.z; out[3] = r.v.w;
    } else if constexpr (sizeof(FT) == 2 && VW == 8) {
        out[0] = bf16_to_f32(r.v.x & 0xFFFFu); out[1] = bf16_to_f32(r.v.x >> 16);
        out[2] = bf16_to_f32(r.v.y & 0xFFFFu); out[3] = bf16_to_f32(r.v.y >> 16);
        out[4] = bf16_to_f32(r.v.z & 0xFFFFu); out[5] = bf16_to_f32(r.v.z >> 16);
        out[6] = bf16_to_f32(r.v.w & 0xFFFFu); out[7] = bf16_to_f32(r.v.w >> 16);
    } else if constexpr (sizeof(FT) == 4 && VW == 2) {
        out[0] = r.v.x; out[1] = r.v.y;
    } else if constexpr (sizeof(FT) == 4 && VW == 1) {
        out[0] = r.v;
    } else if constexpr (sizeof(FT) == 2 && VW == 2) {
        out[0] = bf16_to_f32(r.v & 0xFFFFu);
        out[1] = bf16_to_f32(r.v >> 16);
    } else if constexpr (sizeof(FT) == 2 && VW == 4) {
        out[0] = bf16_to_f32(r.v.x & 0xFFFFu); out[1] = bf16_to_f32(r.v.x >> 16);
        out[2] = bf16_to_f32(r.v.y & 0xFFFFu); out[3] = bf16_to_f32(r.v.y >> 16);
    } else {
        out[0] = bf16_to_f32(r.v);
    }
}

template <typename FT, int VW>
__device__ __forceinline__ void load_row(const FT *__restrict__ p, float (&out)[VW])
{
    Raw<FT, VW> r;
    load_raw<FT, VW>(p, r);
    to_float<FT, VW>(r, out);
}

template <int VW>
__device__ __forceinline__ void store_row(float *__restrict__ p, const float (&v)[VW])
{
    if constexpr (VW % 4 == 0) {
#pragma unroll
        for (int k = 0; k < VW; k += 4)
            *reinterpret_cast<float4e *>(p + k) = float4e{v[k], v[k + 1], v[k + 2], v[k + 3]};
    } else if constexpr (VW == 2) {
        *reinterpret_cast<float2e *>(p) = float2e{v[0], v[1]};
    } else {
#pragma unroll
        for (int k = 0; k < VW; ++k) p[k] = v[k];
    }
}

// The same, as streaming stores (bypass the cache's reuse policy): for
// outputs written once and not read back by the kernel.
template <int VW>
__device__ __forceinline__ void store_row_stream(float *__restrict__ p, const float (&v)[VW])
{
    if constexpr (VW % 4 == 0) {
#pragma unroll
        for (int k = 0; k < VW; k += 4) {
            const float4e x = {v[k], v[k + 1], v[k + 2], v[k + 3]};
            __builtin_nontemporal_store(x, reinterpret_cast<float4e *>(p + k));
        }
    } else if constexpr (VW == 2) {
        const float2e x = {v[0], v[1]};
        __builtin_nontemporal_store(x, reinterpret_cast<float2e *>(p));
    } else {
#pragma unroll
        for (int k = 0; k < VW; ++k) __builtin_nontemporal_store(v[k], p + k);
    }
}

}  // namespace dev
}  // namespace fcoo
