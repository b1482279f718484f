// Device helpers shared by the retrieval and graph-search kernels:
// 16-byte dot products, 64-bit wave exchanges and buffer loads.
#pragma once

#include "common.hpp"

namespace is {

// ---- 16-byte dot products (one 128-bit load of each operand) -------------

struct F32Tag {};
struct BF16Tag {};

__device__ __forceinline__ float dot16(uint4 a, uint4 b, F32Tag) {
    float s = __uint_as_float(a.x) * __uint_as_float(b.x);
    s = fmaf(__uint_as_float(a.y), __uint_as_float(b.y), s);
    s = fmaf(__uint_as_float(a.z), __uint_as_float(b.z), s);
    s = fmaf(__uint_as_float(a.w), __uint_as_float(b.w), s);
    return s;
}

__device__ __forceinline__ float dot16(uint4 a, uint4 b, BF16Tag) {
    // bf16 x bf16 products are exact in fp32
    float s = bf16_lo(a.x) * bf16_lo(b.x);
    s = fmaf(bf16_hi(a.x), bf16_hi(b.x), s);
    s = fmaf(bf16_lo(a.y), bf16_lo(b.y), s);
    s = fmaf(bf16_hi(a.y), bf16_hi(b.y), s);
    s = fmaf(bf16_lo(a.z), bf16_lo(b.z), s);
    s = fmaf(bf16_hi(a.z), bf16_hi(b.z), s);
    s = fmaf(bf16_lo(a.w), bf16_lo(b.w), s);
    s = fmaf(bf16_hi(a.w), bf16_hi(b.w), s);
    return s;
}

// s + <a, b> over one 16-byte unit of each operand in binary64 (exact products).
__device__ __forceinline__ double dot16_f64(uint4 a, uint4 b, double s, F32Tag) {
    s = fma((double)__uint_as_float(a.x), (double)__uint_as_float(b.x), s);
    s = fma((double)__uint_as_float(a.y), (double)__uint_as_float(b.y), s);
    s = fma((double)__uint_as_float(a.z), (double)__uint_as_float(b.z), s);
    return fma((double)__uint_as_float(a.w), (double)__uint_as_float(b.w), s);
}
__device__ __forceinline__ double dot16_f64(uint4 a, uint4 b, double s, BF16Tag) {
    const uint32_t x[4] = {a.x, a.y, a.z, a.w}, y[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s = fma((double)bf16_lo(x[i]), (double)bf16_lo(y[i]), s);
        s = fma((double)bf16_hi(x[i]), (double)bf16_hi(y[i]), s);
    }
    return s;
}

// ---- wave helpers ----------------------------------------------------------

__device__ __forceinline__ uint64_t shfl_xor64(uint64_t v, int off) {
    const uint32_t lo = __shfl_xor((uint32_t)v, off, kWave);
    const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), off, kWave);
    return ((uint64_t)hi << 32) | lo;
}

// Largest value of each 16-lane row, in all of its lanes: DPP quad, half-row and
// row exchanges.
__device__ __forceinline__ uint32_t row16_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false));
    return v;
}

// Largest value over the 64 lanes of a wave (uniform result): the four rows'
// are combined in scalar registers.
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
    v = row16_max_u32(v);
    const uint32_t r0 = __builtin_amdgcn_readlane(v, 0), r1 = __builtin_amdgcn_readlane(v, 16);
    const uint32_t r2 = __builtin_amdgcn_readlane(v, 32), r3 = __builtin_amdgcn_readlane(v, 48);
    return max(max(r0, r1), max(r2, r3));
}

// Lanes below this one whose bit is set in a wave-wide mask.
__device__ __forceinline__ uint32_t lanes_below(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// ---- buffer loads ----------------------------------------------------------

// Raw buffer descriptors: loads at byte offsets >= the descriptor's size
// read zero, which pads ragged row tiles and reduction chunks for free.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;  // gfx9-family raw buffer format word

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes,
                                             kRsrcWord3);
}

__device__ __forceinline__ uint4 buffer_load16(rsrc_t r, uint32_t off, uint32_t soff = 0) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)soff, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}
// The same with the non-temporal hint (cache-policy bit 1): bank rows are
// streamed once per call (3% less time for the 1M-row scan than ordinary
// loads); the queries, re-read for every row tile, keep ordinary loads.
__device__ __forceinline__ uint4 buffer_load16_stream(rsrc_t r, uint32_t off, uint32_t soff = 0) {
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, (int)soff, 2);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

}  // namespace is
