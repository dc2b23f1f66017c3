// Device helpers for the gfx950 COUNTDOWN kernels: 16-byte bf16 row loads,
// bf16 dot products on v_dot2_f32_bf16, DPP wavefront reductions, SiLU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cdk {

constexpr int kWave = 64;                     // CDNA wavefront width
constexpr int kBlock = 256;                   // threads per workgroup (4 waves)
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kColsPerLoad = kWave * 8;       // bf16 columns covered by one wave-wide 16 B load
constexpr int kMaxRowsPerBlock = 64;          // one ballot word of local rows

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ u32x4 load16(const uint16_t *p)
{
    return *reinterpret_cast<const u32x4 *>(p);
}

__device__ __forceinline__ u32x4 zero16()
{
    u32x4 z = {0u, 0u, 0u, 0u};
    return z;
}

// a.lo*b.lo + a.hi*b.hi + c for two packed bf16 pairs, fp32 accumulate
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c)
{
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a),
                                           __builtin_bit_cast(bf16x2_t, b), c, false);
}

// 8-element bf16 dot product of two 16-byte chunks added to acc
__device__ __forceinline__ float dot8(const u32x4 &w, const u32x4 &x, float acc)
{
    acc = dot2_bf16(w.x, x.x, acc);
    acc = dot2_bf16(w.y, x.y, acc);
    acc = dot2_bf16(w.z, x.z, acc);
    acc = dot2_bf16(w.w, x.w, acc);
    return acc;
}

// exact bf16 -> fp32 of the low / high half of a packed pair
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }

// DPP move of v with controls CTRL; lanes outside ROW_MASK return 0
template <int CTRL, int ROW_MASK = 0xF>
__device__ __forceinline__ float dpp0(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xF, false));
}

constexpr int kDppQuadSwap1 = 0xB1;   // quad_perm [1,0,3,2]
constexpr int kDppQuadSwap2 = 0x4E;   // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // row_half_mirror
constexpr int kDppMirror = 0x140;     // row_mirror
constexpr int kDppBcast15 = 0x142;    // row_bcast:15
constexpr int kDppBcast31 = 0x143;    // row_bcast:31

// Sum over aligned segments of 2^LOG lanes (LOG in 0..6). Afterwards the
// last lane of every segment holds the segment sum (for LOG <= 4 every lane
// of the segment does).
template <int LOG>
__device__ __forceinline__ float segment_sum(float v)
{
    if constexpr (LOG >= 1) v += dpp0<kDppQuadSwap1>(v);
    if constexpr (LOG >= 2) v += dpp0<kDppQuadSwap2>(v);
    if constexpr (LOG >= 3) v += dpp0<kDppHalfMirror>(v);
    if constexpr (LOG >= 4) v += dpp0<kDppMirror>(v);
    if constexpr (LOG >= 5) v += dpp0<kDppBcast15, 0xA>(v);
    if constexpr (LOG >= 6) v += dpp0<kDppBcast31, 0xC>(v);
    return v;
}

// Sum over the 64 lanes of a wave, returned uniformly to every lane.
__device__ __forceinline__ float wave_sum(float v)
{
    v = segment_sum<6>(v);
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// SiLU(z) = z * sigmoid(z) (the Gated-MLP activation); saturates to -0 / z
// without NaN for large |z|.
__device__ __forceinline__ float silu(float z)
{
    return z / (1.0f + expf(-z));
}

__device__ __forceinline__ uint64_t ballot(bool p)
{
    return __ballot(p);
}

// number of set bits of m below this lane
__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Lanes whose chunk lies past the end of a row (ragged d_model) or of the
// token batch load these 16 zero bytes instead: an address select before the
// load rather than a select of the loaded data, which would make the compiler
// wait for each load on its own.
inline __device__ __align__(16) uint32_t kZeroChunk[4] = {0u, 0u, 0u, 0u};  // never written

template <class T>
__device__ __forceinline__ const T *or_zero(bool ok, const T *p)
{
    return ok ? p : reinterpret_cast<const T *>(kZeroChunk);
}

// ---- matrix cores: one 16 x 16 tile, 32 columns of the contraction per step

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTile = 16;

__device__ __forceinline__ f32x4_t mfma16(const u32x4 &a, const u32x4 &b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                    __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// ---- packed ternary weights (layout: countdown.h, countdown_ternary_pack)

constexpr uint32_t kTernLut = 0x00BF3F00u;  // bytes: code 0 -> 0x00, 1 -> 0x3F, 2 -> 0xBF
constexpr uint32_t kTernPairMask = 0x03000300u;

// bf16 pair (weights 2m, 2m + 1 of unit j's half of word W), each 0 or +-0.5
// (in the FFN kernels j and m are compile-time constants after unrolling)
__device__ __forceinline__ uint32_t tern_pair(uint32_t W, int j, int m)
{
    const uint32_t sel = (j & 1) ? (W << (8 - 2 * m)) & kTernPairMask : (W >> (2 * m)) & kTernPairMask;
    return __builtin_amdgcn_perm(0u, kTernLut, sel);
}

} // namespace cdk
