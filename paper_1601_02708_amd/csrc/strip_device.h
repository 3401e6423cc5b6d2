// What the strip kernels share: lane shifts, the bounce-back select, the cut of a
// rectangle of nodes into strips and bands.
#pragma once

#include "lbm_device.h"

#include <type_traits>

namespace hyb {
namespace {

// dst lane i takes lane i-1 (from_left) or i+1 (from_right); lanes without a
// source take 0 (ring lanes, whose results are not used)
__device__ __forceinline__ float lane_from_left(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_from_right(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), 0x130, 0xf, 0xf, true));
}
struct TwoWords {
    int lo, hi;
};
__device__ __forceinline__ double lane_from_left(double x) {
    TwoWords w = __builtin_bit_cast(TwoWords, x);
    w.lo = __builtin_amdgcn_update_dpp(0, w.lo, 0x138, 0xf, 0xf, true);
    w.hi = __builtin_amdgcn_update_dpp(0, w.hi, 0x138, 0xf, 0xf, true);
    return __builtin_bit_cast(double, w);
}
__device__ __forceinline__ double lane_from_right(double x) {
    TwoWords w = __builtin_bit_cast(TwoWords, x);
    w.lo = __builtin_amdgcn_update_dpp(0, w.lo, 0x130, 0xf, 0xf, true);
    w.hi = __builtin_amdgcn_update_dpp(0, w.hi, 0x130, 0xf, 0xf, true);
    return __builtin_bit_cast(double, w);
}

// back where bit q of m is set, else pull.  The bit is widened to a word mask
// and the words merged (one v_bfe_i32, one v_bfi_b32 per word); the empty asm
// keeps the compiler from turning that back into a compare and a select.
__device__ __forceinline__ int bit_mask(unsigned m, int q) {
    int s = __builtin_amdgcn_sbfe(static_cast<int>(m), q, 1);
    asm("" : "+v"(s));
    return s;
}
__device__ __forceinline__ float back_or_pull(unsigned m, int q, float back, float pull) {
    const int s = bit_mask(m, q);
    const int b = __builtin_bit_cast(int, back), p = __builtin_bit_cast(int, pull);
    return __builtin_bit_cast(float, (s & b) | (~s & p));
}
__device__ __forceinline__ double back_or_pull(unsigned m, int q, double back, double pull) {
    const int s = bit_mask(m, q);
    const TwoWords b = __builtin_bit_cast(TwoWords, back), p = __builtin_bit_cast(TwoWords, pull);
    const TwoWords o = {(s & b.lo) | (~s & p.lo), (s & b.hi) | (~s & p.hi)};
    return __builtin_bit_cast(double, o);
}

// The nodes of a launch, cut into strips of 64 - 2K columns and bands of rows;
// a workgroup is four neighbouring strips of one band.
struct StreamMap {
    NodeRect nodes;
    int strips, groups_x, rows;             // rows per band
    int count;                              // workgroups
};

constexpr int kStreamWaves = 4;
constexpr int kComputeUnits = 256;
constexpr int kNonTemporal = 2;          // cache policy bit of the buffer store
typedef unsigned Quad __attribute__((ext_vector_type(4)));

// The strips and bands of a launch of K steps, `waves` wavefronts per SIMD
// resident.  Bands: as many workgroups as are resident at once, so that none
// starts late with a whole band before it (4096^2 FP32: 335 us; two rounds of
// them 351; bands of 16 rows 357, which recompute 2K rows each).
inline StreamMap stream_map(const NodeRect &nodes, int K, int waves) {
    const int OW = 64 - 2 * K;
    StreamMap m{};
    m.nodes = nodes;
    m.strips = (nodes.x1 - nodes.x0 + OW) / OW;
    m.groups_x = (m.strips + kStreamWaves - 1) / kStreamWaves;
    const int h = nodes.y1 - nodes.y0 + 1;
    const int slots = kComputeUnits * waves;
    const int bands = slots / m.groups_x > 1 ? slots / m.groups_x : 1;
    m.rows = (h + bands - 1) / bands;
    if (m.rows < 4) m.rows = 4;
    m.count = m.groups_x * ((h + m.rows - 1) / m.rows);
    return m;
}

}  // namespace
}  // namespace hyb
