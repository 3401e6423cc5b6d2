// Device code shared by the lattice kernels: collision, Dirichlet closure,
// surface reaction, event counts, raw buffer access, workgroup order.
#pragma once

#include "hyb_impl.h"

namespace hyb {
namespace {

// BGK collision with reaction, written as
//   f*_i = (1 - w) f_i + w_i [ w u (1 + 3 e.v + 9/2 (e.v)^2 - 3/2 v.v) - k u ],
// w = 1/tau; u = sum_i f_i (eq. LBM_Macro); the bracket's polynomial is the
// equilibrium of eq. (LBM_feq) with c_s^2 = 1/3 and the quadratic term read
// as -v.v/(2 c_s^2).  Returns u.
//
// Every multiply-add is written out (contraction is off), so a node takes the
// same roundings in every kernel whatever the compiler makes of the code
// around the call: single-step, tile and strip sweeps agree bit for bit.
// Directions pair up as e and -e: with odd = (3 w_q A) d, d = e.v, they take
// (1 - w) f +- odd + w_q (base + odd (3/2 d) / w_q).  The last multiply-add
// takes w_q (..) unrounded, so that no rounding is common to the directions of a
// weight, which would add up in their sum (FP32 states: the relative error
// against 64 bits fell by a few per cent).
template <typename T>
__device__ __forceinline__ T fma_t(T a, T b, T c);
template <> __device__ __forceinline__ double fma_t<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <> __device__ __forceinline__ float fma_t<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename T>
__device__ __forceinline__ T collide(T (&f)[kQ], T vx, T vy, T omega, T k) {
#pragma clang fp contract(off)
    const T u = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7])) + f[8];
    const T A = omega * u;
    const T vv = fma_t(vx, vx, vy * vy);
    const T base = fma_t(A, fma_t(T(-1.5), vv, T(1)), -(k * u));
    const T keep = T(1) - omega;
    const T c1 = T(3.0 * kW[1]) * A, c5 = T(3.0 * kW[5]) * A;
    f[0] = fma_t(T(kW[0]), base, keep * f[0]);
    auto pair = [&](T &fp, T &fm, T d, T c, double w) {
#pragma clang fp contract(off)
        const T odd = c * d;
        const T even = fma_t(odd, T(1.5 / w) * d, base);
        fp = fma_t(T(w), even, fma_t(keep, fp, odd));
        fm = fma_t(T(w), even, fma_t(keep, fm, -odd));
    };
    pair(f[1], f[3], vx, c1, kW[1]);
    pair(f[2], f[4], vy, c1, kW[1]);
    pair(f[5], f[7], vx + vy, c5, kW[5]);
    pair(f[6], f[8], vy - vx, c5, kW[5]);
    return u;
}

// Transpose of the collision: l = dJ/df* after it becomes dJ/df before it,
//   l_p <- (1 - w) l_p + sum_q l_q w_q (w P_q(v) - k),
// P_q = 1 + 3 e.v + 9/2 (e.v)^2 - 3/2 v.v.  Returns sum_q w_q l_q (dJ/dk of the
// node is -u times that).  Written out as the collision, for the same reason;
// taking e and -e (or v and -v) for each other changes no bit of the result.
template <typename T>
__device__ __forceinline__ T collide_transposed(T (&l)[kQ], T vx, T vy, T omega, T k) {
#pragma clang fp contract(off)
    const T s1 = l[1] + l[3], s2 = l[2] + l[4], s5 = l[5] + l[7], s6 = l[6] + l[8];
    const T wl = fma_t(T(kW[5]), s5 + s6, fma_t(T(kW[1]), s1 + s2, T(kW[0]) * l[0]));
    const T vv = fma_t(vx, vx, vy * vy);
    const T even = fma_t(omega, fma_t(T(-1.5), vv, T(1)), -k);
    auto pair = [](T s, T d, T ev) {
#pragma clang fp contract(off)
        return ev * fma_t(T(1.5) * ev, s, d);
    };
    const T q1 = pair(s1, l[1] - l[3], vx) + pair(s2, l[2] - l[4], vy);
    const T q5 = pair(s5, l[5] - l[7], vx + vy) + pair(s6, l[6] - l[8], vy - vx);
    const T S = fma_t(wl, even, omega * fma_t(T(3.0 * kW[1]), q1, T(3.0 * kW[5]) * q5));
    const T keep = T(1) - omega;
#pragma unroll
    for (int q = 0; q < kQ; ++q) l[q] = fma_t(keep, l[q], S);
    return wl;
}

__device__ __forceinline__ bool finite_val(double x) { return x - x == 0.0; }
__device__ __forceinline__ bool finite_val(float x) { return x - x == 0.0f; }

// Adds the number of active lanes whose flag is set to *ctr with one atomic
// per wavefront (the one-node-per-thread kernels).
__device__ __forceinline__ void count_lanes(unsigned long long *ctr, bool flag) {
    const unsigned long long lanes = __ballot(flag);
    if (lanes == 0ull) return;
    if (__lane_id() == __ffsll(static_cast<long long>(lanes)) - 1) atomicAdd(ctr, static_cast<unsigned long long>(__popcll(lanes)));
}

// Event counts of one lane over a whole multi-step launch.  At the patch
// edge a wavefront holds one perimeter node per round, so per-wavefront
// aggregation still leaves one atomic per event; and device-scope atomics
// on one address, issued from every XCD, serialise at the memory side and
// hold up the sweep's own loads and stores there.  The sweeps therefore
// count in registers and add to the device counters once per workgroup.
struct Tally {
    unsigned bad = 0u;          // infeasible closures at owned perimeter nodes
    unsigned nonfinite = 0u;    // owned nodes whose concentration is not finite
};

__device__ __forceinline__ unsigned wave_sum(unsigned v) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

// Adds a workgroup's tallies to the device counters.  `edge` is uniform
// over the workgroup (whether the tile with its ring reaches the patch
// perimeter) and false where no closure ran, so only edge tiles take the
// extra barrier; a non-finite value is rare enough to count per wavefront.
template <int NT>
__device__ __forceinline__ void flush_tally(const LbmArgs &a, const Tally &t, bool edge) {
    if (__ballot(t.nonfinite != 0u) != 0ull) {
        const unsigned s = wave_sum(t.nonfinite);
        if (__lane_id() == 0) atomicAdd(&a.counters[kCntNonfinite], static_cast<unsigned long long>(s));
    }
    if (edge) {
        __shared__ unsigned part[NT / 64];
        const unsigned s = wave_sum(t.bad);
        if (__lane_id() == 0) part[threadIdx.x / 64] = s;
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long sum = 0ull;
#pragma unroll
            for (int w = 0; w < NT / 64; ++w) sum += part[w];
            if (sum != 0ull) atomicAdd(&a.counters[kCntInfeasible], sum);
        }
    }
}

// per-node reaction rate (k field in the arithmetic type) or the uniform one
template <typename T>
__device__ __forceinline__ T node_k(const LbmArgs &a, int n) {
    return a.kfield ? static_cast<const T *>(a.kfield)[n] : T(a.k);
}

// Perimeter slot of perimeter node (i, j) (inverse of slot_to_node).
__device__ __forceinline__ int perimeter_slot(int N, int i, int j) {
    if (j == 0) return i;
    if (j == N - 1) return N + i;
    if (i == 0) return 2 * N + j - 1;
    return 3 * N - 2 + j - 1;
}

// bit q set: the upstream node x - e_q lies outside the patch
__device__ __forceinline__ unsigned outside_bits(int N, int i, int j) {
    unsigned u = 0;
#pragma unroll
    for (int q = 1; q < kQ; ++q) {
        const int si = i - kCx[q], sj = j - kCy[q];
        if (si < 0 || si >= N || sj < 0 || sj >= N) u |= 1u << q;
    }
    return u;
}

// Interface value of eq. (MTS) at weight lam.
__device__ __forceinline__ double mts_value(double a, double b, double lam) {
#pragma clang fp contract(off)
    return (1.0 - lam) * a + lam * b;
}

// Dirichlet closure of eq. (LBM_Dir): the unknowns U share the mass deficit
// R = u^p - sum_known f in proportion to w_i; sums in FP64.  The weights of U
// sum to 1/6 on an edge of the patch and to 11/36 at a corner.  R < 0 (no
// non-negative solution) is reported; with clamp the unknowns become 0,
// otherwise the closed form is kept.
template <typename T>
__device__ __forceinline__ bool dirichlet_close_to(T (&f)[kQ], unsigned unknown, double up, int clamp) {
#pragma clang fp contract(off)
    double known = 0.0;
#pragma unroll
    for (int q = 0; q < kQ; ++q) known += ((unknown >> q) & 1u) ? 0.0 : double(f[q]);
    double R = up - known;
    const bool bad = R < 0.0;
    if (bad && clamp) R = 0.0;
    const double scale = R * (__builtin_popcount(unknown) == 3 ? 6.0 : 36.0 / 11.0);
#pragma unroll
    for (int q = 0; q < kQ; ++q) f[q] = ((unknown >> q) & 1u) ? T(kW[q] * scale) : f[q];
    return bad;
}
// the same at perimeter slot p, weight lam
template <typename T>
__device__ __forceinline__ bool dirichlet_close(const LbmArgs &a, T (&f)[kQ], unsigned unknown, int p,
                                                double lam) {
    return dirichlet_close_to<T>(f, unknown, mts_value(a.bc_a[p], a.bc_b[p], lam), a.clamp);
}

// Workgroups are handed to the 8 XCDs (each with its own L2) in
// round-robin order.  Tile t of T is given to workgroup b so that XCD b % 8
// sweeps one contiguous eighth of the tiles in row-major order: the lines a
// tile shares with its neighbours (pulls, halos) are then fetched into the
// same L2.
__device__ __forceinline__ int xcd_tile(int b, int T) {
    const int x = b & 7, k = b >> 3;
    const int q = T >> 3, r = T & 7;
    return x * q + (x < r ? x : r) + k;
}

// Bounce-back value across a link to a solid node with the surface reaction
// of dissolving solids: (1 - kappa_s) f + kappa_s w_q c_sat (f itself when
// the reaction is off).
template <typename T>
__device__ __forceinline__ T reactive(const LbmArgs &a, T f, int q) {
#pragma clang fp contract(off)
    if (a.kappa_s == 0.0) return f;
    return T((1.0 - a.kappa_s) * double(f) + a.kappa_s * kW[q] * a.c_sat);
}

// Raw buffer access (gfx9 buffer instructions): the array base and size
// live in one SGPR resource and each lane supplies a 32-bit byte offset
// (stores add the plane offset q * plane as the scalar offset), so a pull
// or a store costs no 64-bit address arithmetic.  Offsets at or past
// num_records read as 0 without touching memory.
typedef __amdgpu_buffer_rsrc_t BufRsrc;
__device__ __forceinline__ BufRsrc buf_rsrc(const void *p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename S> struct Buf;
template <> struct Buf<float> {
    static __device__ __forceinline__ float load(BufRsrc r, unsigned v, unsigned s) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, v, s, 0));
    }
    static __device__ __forceinline__ void store_nt(float x, BufRsrc r, unsigned v, unsigned s) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, x), r, v, s, 2);
    }
};
template <> struct Buf<double> {
    typedef decltype(__builtin_amdgcn_raw_buffer_load_b64(BufRsrc(), 0, 0, 0)) Raw;
    static __device__ __forceinline__ double load(BufRsrc r, unsigned v, unsigned s) {
        return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, v, s, 0));
    }
    static __device__ __forceinline__ void store_nt(double x, BufRsrc r, unsigned v, unsigned s) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(Raw, x), r, v, s, 2);
    }
};
template <> struct Buf<_Float16> {
    static __device__ __forceinline__ _Float16 load(BufRsrc r, unsigned v, unsigned s) {
        return __builtin_bit_cast(_Float16, __builtin_amdgcn_raw_buffer_load_b16(r, v, s, 0));
    }
    static __device__ __forceinline__ void store_nt(_Float16 x, BufRsrc r, unsigned v, unsigned s) {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, x), r, v, s, 2);
    }
};

}  // namespace
}  // namespace hyb
