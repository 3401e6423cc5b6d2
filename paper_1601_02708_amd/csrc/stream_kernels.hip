// K fine steps per launch (K = 3 .. 5) on a rectangle of nodes clear of the
// patch perimeter, one wavefront per strip of columns.
//
// A wavefront owns a strip of 64 - 2K columns (its 64 lanes less K ring
// columns on each side) and a band of rows, and walks up the rows with all K
// steps in flight: when row r of the source state has arrived, step 1 finishes
// row r-1, step 2 row r-2, .. step K row r-K, which is stored.  A pull from a
// neighbouring column is a lane shift (DPP), one from a neighbouring row reads
// registers, so the state between the steps needs no LDS and no barrier, and
// wavefronts never wait for each other.
//
// What a step keeps of the rows below (nine values): when row r of its input
// is there, directions 0, 1, 3 (same row) and 2, 5, 6 (row r-1) of row r can be
// gathered and bounced back at once; 4, 7, 8 pull from row r+1 and bounce back
// 2, 5, 6 of row r, which row r+1 pulls anyway.
//
// Bound, four steps at 4096^2: FP64 and FP32 by HBM (counters: 2.67 GB in 538 us
// and 1.48 GB in 285 us, 5.0 and 5.2 TB/s, where a large copy reaches 4.9; VALU 42%
// and 57% of the issue slots), binary16 by VALU issue (92%).  Per four-step launch at 4096^2, porosity 0.6, with
// the frame of tiles (about 28 us): FP64 582 us, FP32 323, binary16 228; the
// LDS tiles, bound by latency at the occupancy their tile allows, took 757, 455
// and 390.
#include "strip_device.h"

namespace hyb {
namespace {

// Wavefronts per SIMD the register budget is set for, and rows taken per turn
// of the row loop.  Two rows a turn spare the copies that return what a step
// keeps to the registers the loop starts with (a tenth of the instructions) for
// a quarter more registers: 4096^2, four steps, binary16 236 us against 252
// with one row and five wavefronts, FP32 329 against 335; FP64 would spill.
template <typename S, int K>
constexpr bool two_rows() { return sizeof(S) < 8 && K <= 4; }
template <typename S, int K>
constexpr int stream_waves_per_simd() { return sizeof(S) == 8 ? (K <= 4 ? 3 : 2) : 4; }

template <typename S, int K, bool KF, bool REC>
__global__ void __launch_bounds__(64 * kStreamWaves, (stream_waves_per_simd<S, K>())) lbm_stream_kernel(LbmArgs a, StreamMap map) {
    typedef typename Pop<S>::T T;
    constexpr int UNR = two_rows<S, K>() ? 2 : 1;
    constexpr int OW = 64 - 2 * K;
    constexpr unsigned sz = sizeof(S), tsz = sizeof(T);
    const int t = xcd_tile(blockIdx.x, map.count);
    const int strip = (t % map.groups_x) * kStreamWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // wavefronts past the last strip run along (the workgroup's barriers count
    // on them) on the last strip's columns
    const int xs = map.nodes.x0 + (strip < map.strips ? strip : map.strips - 1) * OW, y0 = map.nodes.y0 + (t / map.groups_x) * map.rows;
    const int yend = y0 + map.rows < map.nodes.y1 + 1 ? y0 + map.rows : map.nodes.y1 + 1;
    const unsigned P = static_cast<unsigned>(a.pitch), SP = static_cast<unsigned>(a.plane);
    const BufRsrc fsrc = buf_rsrc(a.src, kQ * SP * sz);
    const BufRsrc fdst = buf_rsrc(a.dst, kQ * SP * sz);
    const unsigned NP = static_cast<unsigned>(a.N) * P;
    const BufRsrc mrs = buf_rsrc(a.mask, NP * 2u);
    const BufRsrc vxr = buf_rsrc(a.vx, NP * 4u);
    const BufRsrc vyr = buf_rsrc(a.vy, NP * 4u);
    const BufRsrc kfr = buf_rsrc(KF ? a.kfield : a.vx, NP * tsz);
    const T omega = T(a.omega);
    const T kuni = T(a.k);
    const int lane = __lane_id();
    // lanes past the rectangle read the row's remainder (or the next row, still
    // inside the plane) and are not stored
    const unsigned i = static_cast<unsigned>(xs - K + lane);
    const bool owned = lane >= K && lane < K + OW && static_cast<int>(i) <= map.nodes.x1 && strip < map.strips;
    const unsigned long long owned_lanes = __builtin_amdgcn_ballot_w64(owned);
    const int rend = y0 - K + ((yend - y0 + 2 * K + UNR - 1) / UNR) * UNR;     // rows taken: a multiple of UNR
    unsigned nonfinite = 0u;

    // A finished row leaves through LDS: the four strips' columns together are
    // whole 128-byte lines (FP16S: half lines), stored 16 bytes a lane.  (Rows
    // stored by each wavefront alone begin and end inside lines; full-width
    // lines half as wide were faster than that.)
    constexpr int GW = OW * kStreamWaves, NT = 64 * kStreamWaves, CHUNK = 16 / sz, PER = GW / CHUNK;
    constexpr int ROUNDS_OUT = (kQ * PER + NT - 1) / NT;
    static_assert(GW % CHUNK == 0, "whole chunks");
    __shared__ __align__(16) S rows_out[2][kQ * GW];
    // a recording launch sends u of each step's row the same way: step s+1's
    // is K-1-s rows above the finished row
    constexpr int ROUNDS_U = REC ? (K * PER + NT - 1) / NT : 1;
    __shared__ __align__(16) T rows_u[REC ? 2 : 1][REC ? K * GW : 4];
    const BufRsrc urs = buf_rsrc(REC ? a.u_out : a.dst, static_cast<unsigned>(K * a.u_step));
    unsigned u_at[ROUNDS_U];
    int u_row[ROUNDS_U];                     // rows above row r - K
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    unsigned out_at[ROUNDS_OUT];
    bool out_on[ROUNDS_OUT];
    {
        const int gx0 = map.nodes.x0 + (t % map.groups_x) * GW;
#pragma unroll
        for (int c = 0; c < ROUNDS_OUT; ++c) {
            const int chunk = static_cast<int>(threadIdx.x) + NT * c, q = chunk / PER, col = gx0 + (chunk % PER) * CHUNK;
            out_on[c] = chunk < kQ * PER && col <= map.nodes.x1;
            out_at[c] = (q * SP + static_cast<unsigned>(col)) * sz;
        }
        if constexpr (REC) {
#pragma unroll
            for (int c = 0; c < ROUNDS_U; ++c) {
                const int chunk = static_cast<int>(threadIdx.x) + NT * c, s = chunk / PER, col = gx0 + (chunk % PER) * CHUNK;
                u_row[c] = chunk < K * PER && col <= map.nodes.x1 ? K - 1 - s : -(1 << 30);
                u_at[c] = static_cast<unsigned>(s * a.u_step) + (static_cast<unsigned>(K - 1 - s) * P + static_cast<unsigned>(col)) * tsz;
            }
        }
    }

    struct Row {
        S f[kQ];
        unsigned m;
        float vx, vy;
        T k;
    };
    auto fetch = [&](int r, Row &w) {
        const unsigned at = static_cast<unsigned>(r) * P;
#pragma unroll
        for (int q = 0; q < kQ; ++q) w.f[q] = Buf<S>::load(fsrc, i * sz, (q * SP + at) * sz);
        w.m = __builtin_amdgcn_raw_buffer_load_b16(mrs, i * 2u, at * 2u, 0);
        w.vx = Buf<float>::load(vxr, i * 4u, at * 4u);
        w.vy = Buf<float>::load(vyr, i * 4u, at * 4u);
        if constexpr (KF) w.k = Buf<T>::load(kfr, i * tsz, at * tsz);
    };

    // per step s+1: gathered directions 0, 1, 3, 2, 5, 6 of the row it works
    // on, and directions 2, 5, 6 of that row of its input
    T part[K][6], own[K][3];
#pragma unroll
    for (int s = 0; s < K; ++s) {
#pragma unroll
        for (int c = 0; c < 6; ++c) part[s][c] = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) own[s][c] = T(0);
    }
    // flag words, owned fluid lanes, velocities and rates of the last K+1 rows
    unsigned mk[K + 1];
    unsigned long long live[K + 1];
    float vx[K + 1], vy[K + 1];
    T kn[K + 1];
#pragma unroll
    for (int d = 0; d <= K; ++d) {
        mk[d] = kMaskSolid;
        live[d] = 0ull;
        vx[d] = vy[d] = 0.f;
        kn[d] = kuni;
    }

    Row next;
    fetch(y0 - K, next);
    auto row = [&](int r) {
        __builtin_amdgcn_sched_barrier(0);
        T g[kQ];
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = Pop<S>::ld(next.f[q], q, a);
        mk[0] = next.m;
        live[0] = __builtin_amdgcn_ballot_w64(!(next.m & kMaskSolid)) & owned_lanes;
        vx[0] = next.vx;
        vy[0] = next.vy;
        if constexpr (KF) kn[0] = next.k;
        fetch(r + 1 < rend ? r + 1 : r, next);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < K; ++s) {
            // finish row r-s-1 of step s+1
            const unsigned m = mk[s + 1], mn = mk[s];
            T f[kQ];
            f[0] = part[s][0];
            f[1] = part[s][1];
            f[3] = part[s][2];
            f[2] = part[s][3];
            f[5] = part[s][4];
            f[6] = part[s][5];
            f[4] = back_or_pull(m, 4, own[s][0], g[4]);
            f[7] = back_or_pull(m, 7, own[s][1], lane_from_right(g[7]));
            f[8] = back_or_pull(m, 8, own[s][2], lane_from_left(g[8]));
            // gather what row r-s has
            part[s][0] = g[0];
            part[s][1] = back_or_pull(mn, 1, g[3], lane_from_left(g[1]));
            part[s][2] = back_or_pull(mn, 3, g[1], lane_from_right(g[3]));
            part[s][3] = back_or_pull(mn, 2, g[4], own[s][0]);
            part[s][4] = back_or_pull(mn, 5, g[7], lane_from_left(own[s][1]));
            part[s][5] = back_or_pull(mn, 6, g[8], lane_from_right(own[s][2]));
            own[s][0] = g[2];
            own[s][1] = g[5];
            own[s][2] = g[6];
            // made here and now: left to itself the compiler defers these
            // selects to the end of the row and carries their operands (twice
            // the registers) through the later steps
#pragma unroll
            for (int c = 0; c < 6; ++c) asm volatile("" : "+v"(part[s][c]));
#pragma unroll
            for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(own[s][c]));
            const T u = collide<T>(f, T(vx[s + 1]), T(vy[s + 1]), omega, KF ? kn[s + 1] : kuni);
            if constexpr (REC) {
                if (lane >= K && lane < K + OW) rows_u[r & 1][s * GW + wave * OW + lane - K] = u;
            }
            const int j = r - s - 1;
            const unsigned long long nf = __builtin_amdgcn_ballot_w64(!__builtin_isfinite(u)) & live[s + 1];
            nonfinite += j >= y0 && j < yend ? static_cast<unsigned>(__popcll(nf)) : 0u;
#pragma unroll
            for (int q = 0; q < kQ; ++q) g[q] = f[q];
            // keep the scheduler from starting every step's selects at once
            // (their masks alone would take eight registers a step)
            __builtin_amdgcn_sched_barrier(0);
        }
        // The next row has to be here before this one is stored: the counter
        // the loads are waited on also counts stores, so a wait after them
        // would wait for them too.
#pragma unroll
        for (int q = 0; q < kQ; ++q) asm volatile("" : "+v"(next.f[q]));
        asm volatile("" : "+v"(next.m), "+v"(next.vx), "+v"(next.vy));
        if constexpr (KF) asm volatile("" : "+v"(next.k));
        __builtin_amdgcn_sched_barrier(0);
        // row r-K has taken all K steps
        const int j = r - K;
        if (REC || (j >= y0 && j < yend)) {
            S *out = rows_out[j & 1];
            if (lane >= K && lane < K + OW) {
#pragma unroll
                for (int q = 0; q < kQ; ++q) out[q * GW + wave * OW + lane - K] = Pop<S>::st(g[q], q, a);
            }
            // one barrier a row: a row's buffer is written again two rows on,
            // after the barrier that follows its last read
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const unsigned at = static_cast<unsigned>(j) * P * sz;
#pragma unroll
            for (int c = 0; c < ROUNDS_OUT; ++c)
                if (out_on[c] && (!REC || (j >= y0 && j < yend))) {
                    const Quad v = *reinterpret_cast<const Quad *>(out + (threadIdx.x + NT * c) * CHUNK);
                    __builtin_amdgcn_raw_buffer_store_b128(v, fdst, out_at[c], at, kNonTemporal);
                }
            if constexpr (REC) {
#pragma unroll
                for (int c = 0; c < ROUNDS_U; ++c)
                    if (j + u_row[c] >= y0 && j + u_row[c] < yend) {
                        const Quad v = *reinterpret_cast<const Quad *>(&rows_u[r & 1][(threadIdx.x + NT * c) * CHUNK]);
                        __builtin_amdgcn_raw_buffer_store_b128(v, urs, u_at[c] + static_cast<unsigned>(j) * P * tsz, 0, kNonTemporal);
                    }
            }
        }
#pragma unroll
        for (int d = K; d > 0; --d) {
            mk[d] = mk[d - 1];
            live[d] = live[d - 1];
            vx[d] = vx[d - 1];
            vy[d] = vy[d - 1];
            kn[d] = kn[d - 1];
            // (no values derived from these are kept from one step of a node
            // to its next: they would not fit the registers)
            asm volatile("" : "+v"(mk[d]), "+v"(vx[d]), "+v"(vy[d]));
        }
    };
#pragma unroll 1
    for (int r = y0 - K; r < rend; r += UNR) {
#pragma unroll
        for (int n = 0; n < UNR; ++n) row(r + n);
    }
    if (nonfinite && lane == 0) atomicAdd(&a.counters[kCntNonfinite], static_cast<unsigned long long>(nonfinite));
}

template <typename S, int K>
hipError_t stream_impl(const LbmArgs &a, const NodeRect &nodes, hipStream_t s) {
    const StreamMap m = stream_map(nodes, K, stream_waves_per_simd<S, K>());
    const dim3 grid(m.count), block(64 * kStreamWaves);
    if (a.u_out) {
        if constexpr (sizeof(S) >= 4) {
            if (a.kfield) hipLaunchKernelGGL((lbm_stream_kernel<S, K, true, true>), grid, block, 0, s, a, m);
            else hipLaunchKernelGGL((lbm_stream_kernel<S, K, false, true>), grid, block, 0, s, a, m);
            return hipGetLastError();
        }
        return hipErrorInvalidValue;
    }
    if (a.kfield) hipLaunchKernelGGL((lbm_stream_kernel<S, K, true, false>), grid, block, 0, s, a, m);
    else hipLaunchKernelGGL((lbm_stream_kernel<S, K, false, false>), grid, block, 0, s, a, m);
    return hipGetLastError();
}

template <typename S>
hipError_t stream_steps(const LbmArgs &a, int K, const NodeRect &nodes, hipStream_t s) {
    if (K == 3) return stream_impl<S, 3>(a, nodes, s);
    if (K == 4) return stream_impl<S, 4>(a, nodes, s);
    if (K == 5) return stream_impl<S, 5>(a, nodes, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_lbm_stream(const LbmArgs &a, int prec, int K, const NodeRect &nodes, hipStream_t s) {
    if (a.flux || a.kappa_s != 0.0 || a.keep_solid || a.mid) return hipErrorInvalidValue;
    if (nodes.x1 < nodes.x0 || nodes.y1 < nodes.y0) return hipSuccess;
    // every pull of every step stays inside the patch and off its perimeter nodes
    if (nodes.x0 < K || nodes.y0 < K || nodes.x1 > a.N - 1 - K || nodes.y1 > a.N - 1 - K) return hipErrorInvalidValue;
    if (prec == HYB_FP64) return stream_steps<double>(a, K, nodes, s);
    if (prec == HYB_FP32) return stream_steps<float>(a, K, nodes, s);
    return stream_steps<_Float16>(a, K, nodes, s);
}

}  // namespace hyb
