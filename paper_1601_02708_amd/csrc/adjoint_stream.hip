// K reversed fine steps per launch (K = 2 .. 5) on a rectangle of nodes clear of
// the patch perimeter, one wavefront per strip of columns.
//
// Written in flipped directions, L_q = l_opp(q), a reversed step streams as a
// forward one does: L_q(y) is the opposite value of y itself where y bounced
// back along q, else the value of y - e_q after the transposed collision.  So
// the forward strips' walk serves: row r arrives and is collided (the step
// reversed first), and each further step finishes one row below the one before
// it, every pull a lane shift or a register.  The collision comes before the
// pull here, so step s collides row r-s and row r-K leaves.
//
// A node's dJ/dk terms, one a step, travel with its row in FP64 and are taken
// off the gradient once per launch.  Cotangents and gradients leave through LDS
// as the forward rows do.  A launch that adds to the dense FP64 array is bound by
// that array's traffic (2048^2 FP32, five steps: 203 us, one that overwrites it 136).
//
// Bound: FP64 by HBM, FP32 by a row's latency at three wavefronts a SIMD.  2048^2 FP32,
// five steps: 124 us (150 G node-steps a second), the tiles 290; pairs of steps in
// tiles took 214 each.
#include "strip_device.h"

namespace hyb {
namespace {

// ADD: the result is added to the dense array, whose row is fetched a row's time
// before (a wavefront less at K = 4 for the registers)
template <typename T, int K, bool ADD = false>
constexpr int adjoint_waves_per_simd() { return sizeof(T) == 8 ? (K <= 2 ? 3 : 2) : (K <= (ADD ? 3 : 4) ? 4 : 3); }

template <typename T, int K, bool KF, bool DENSE, bool ADD>
__global__ void __launch_bounds__(64 * kStreamWaves, (adjoint_waves_per_simd<T, K, ADD>()))
    adj_stream_kernel(AdjSteps A, StreamMap map, NodeRect own_rect) {
    constexpr int OW = 64 - 2 * K;
    constexpr unsigned sz = sizeof(T);
    const LbmArgs &a = A.a;
    const int N = a.N;
    const int t = xcd_tile(blockIdx.x, map.count);
    const int strip = (t % map.groups_x) * kStreamWaves + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // wavefronts past the last strip run along on the last strip's columns
    const int xs = map.nodes.x0 + (strip < map.strips ? strip : map.strips - 1) * OW, y0 = map.nodes.y0 + (t / map.groups_x) * map.rows;
    const int yend = y0 + map.rows < map.nodes.y1 + 1 ? y0 + map.rows : map.nodes.y1 + 1;
    const unsigned P = static_cast<unsigned>(a.pitch), SP = static_cast<unsigned>(a.plane);
    const BufRsrc fsrc = buf_rsrc(A.lam, kQ * SP * sz);
    const BufRsrc fdst = buf_rsrc(A.out, kQ * SP * sz);
    const unsigned NP = static_cast<unsigned>(N) * P;
    const BufRsrc mrs = buf_rsrc(a.mask, NP * 2u);
    const BufRsrc vxr = buf_rsrc(a.vx, NP * 4u);
    const BufRsrc vyr = buf_rsrc(a.vy, NP * 4u);
    const BufRsrc kfr = buf_rsrc(KF ? a.kfield : a.vx, NP * sz);
    // without dJ/dk these are empty: loads read 0, stores are dropped
    const unsigned u_step = static_cast<unsigned>(a.u_step);
    const BufRsrc urs = buf_rsrc(static_cast<const char *>(a.u_rec) - (K - 1) * a.u_step,
                                 A.grad_k ? (K - 1) * u_step + NP * sz : 0u);
    const BufRsrc grs = buf_rsrc(A.grad_k, A.grad_k ? static_cast<unsigned>(N) * static_cast<unsigned>(N) * 8u : 0u);
    const T omega = T(a.omega);
    const T kuni = T(a.k);
    const int lane = __lane_id();
    const unsigned i = static_cast<unsigned>(xs - K + lane);
    const int rend = yend + K;

    // rows on their way out: cotangents (FP64 when they go to the dense array),
    // dJ/dk
    typedef typename std::conditional<DENSE, double, T>::type O;
    constexpr int GW = OW * kStreamWaves, NT = 64 * kStreamWaves, CHUNK = 16 / sz, PER = GW / CHUNK;
    constexpr int ROUNDS_OUT = DENSE ? 1 : (kQ * PER + NT - 1) / NT;
    static_assert(GW % CHUNK == 0 && GW <= NT, "whole chunks, a column a thread");
    __shared__ __align__(16) O rows_out[2][kQ * GW];
    __shared__ double rows_k[2][GW];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int gx0 = map.nodes.x0 + (t % map.groups_x) * GW;
    unsigned out_at[ROUNDS_OUT];
    bool out_on[ROUNDS_OUT];
    if constexpr (!DENSE) {
#pragma unroll
        for (int c = 0; c < ROUNDS_OUT; ++c) {
            const int chunk = static_cast<int>(threadIdx.x) + NT * c, q = chunk / PER, col = gx0 + (chunk % PER) * CHUNK;
            out_on[c] = chunk < kQ * PER && col <= map.nodes.x1;
            out_at[c] = (q * SP + static_cast<unsigned>(col)) * sz;
        }
    }
    const int my_col = gx0 + static_cast<int>(threadIdx.x);          // column this thread stores
    const bool col_on = static_cast<int>(threadIdx.x) < GW && my_col <= map.nodes.x1;
    const bool k_on = col_on && my_col >= own_rect.x0 && my_col <= own_rect.x1;

    struct Row {
        T f[kQ];
        unsigned m;
        float vx, vy;
        T k;
        T u[K];
        double gk;
    };
    // row r, with u of step s at row r-s and dJ/dk of the row that leaves
    auto fetch = [&](int r, Row &w) {
        const unsigned at = static_cast<unsigned>(r) * P;
#pragma unroll
        for (int q = 0; q < kQ; ++q) w.f[q] = Buf<T>::load(fsrc, i * sz, (kOpp[q] * SP + at) * sz);
        w.m = __builtin_amdgcn_raw_buffer_load_b16(mrs, i * 2u, at * 2u, 0);
        w.vx = Buf<float>::load(vxr, i * 4u, at * 4u);
        w.vy = Buf<float>::load(vyr, i * 4u, at * 4u);
        if constexpr (KF) w.k = Buf<T>::load(kfr, i * sz, at * sz);
#pragma unroll
        for (int s = 0; s < K; ++s) {
            // (rows below the band's first ring are not used)
            const unsigned row = static_cast<unsigned>(r - s > 0 ? r - s : 0);
            w.u[s] = Buf<T>::load(urs, i * sz, (K - 1 - s) * u_step + row * P * sz);
        }
        const int j = r - (K - 1);
        w.gk = Buf<double>::load(grs, k_on ? static_cast<unsigned>(my_col) * 8u : 0u,
                                 j >= y0 ? static_cast<unsigned>(j) * static_cast<unsigned>(N) * 8u : 0u);
    };

    // as in the forward strips
    T part[K][6], own[K][3];
#pragma unroll
    for (int s = 0; s < K; ++s) {
#pragma unroll
        for (int c = 0; c < 6; ++c) part[s][c] = T(0);
#pragma unroll
        for (int c = 0; c < 3; ++c) own[s][c] = T(0);
    }
    unsigned mk[K + 1];
    float vx[K], vy[K];
    T kn[K];
    double sum[K];                           // dJ/dk terms of the row each step finished last
    mk[K] = kMaskSolid;
#pragma unroll
    for (int d = 0; d < K; ++d) {
        mk[d] = kMaskSolid;
        vx[d] = vy[d] = 0.f;
        kn[d] = kuni;
        sum[d] = 0.0;
    }

    Row next;
    fetch(y0 - K, next);
#pragma unroll 1
    for (int r = y0 - K; r < rend; ++r) {
        __builtin_amdgcn_sched_barrier(0);
        T g[kQ], u[K];
#pragma unroll
        for (int q = 0; q < kQ; ++q) g[q] = next.f[q];
#pragma unroll
        for (int s = 0; s < K; ++s) u[s] = next.u[s];
        const double gk_old = next.gk;
        mk[0] = next.m;
        vx[0] = -next.vx;                    // flipped directions
        vy[0] = -next.vy;
        if constexpr (KF) kn[0] = next.k;
        double there[ADD ? kQ : 1];
        if constexpr (ADD) {
            if (col_on && r - K >= y0) {
#pragma unroll
                for (int q = 0; q < kQ; ++q) there[q] = A.out_dense[((size_t)q * N + r - K) * N + my_col];
            }
        }
        fetch(r + 1 < rend ? r + 1 : r, next);
        __builtin_amdgcn_sched_barrier(0);
        double term;
        {
            const T wl = collide_transposed<T>(g, T(vx[0]), T(vy[0]), omega, KF ? kn[0] : kuni);
            term = double(u[0]) * double(wl);
        }
#pragma unroll
        for (int s = 0; s < K; ++s) {
            // pull row r-s-1 of step s, then collide it as step s+1
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
            part[s][0] = g[0];
            part[s][1] = back_or_pull(mn, 1, g[3], lane_from_left(g[1]));
            part[s][2] = back_or_pull(mn, 3, g[1], lane_from_right(g[3]));
            part[s][3] = back_or_pull(mn, 2, g[4], own[s][0]);
            part[s][4] = back_or_pull(mn, 5, g[7], lane_from_left(own[s][1]));
            part[s][5] = back_or_pull(mn, 6, g[8], lane_from_right(own[s][2]));
            own[s][0] = g[2];
            own[s][1] = g[5];
            own[s][2] = g[6];
            // made here and now, as in the forward strips
#pragma unroll
            for (int c = 0; c < 6; ++c) asm volatile("" : "+v"(part[s][c]));
#pragma unroll
            for (int c = 0; c < 3; ++c) asm volatile("" : "+v"(own[s][c]));
            if (s + 1 < K) {
                const T wl = collide_transposed<T>(f, T(vx[s + 1 < K ? s + 1 : 0]), T(vy[s + 1 < K ? s + 1 : 0]), omega,
                                                   KF ? kn[s + 1 < K ? s + 1 : 0] : kuni);
                const double before = sum[s];
                sum[s] = term;
                term = before + double(u[s + 1 < K ? s + 1 : 0]) * double(wl);
            }
#pragma unroll
            for (int q = 0; q < kQ; ++q) g[q] = f[q];
            __builtin_amdgcn_sched_barrier(0);
        }
        // the next row is here before this one is stored (see the forward strips)
#pragma unroll
        for (int q = 0; q < kQ; ++q) asm volatile("" : "+v"(next.f[q]));
#pragma unroll
        for (int s = 0; s < K; ++s) asm volatile("" : "+v"(next.u[s]));
        asm volatile("" : "+v"(next.m), "+v"(next.vx), "+v"(next.vy), "+v"(next.gk));
        if constexpr (KF) asm volatile("" : "+v"(next.k));
        __builtin_amdgcn_sched_barrier(0);
        // row r-K is done, and the dJ/dk terms of row r-K+1
        const int j = r - K;
        O *out = rows_out[r & 1];
        if (lane >= K && lane < K + OW) {
            const bool fluid = !(mk[K] & kMaskSolid);
#pragma unroll
            for (int q = 0; q < kQ; ++q) out[kOpp[q] * GW + wave * OW + lane - K] = fluid ? O(g[q]) : O(0);
            rows_k[r & 1][wave * OW + lane - K] = (mk[K - 1] & kMaskSolid) ? 0.0 : term;
        }
        // one barrier a row: a buffer is written again two rows on, after the
        // barrier that follows its last read
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (j >= y0 && j < yend) {
            if constexpr (DENSE) {
                if (col_on) {
#pragma unroll
                    for (int q = 0; q < kQ; ++q) {
                        double *row = A.out_dense + ((size_t)q * N + j) * N;
                        row[my_col] = ADD ? there[ADD ? q : 0] + out[q * GW + threadIdx.x] : out[q * GW + threadIdx.x];
                    }
                }
            } else {
                const unsigned at = static_cast<unsigned>(j) * P * sz;
#pragma unroll
                for (int c = 0; c < ROUNDS_OUT; ++c)
                    if (out_on[c]) {
                        const Quad v = *reinterpret_cast<const Quad *>(out + (threadIdx.x + NT * c) * CHUNK);
                        __builtin_amdgcn_raw_buffer_store_b128(v, fdst, out_at[c], at, kNonTemporal);
                    }
            }
        }
        if (k_on && j + 1 >= y0 && j + 1 < yend && j + 1 >= own_rect.y0 && j + 1 <= own_rect.y1)
            Buf<double>::store_nt(gk_old - rows_k[r & 1][threadIdx.x], grs, static_cast<unsigned>(my_col) * 8u,
                                  static_cast<unsigned>(j + 1) * static_cast<unsigned>(N) * 8u);
#pragma unroll
        for (int d = K; d > 0; --d) {
            mk[d] = mk[d - 1];
            asm volatile("" : "+v"(mk[d]));
            if (d < K) {
                vx[d] = vx[d - 1];
                vy[d] = vy[d - 1];
                kn[d] = kn[d - 1];
                asm volatile("" : "+v"(vx[d]), "+v"(vy[d]));
            }
        }
    }
}

template <typename T, int K>
hipError_t strips_impl(const AdjSteps &A, const NodeRect &nodes, const NodeRect &own, hipStream_t s) {
    const dim3 block(64 * kStreamWaves);
    if constexpr (sizeof(T) == 4) {
        if (A.accumulate) {
            const StreamMap m = stream_map(nodes, K, adjoint_waves_per_simd<T, K, true>());
            if (A.a.kfield) hipLaunchKernelGGL((adj_stream_kernel<T, K, true, true, true>), dim3(m.count), block, 0, s, A, m, own);
            else hipLaunchKernelGGL((adj_stream_kernel<T, K, false, true, true>), dim3(m.count), block, 0, s, A, m, own);
            return hipGetLastError();
        }
    }
    const StreamMap m = stream_map(nodes, K, adjoint_waves_per_simd<T, K>());
    const dim3 grid(m.count);
    if (A.a.kfield && A.out_dense) hipLaunchKernelGGL((adj_stream_kernel<T, K, true, true, false>), grid, block, 0, s, A, m, own);
    else if (A.a.kfield) hipLaunchKernelGGL((adj_stream_kernel<T, K, true, false, false>), grid, block, 0, s, A, m, own);
    else if (A.out_dense) hipLaunchKernelGGL((adj_stream_kernel<T, K, false, true, false>), grid, block, 0, s, A, m, own);
    else hipLaunchKernelGGL((adj_stream_kernel<T, K, false, false, false>), grid, block, 0, s, A, m, own);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_adjoint_strips(const AdjSteps &A, int prec, const NodeRect &nodes, const NodeRect &own,
                                 hipStream_t s) {
    const int K = A.K, chunk = prec == HYB_FP64 ? 2 : 4;
    if (A.a.clamp || A.a.kappa_s != 0.0 || A.inj || (A.accumulate && (!A.out_dense || prec != HYB_FP32)) || A.lam_dense || !A.lam) return hipErrorInvalidValue;
    if (A.grad_k && !A.a.u_rec) return hipErrorInvalidValue;
    if (nodes.x1 < nodes.x0 || nodes.y1 < nodes.y0) return hipSuccess;
    // no pull reaches a perimeter node's row or column
    if (nodes.x0 <= K || nodes.y0 <= K || nodes.x1 >= A.a.N - 1 - K || nodes.y1 >= A.a.N - 1 - K || nodes.x0 % chunk)
        return hipErrorInvalidValue;
    if (prec == HYB_FP64) {
        if (K == 2) return strips_impl<double, 2>(A, nodes, own, s);
        if (K == 3) return strips_impl<double, 3>(A, nodes, own, s);
        if (K == 4) return strips_impl<double, 4>(A, nodes, own, s);
    } else if (prec == HYB_FP32) {
        if (K == 2) return strips_impl<float, 2>(A, nodes, own, s);
        if (K == 3) return strips_impl<float, 3>(A, nodes, own, s);
        if (K == 4) return strips_impl<float, 4>(A, nodes, own, s);
        if (K == 5) return strips_impl<float, 5>(A, nodes, own, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace hyb
