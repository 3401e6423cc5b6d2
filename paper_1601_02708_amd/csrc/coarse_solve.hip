// The coarse solve in one launch: right-preconditioned BiCGSTAB on (A P) y = r0
// (the recurrences, the shadow residual and the stop test of coarse_kernels.hip)
// with the mesh cut into tiles of 17 x 17 nodes, one workgroup each, for meshes
// of up to 64 tiles (M <= 135).
//
// Bound: latency.  An iteration is two stencil products of a few hundred
// thousand multiply-adds and two sums over the mesh; as two kernels (one per
// sum) it took 11-20 us, nearly all of it launch, drain and first loads, and the
// host had to enqueue iterations for the worst case.  Here a row's operator
// coefficients (49 doubles) and its entries of all Krylov vectors stay in the
// registers of one lane from the first product to the last, neighbours' entries
// of the one vector a product reads come through LDS, and what crosses
// workgroups -- three rings of that vector and two to four partial sums -- goes
// through global memory once per product.  Per solve (seven iterations, kernel
// trace): M = 16 30 us against 110 us of kernels, M = 64 55 against 135, M = 128
// beside a sweep 86 against 180; then 3.5 us less (M = 16) and 5.5 us less (M = 64,
// 128) from a row pitch free of bank conflicts, barriers that do not wait for
// published words and first loads asked for at once.  What is left, in cycles of a
// phase: the product 1000-1600 (49 LDS reads a row), the sums 1500, and between
// workgroups 2500-4500 from publishing a word to seeing it on another XCD; before
// the first phase some 8000 for cold instructions, operands and coefficients.
//
// Between workgroups: every double is published as two 64-bit words, each half
// of it under a 32-bit tag that names the launch and the phase, written and
// polled with agent-scope relaxed atomics.  A word is one atomic access and
// carries its own tag, so a reader needs no fence and no flag, and a word left
// over from an earlier phase or launch is never taken for the expected one.
// What orders the writing of a word over what it held: a workgroup gives its sums
// of a phase after it has collected everything of the phase before, and goes on
// only with everyone's sums.  So whoever has the sums of a phase may write what was
// collected before they were given -- the words of the phase before -- but not what
// is collected beside them: r0, s and t go through vec_at[0] and v through
// vec_at[1] in turn, and y, published behind the last sums of B, whose v others
// may still be waiting for, through vec_at[0].
//
// A wait ends after c.polls polls (some seconds: a workgroup that cannot become
// resident beside the others).  Whether the launch is given up is settled once for
// all its workgroups: the first that gives up, or that has its part of the result,
// says so in one word, and the others follow it.  Once a workgroup has its part,
// everyone has given all that is still waited for, so a wait goes on; once one has
// given up, none stores a result, and the last to end solves alone, from the same
// inputs.  It sets `lost`, after which the host takes the kernels of
// coarse_kernels.hip.
#include "hyb_impl.h"

namespace hyb {
namespace {

// kX: row pitch of the vector in LDS, 17 modulo the 32 doubles of the banks, so that
// the 17-node rows one wavefront reads follow each other through the banks (at a
// pitch of 23 half the reads met in a bank: 1900 cycles a product against 1000)
constexpr int kT = kSolveTile, kX = kT + 32, kF = kT + 2 * kCoarseHalo, kRows = kT * kT, kRing = kF * kF - kRows;
constexpr int kLanes = 384, kWaves = kLanes / 64;
constexpr int kSumWave = kWaves - 1;       // polls the partial sums (no ring node of its own)
static_assert(kRows <= kLanes && kRing <= kSumWave * 64 && kSolveTiles <= 64, "one row, one ring node, one tile a lane");
static_assert(kCoarseHalo == kApW / 2, "ring of the operator's radius");

typedef unsigned long long Word;

__device__ __forceinline__ void publish(Word *at, double x, unsigned tag) {
    const Word b = __builtin_bit_cast(Word, x), t = static_cast<Word>(tag) << 32;
    __hip_atomic_store(at, t | (b & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(at + 1, t | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned uniform(unsigned x) {
    return static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(x)));
}

__device__ __forceinline__ double uniform(double x) {
    const Word w = __builtin_bit_cast(Word, x);
    const Word high = uniform(static_cast<unsigned>(w >> 32));
    return __builtin_bit_cast(double, high << 32 | uniform(static_cast<unsigned>(w)));
}

// How a launch ends: the word at `at` holds 2 launch + 1 once it is given up, 2 launch
// once a workgroup has its part of the result, else an earlier launch's (`before`).
struct Ending {
    Word *at;
    Word before, launch;
    int polls;
};

// Settles it, unless another has: whether the launch is given up.
__device__ __forceinline__ bool given_up(const Ending &e, bool lost) {
    Word now = e.before;
    if (now >> 1 != e.launch &&
        __hip_atomic_compare_exchange_strong(e.at, &now, 2 * e.launch + (lost ? 1 : 0), __ATOMIC_RELAXED,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        return lost;
    return now & 1;
}

// the NV doubles at `at` once all carry the tag; false: the launch is given up
template <int NV>
__device__ __forceinline__ bool collect(const Word *at, unsigned tag, double (&x)[NV], const Ending &e) {
    for (unsigned n = 0;; ++n) {
        if (n == static_cast<unsigned>(e.polls)) {
            if (given_up(e, true)) return false;
        } else if ((n & 1023u) == 1023u) {
            if (__hip_atomic_load(e.at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 2 * e.launch + 1) return false;
        }
        Word w[2 * NV];
#pragma unroll
        for (int k = 0; k < 2 * NV; ++k) w[k] = __hip_atomic_load(at + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool all = true;
#pragma unroll
        for (int k = 0; k < 2 * NV; ++k) all = all && static_cast<unsigned>(w[k] >> 32) == tag;
        if (all) {
#pragma unroll
            for (int v = 0; v < NV; ++v)
                x[v] = __builtin_bit_cast(double, (w[2 * v] & 0xffffffffull) | (w[2 * v + 1] << 32));
            return true;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// Barrier for what goes through LDS: published words are not waited for, which
// __syncthreads would do (about 1200 cycles a product).
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Sum over the wavefront, in lane 63: lane shifts within rows of sixteen, then
// the row totals (no LDS round trips, which cost ds_bpermute ~100 cycles each).
template <int CTRL, int ROWS>
__device__ __forceinline__ double add_lanes(double x) {
    struct Two {
        int lo, hi;
    };
    Two w = __builtin_bit_cast(Two, x);
    w.lo = __builtin_amdgcn_update_dpp(0, w.lo, CTRL, ROWS, 0xf, true);
    w.hi = __builtin_amdgcn_update_dpp(0, w.hi, CTRL, ROWS, 0xf, true);
    return x + __builtin_bit_cast(double, w);
}
__device__ __forceinline__ double wave_total(double x) {
    x = add_lanes<0x111, 0xf>(x);          // row_shr:1, 2, 4, 8: lane 15 of a row has its total
    x = add_lanes<0x112, 0xf>(x);
    x = add_lanes<0x114, 0xf>(x);
    x = add_lanes<0x118, 0xf>(x);
    x = add_lanes<0x142, 0xa>(x);          // row_bcast:15 into rows 1 and 3
    return add_lanes<0x143, 0xc>(x);       // row_bcast:31 into rows 2 and 3
}

// Dense part of the shadow residual: the MurmurHash3 32-bit finaliser of the
// node index, mapped to [-1, 1).
__device__ __forceinline__ double shadow_hash(int node) {
    unsigned x = static_cast<unsigned>(node) * 0x9E3779B9u + 0x7F4A7C15u;
    x ^= x >> 16;
    x *= 0x85EBCA6Bu;
    x ^= x >> 13;
    x *= 0xC2B2AE35u;
    x ^= x >> 16;
    return double(x) * (2.0 / 4294967296.0) - 1.0;
}

// The solve of a launch that was given up, by one workgroup: the recurrences of
// coarse_kernels.hip on the vectors in global memory, every lane a row in kLanes.
template <bool GIVEN>
__device__ __forceinline__ void solve_alone(const CoarseDev &c, const double *given, double *out, int extrapolate,
                                            int max_iter, double tol, double (*red)[4]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, m1 = c.M + 1;
    auto place = [&](int node) { return (node / m1 + kCoarseHalo) * c.S + node % m1 + kCoarseHalo; };
    auto start = [&](int p) { return extrapolate ? 2.0 * c.xn[p] - c.xprev[p] : c.x1[p]; };
    auto product = [&](const double *x, int node, int p) {
        double a = 0.0;
        for (int o = 0; o < kApW * kApW; ++o)
            a += c.AP[(size_t)node * (kApW * kApW) + o] * x[p + (o / kApW - kCoarseHalo) * c.S + o % kApW - kCoarseHalo];
        return a;
    };
    auto sum = [&](auto &v) {
        constexpr int NV = sizeof(v) / sizeof(double);
        __syncthreads();
        for (int k = 0; k < NV; ++k) {
            const double x = wave_total(v[k]);
            if (lane == 63) red[wave][k] = x;
        }
        __syncthreads();
        for (int k = 0; k < NV; ++k) {
            v[k] = 0.0;
            for (int w = 0; w < kWaves; ++w) v[k] += red[w][k];
        }
    };
    double first[3] = {0.0, 0.0, 0.0};
    for (int node = tid; node < c.n; node += kLanes) {
        const int p = place(node);
        double r, b = 0.0;
        if (GIVEN) {
            r = b = given[p];
        } else {
            double ax = 0.0;
            for (int o = 0; o < 9; ++o) {
                const int q = p + (o / 3 - 1) * c.S + o % 3 - 1;
                ax += c.A9[(size_t)o * c.n + node] * start(q);
                b += c.B9[(size_t)o * c.n + node] * c.xn[q];
            }
            const int kind = c.dkind[node];
            if (kind != -1) b = c.A9[(size_t)4 * c.n + node] * (kind == -2 ? c.outer_value : c.ufc[kind]);
            r = b - ax;
        }
        c.r[p] = r;
        c.p[p] = c.v[p] = c.z[p] = c.y[p] = 0.0;
        first[0] += b * b;
        first[1] += r * r;
        first[2] += shadow_hash(node) * r;
    }
    sum(first);
    const double bnorm = sqrt(first[0]), scale = bnorm > 0.0 ? bnorm : 1.0, gamma = sqrt(first[1] / c.n);
    double rho = first[1] + gamma * first[2], alpha = 1.0, omega = 0.0, beta = 0.0, rnorm;
    bool breakdown = false;
    int k = 0;
    for (;; ++k) {
        // r is there, and every lane's vectors (sum's barriers)
        double two[2] = {0.0, 0.0};
        for (int node = tid; node < c.n; node += kLanes) {
            const int p = place(node);
            const double r = c.r[p], w = product(c.r, node, p), v = c.v[p];
            if (k == 0) c.rh[p] = r + gamma * shadow_hash(node);
            c.p[p] = r + beta * (c.p[p] - omega * v);
            c.w[p] = w;
            c.v[p] = w + beta * (v - omega * c.z[p]);
            two[0] += c.rh[p] * c.v[p];
            two[1] += r * r;
        }
        sum(two);
        rnorm = sqrt(two[1]);
        if (rnorm <= tol * scale || breakdown || k >= max_iter || !(rnorm == rnorm)) break;
        alpha = rho / two[0];
        double four[4] = {0.0, 0.0, 0.0, 0.0};
        for (int node = tid; node < c.n; node += kLanes) {
            const int p = place(node);
            const double z = product(c.v, node, p), s = c.r[p] - alpha * c.v[p], t = c.w[p] - alpha * z;
            c.z[p] = z;
            c.s[p] = s;
            c.t[p] = t;
            four[0] += t * s;
            four[1] += t * t;
            four[2] += c.rh[p] * s;
            four[3] += c.rh[p] * t;
        }
        sum(four);
        omega = four[1] > 0.0 ? four[0] / four[1] : 0.0;
        const double next = four[2] - omega * four[3];
        breakdown = omega == 0.0 || next == 0.0;
        beta = breakdown ? 0.0 : (next / rho) * (alpha / omega);
        rho = next;
        for (int node = tid; node < c.n; node += kLanes) {
            const int p = place(node);
            c.y[p] += alpha * c.p[p] + omega * c.s[p];
            c.r[p] = c.s[p] - omega * c.t[p];
        }
        __syncthreads();
    }
    for (int node = tid; node < c.n; node += kLanes) {
        const int p = place(node);
        double x = GIVEN ? c.y[p] : start(p);
        if (!GIVEN)
            for (int o = 0; o < kSpaiW * kSpaiW; ++o)
                x += c.P[(size_t)o * c.n + node] * c.y[p + (o / kSpaiW - kSpaiRadius) * c.S + o % kSpaiW - kSpaiRadius];
        out[p] = x;
    }
    if (tid == 0) {
        c.result->iters = k;
        c.result->converged = rnorm <= tol * scale ? 1 : 0;
        c.result->relres = rnorm / scale;
        c.result->lost = 1;
    }
}

// GIVEN: r0 is a given vector, the guess 0 and the result y itself (a solve
// with c.AP); else r0 = b - A guess of the trapezoidal step, and the result
// guess + P y.
template <bool GIVEN>
__global__ void __launch_bounds__(kLanes) coarse_solve_kernel(CoarseDev c, const double *__restrict__ given,
                                                              double *__restrict__ out, int tiles_x, int extrapolate,
                                                              int max_iter, double tol) {
    // (one of each for either product, so that a phase may write its own while
    // others still read the other one's)
    __shared__ double X[2][kF * kX];
    __shared__ double red[2][kWaves][4];
    __shared__ double tot[4];
    __shared__ int lost, arrived;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m1 = c.M + 1, nb = gridDim.x;
    const int k0 = (blockIdx.x % tiles_x) * kT, l0 = (blockIdx.x / tiles_x) * kT;
    // this lane's row
    const int dk = tid % kT, dl = tid / kT;
    const bool row = tid < kRows && k0 + dk < m1 && l0 + dl < m1;
    const int node = row ? (l0 + dl) * m1 + k0 + dk : 0;
    const int pi = (node / m1 + kCoarseHalo) * c.S + (node % m1 + kCoarseHalo);
    const int xi = (dl + kCoarseHalo) * kX + dk + kCoarseHalo;
    const bool shown = row && nb > 1 && (dk < kCoarseHalo || dl < kCoarseHalo || dk >= kT - kCoarseHalo || dl >= kT - kCoarseHalo);
    // and its ring node
    int rk, rl;
    if (tid < 2 * kCoarseHalo * kF) {
        rk = tid % kF;
        rl = tid / kF;
        if (rl >= kCoarseHalo) rl += kT;
    } else {
        const int e = tid - 2 * kCoarseHalo * kF, w = e % (2 * kCoarseHalo);
        rk = w < kCoarseHalo ? w : w + kT;
        rl = kCoarseHalo + e / (2 * kCoarseHalo);
    }
    const int gk = k0 + rk - kCoarseHalo, gl = l0 + rl - kCoarseHalo;
    const bool ring = tid < kRing && nb > 1 && gk >= 0 && gl >= 0 && gk < m1 && gl < m1;
    const int rnode = ring ? gl * m1 + gk : 0, ri = ring ? rl * kX + rk : 0;

    // words: the tag base, the launch's ending, who has given up, the partial sums of both phases, two published vectors
    Word *const base_at = c.words;
    Word *const sums_at[2] = {c.words + 16, c.words + 16 + kSolveTiles * 8};
    Word *const vec_at[2] = {c.words + 16 + kSolveTiles * 16, c.words + 16 + kSolveTiles * 16 + (size_t)4 * c.n};
    Word *const arrived_at = c.words + 2;
    const Word base = __hip_atomic_load(base_at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const Word before = __hip_atomic_load(c.words + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    if (tid == 0) lost = 0;
    for (int e = tid; e < 2 * kF * kX; e += kLanes) (&X[0][0])[e] = 0.0;
    // What r0 needs is asked for first and the coefficients behind it, all at once:
    // they are cold, and each wait in a row costs 1-2 us.
    constexpr int NX = GIVEN ? 1 : 9;
    double xn[NX], xg[NX], a9[NX], b9[NX];
    int kind = -1;
    if constexpr (GIVEN) {
        xn[0] = given[pi];
    } else {
        kind = c.dkind[node];
#pragma unroll
        for (int o = 0; o < 9; ++o) {
            const int p = pi + (o / 3 - 1) * c.S + (o % 3 - 1);
            xn[o] = c.xn[p];
            xg[o] = extrapolate ? c.xprev[p] : c.x1[p];
            a9[o] = c.A9[(size_t)o * c.n + node];
            b9[o] = c.B9[(size_t)o * c.n + node];
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    double ap[kApW * kApW];
#pragma unroll
    for (int o = 0; o < kApW * kApW; ++o) ap[o] = c.AP[(size_t)node * (kApW * kApW) + o];
    __builtin_amdgcn_sched_barrier(0);
    // a word of X is cleared by another wavefront than the one that fills it below
    lds_barrier();
    // (in scalar registers, as all that is the same in every lane: the coefficients leave no others)
    unsigned tag = uniform(static_cast<unsigned>(base)) + 1u;
    const Word high = uniform(static_cast<unsigned>(before >> 32));
    const Ending end{c.words + 1, high << 32 | uniform(static_cast<unsigned>(before)), tag, c.polls};

    auto product = [&](const double *x) {
        double s[kApW];
#pragma unroll
        for (int a = 0; a < kApW; ++a) {
            s[a] = 0.0;
#pragma unroll
            for (int b = 0; b < kApW; ++b)
                s[a] += ap[a * kApW + b] * x[(dl + a) * kX + dk + b];
            // two stencil rows of reads in flight: more would not fit the
            // registers beside the coefficients
            if (a & 1) __builtin_amdgcn_sched_barrier(0);
        }
        return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + s[6]);
    };
    // Partial sums of this workgroup into red[ph] (and to the others); ends behind a barrier.
    auto give_sums = [&](auto &v, int ph) {
        constexpr int NV = sizeof(v) / sizeof(double);
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const double x = wave_total(v[k]);
            if (lane == 63) red[ph][wave][k] = x;
        }
        lds_barrier();
        if (nb > 1 && tid < NV) {
            double x = 0.0;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) x += red[ph][w][tid];
            publish(sums_at[ph] + (size_t)blockIdx.x * 8 + 2 * tid, x, tag);
        }
    };
    // Sums over the mesh into v: the same operations in every workgroup.  A lone
    // one adds its wavefronts' sums in every lane, without a further barrier.
    auto take_sums = [&](auto &v, int ph) {
        constexpr int NV = sizeof(v) / sizeof(double);
        if (nb > 1) {
            const Word *at = sums_at[ph];
            if (wave == kSumWave) {
                double x[NV];
#pragma unroll
                for (int k = 0; k < NV; ++k) x[k] = 0.0;
                if (lane < nb && !collect<NV>(at + (size_t)lane * 8, tag, x, end)) lost = 1;
#pragma unroll
                for (int k = 0; k < NV; ++k) {
                    const double y = wave_total(x[k]);
                    if (lane == 63) tot[k] = y;
                }
            }
            lds_barrier();
#pragma unroll
            for (int k = 0; k < NV; ++k) v[k] = tot[k];
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                v[k] = 0.0;
#pragma unroll
                for (int w = 0; w < kWaves; ++w) v[k] += red[ph][w][k];
            }
        }
    };

    // ---- r0 --------------------------------------------------------------
    double r = 0.0, guess = 0.0;
    double first[3] = {0.0, 0.0, 0.0};
    if (row) {
        double b;
        if constexpr (GIVEN) {
            r = xn[0];
            b = r;
        } else {
            double sa = 0.0, sb = 0.0;
#pragma unroll
            for (int o = 0; o < 9; ++o) {
                // the guess: x1 as it stands, or 2 xn - xprev
                const double x = extrapolate ? 2.0 * xn[o] - xg[o] : xg[o];
                if (o == 4) guess = x;
                sa += a9[o] * x;
                sb += b9[o] * xn[o];
            }
            b = kind == -1 ? sb : a9[4] * (kind == -2 ? c.outer_value : c.ufc[kind]);
            r = b - sa;
        }
        first[0] = b * b;
        first[1] = r * r;
        first[2] = shadow_hash(node) * r;
        X[0][xi] = r;
        if (shown) publish(vec_at[0] + (size_t)4 * node, r, tag);
    }
    give_sums(first, 0);

    double p = 0.0, v = 0.0, s = 0.0, t = 0.0, w = 0.0, z = 0.0, y = 0.0, rh = 0.0;
    double rho = 1.0, inv_rho = 1.0, alpha = 1.0, bnorm = 0.0, rnorm = 0.0;
    int iters = 0;
    double met = 0.0, y_met = 0.0;
    bool converged = false, gone = false;
    for (int k = 0;; ++k) {
        // ---- A(k): finish iteration k-1, w = A P r, p, v = A P p ----------
        bool breakdown = false;
        double omega = 0.0, beta = 0.0, ring_x[2] = {0.0, 0.0};
        if (k == 0) {
            double one[1] = {0.0};
            if (ring && !collect<1>(vec_at[0] + (size_t)4 * rnode, tag, one, end)) lost = 1;
            if (ring) X[0][ri] = one[0];
            take_sums(first, 0);
            bnorm = uniform(sqrt(first[0]));
            const double gamma = sqrt(first[1] / c.n);
            rho = uniform(first[1] + gamma * first[2]);
            rh = r + gamma * shadow_hash(node);
        } else {
            double four[4];
            if (ring && !collect<2>(vec_at[0] + (size_t)4 * rnode, tag, ring_x, end)) lost = 1;
            take_sums(four, 0);
            // (1 / omega and 1 / rho_{k-1} on their own: one division deep)
            omega = four[1] > 0.0 ? four[0] / four[1] : 0.0;
            const double inv_omega = four[1] / four[0];
            const double next = four[2] - omega * four[3];
            breakdown = omega == 0.0 || next == 0.0;
            beta = breakdown ? 0.0 : (next * inv_rho) * (alpha * inv_omega);
            rho = uniform(next);
            r = s - omega * t;
            y += alpha * p + omega * s;
            if (row) X[0][xi] = r;
            if (ring) X[0][ri] = ring_x[0] - omega * ring_x[1];
            lds_barrier();
        }
        gone = lost;
        if (gone) break;
        ++tag;
        double two[2] = {0.0, 0.0};
        if (row) {
            w = product(X[0]);
            p = r + beta * (p - omega * v);
            v = w + beta * (v - omega * z);
            two[0] = rh * v;
            two[1] = r * r;
            X[1][xi] = v;
            if (shown) publish(vec_at[1] + (size_t)4 * node, v, tag);
        }
        give_sums(two, 1);
        // ---- B(k): stop test, z = A P v, s, t ------------------------------
        double one[1] = {0.0};
        if (ring && !collect<1>(vec_at[1] + (size_t)4 * rnode, tag, one, end)) lost = 1;
        if (ring) X[1][ri] = one[0];
        take_sums(two, 1);
        gone = lost;
        if (gone) break;
        rnorm = sqrt(two[1]);
        iters = k;
        // An iterate that meets the tolerance by less than a factor of two gets one
        // iteration more: which one first meets a tolerance this near the rounding
        // of r0 is a matter of the order of the sums, and the next (3-6 us, in few
        // solves) is worth a digit.  If it is not better, the first is the result.
        const double scale = bnorm > 0.0 ? bnorm : 1.0;
        if (converged || rnorm <= 0.5 * tol * scale || breakdown || k >= max_iter || !(rnorm == rnorm)) {
            if (converged && !(rnorm <= met)) {
                y = y_met;
                rnorm = met;
                iters = k - 1;
            }
            converged = rnorm <= tol * scale;
            break;
        }
        if (rnorm <= tol * scale) {
            converged = true;
            met = uniform(rnorm);
            y_met = y;
        }
        alpha = uniform(rho / two[0]);
        inv_rho = uniform(1.0 / rho);
        ++tag;
        double four[4] = {0.0, 0.0, 0.0, 0.0};
        if (row) {
            z = product(X[1]);
            s = r - alpha * v;
            t = w - alpha * z;
            four[0] = t * s;
            four[1] = t * t;
            four[2] = rh * s;
            four[3] = rh * t;
            if (shown) {
                publish(vec_at[0] + (size_t)4 * node, s, tag);
                publish(vec_at[0] + (size_t)4 * node + 2, t, tag);
            }
        }
        give_sums(four, 0);
    }

    // ---- the result ---------------------------------------------------------
    ++tag;
    // (a wavefront without ring nodes, beside those that wait for theirs)
    if (nb > 1 && !gone && tid == kSumWave * 64 && given_up(end, false)) lost = 1;
    if constexpr (!GIVEN) {
        double one[1] = {0.0};
        if (shown) publish(vec_at[0] + (size_t)4 * node, y, tag);
        if (ring && !gone && !collect<1>(vec_at[0] + (size_t)4 * rnode, tag, one, end)) lost = 1;
        // (every read of X[0] came before the last sums)
        if (row) X[0][xi] = y;
        if (ring) X[0][ri] = one[0];
    }
    lds_barrier();
    if (lost) {
        if (tid == 0)
            arrived = static_cast<int>(__hip_atomic_fetch_add(arrived_at, Word(1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        __syncthreads();
        if (arrived != nb - 1) return;
        if (tid == 0) {
            // (a workgroup may be a phase ahead of this one)
            __hip_atomic_store(arrived_at, Word(0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(base_at, static_cast<Word>(tag + 4u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // (the arguments read anew: kept from the start they would not fit the registers)
        const CoarseDev *again = (const CoarseDev *)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(again));
        solve_alone<GIVEN>(*again, given, out, extrapolate, max_iter, tol, red[0]);
        return;
    }
    if (row) {
        if constexpr (GIVEN) {
            out[pi] = y;
        } else {
            double acc = 0.0;
#pragma unroll
            for (int o = 0; o < kSpaiW * kSpaiW; ++o)
                acc += c.P[(size_t)o * c.n + node] *
                       X[0][xi + (o / kSpaiW - kSpaiRadius) * kX + (o % kSpaiW - kSpaiRadius)];
            out[pi] = guess + acc;
        }
    }
    if (blockIdx.x == 0 && tid == 0) {
        c.result->iters = iters;
        c.result->converged = converged ? 1 : 0;
        c.result->relres = bnorm > 0.0 ? rnorm / bnorm : rnorm;
        if (GIVEN) c.result->lost = 0;     // (else it sticks: a step has several solves)
        // (every workgroup has read the base: it took part in a later phase)
        __hip_atomic_store(base_at, static_cast<Word>(tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace

size_t coarse_solve_words(int n) { return 16 + (size_t)kSolveTiles * 16 + (size_t)8 * n; }

bool coarse_solve_fits(int M) {
    const int t = (M + 1 + kSolveTile - 1) / kSolveTile;
    return t * t <= kSolveTiles;
}

hipError_t launch_coarse_solve_one(const CoarseDev &c, bool extrapolate, int max_iter, double tol, hipStream_t s) {
    const int t = (c.M + 1 + kSolveTile - 1) / kSolveTile;
    hipLaunchKernelGGL((coarse_solve_kernel<false>), dim3(t * t), dim3(kLanes), 0, s, c, nullptr, c.x1, t,
                       extrapolate ? 1 : 0, max_iter, tol);
    return hipGetLastError();
}

hipError_t launch_coarse_solve_given_one(const CoarseDev &c, const double *rhs, double *out, int max_iter, double tol,
                                         hipStream_t s) {
    const int t = (c.M + 1 + kSolveTile - 1) / kSolveTile;
    hipLaunchKernelGGL((coarse_solve_kernel<true>), dim3(t * t), dim3(kLanes), 0, s, c, rhs, out, t, 0, max_iter, tol);
    return hipGetLastError();
}

}  // namespace hyb
