// The one-launch coarse solve (coarse_solve.hip, included as KERNEL) on the CPU
// under chosen orders of its wavefronts; argv: elements a side, random orders, polls
// of a wait before it is given up, most iterations, tolerance, size of a part of the
// matrix that is not symmetric.  Prints a line per solve: the order, the
// solve, converged, lost, iterations, the true residual over ||b||, a hash of the
// solution, the residual that the solve reports.
#include <cstdio>
#include <random>
#include <string>

#include KERNEL

// ---- lanes as fibers (x86-64) ------------------------------------------------
extern "C" void switch_stack(void **save, void *to);
asm(R"(
.text
.globl switch_stack
switch_stack:
    pushq %rbp
    pushq %rbx
    pushq %r12
    pushq %r13
    pushq %r14
    pushq %r15
    movq %rsp, (%rdi)
    movq %rsi, %rsp
    popq %r15
    popq %r14
    popq %r13
    popq %r12
    popq %rbx
    popq %rbp
    ret
)");

extern char __start_workgroup_memory, __stop_workgroup_memory;

namespace emulated {

Lane *lane = nullptr;
unsigned blocks = 0;
long long stores = 0;
const void *arguments = nullptr;
std::function<size_t(const std::vector<Wave> &)> policy;

static void *scheduler = nullptr;
static const std::function<void()> *kernel = nullptr;
static std::vector<Lane> lanes_of;
static unsigned lanes_a_block = 0;

void wait(Wait w) {
    lane->wait = w;
    lane->seen = stores;
    switch_stack(&lane->sp, scheduler);
}

static void lane_main() {
    (*kernel)();
    wait(kDone);
}

int from_lane(int old, int x, int ctrl, int row_mask) {
    Lane *const me = lane;
    const int turn = me->turn ^= 1, at = static_cast<int>(me->thread.x) & 63, row = at >> 4;
    me->put[turn] = x;
    wait(kWave);
    const Lane *wave = me - at;
    if (!((row_mask >> row) & 1)) return old;
    if (ctrl > 0x110 && ctrl < 0x120) {
        const int n = ctrl - 0x110;
        return (at & 15) >= n ? wave[at - n].put[turn] : 0;
    }
    if (ctrl == 0x142) return row > 0 ? wave[16 * row - 1].put[turn] : old;
    if (ctrl == 0x143) return row > 1 ? wave[31].put[turn] : old;
    std::abort();
}

void run_grid(unsigned grid, unsigned lanes, const std::function<void()> &body) {
    const size_t kStack = 48 << 10, bytes = &__stop_workgroup_memory - &__start_workgroup_memory;
    const int waves = static_cast<int>(lanes / 64);
    blocks = grid;
    lanes_a_block = lanes;
    kernel = &body;
    lanes_of.resize((size_t)grid * lanes);
    std::vector<std::vector<char>> memory(grid, std::vector<char>(bytes, (char)0xa5));
    for (size_t n = 0; n < lanes_of.size(); ++n) {
        Lane &l = lanes_of[n];
        l.stack.resize(kStack);
        l.wait = kReady;
        l.thread = dim3(n % lanes);
        l.block = dim3(n / lanes);
        void **sp = reinterpret_cast<void **>((reinterpret_cast<uintptr_t>(l.stack.data() + kStack) & ~uintptr_t(15)) - 8);
        *--sp = reinterpret_cast<void *>(lane_main);
        for (int r = 0; r < 6; ++r) *--sp = nullptr;
        l.sp = sp;
    }
    int loaded = -1;
    for (;;) {
        // wavefronts that can go on, else those that poll
        std::vector<Wave> ready, polling;
        for (unsigned b = 0; b < grid; ++b)
            for (int w = 0; w < waves; ++w) {
                bool go = false, poll = false;
                for (int e = 0; e < 64; ++e) {
                    const Lane &l = lanes_of[(size_t)b * lanes + 64 * w + e];
                    go = go || l.wait == kReady || (l.wait == kPolled && l.seen != stores);
                    poll = poll || l.wait == kPolled;
                }
                if (go) ready.push_back({(int)b, w});
                else if (poll) polling.push_back({(int)b, w});
            }
        if (ready.empty() && polling.empty()) break;
        const std::vector<Wave> &from = ready.empty() ? polling : ready;
        const Wave next = from[policy(from)];
        if (loaded != next.block) {
            if (loaded >= 0) std::memcpy(memory[loaded].data(), &__start_workgroup_memory, bytes);
            std::memcpy(&__start_workgroup_memory, memory[next.block].data(), bytes);
            loaded = next.block;
        }
        Lane *const first = &lanes_of[(size_t)next.block * lanes], *const wave = first + 64 * next.wave;
        // the wavefront, until each of its lanes waits
        for (bool again = true; again;) {
            again = false;
            int at = 0, live = 0;
            for (int e = 0; e < 64; ++e) {
                Lane &l = wave[e];
                if (l.wait == kReady || (l.wait == kPolled && !again && (ready.empty() || l.seen != stores))) {
                    l.wait = kReady;
                    lane = &l;
                    switch_stack(&scheduler, l.sp);
                }
                live += l.wait != kDone;
                at += l.wait == kWave;
            }
            if (live && at == live) {
                for (int e = 0; e < 64; ++e)
                    if (wave[e].wait == kWave) wave[e].wait = kReady;
                again = true;
            }
        }
        // a barrier that every live lane of the workgroup has reached
        unsigned at = 0, live = 0;
        for (unsigned e = 0; e < lanes; ++e) {
            live += first[e].wait != kDone;
            at += first[e].wait == kBarrier;
        }
        if (live && at == live)
            for (unsigned e = 0; e < lanes; ++e)
                if (first[e].wait == kBarrier) first[e].wait = kReady;
    }
    for (const Lane &l : lanes_of)
        if (l.wait != kDone) {
            std::printf("a lane never ended\n");
            std::exit(2);
        }
}

}  // namespace emulated

// ---- a system to solve -------------------------------------------------------
using namespace hyb;

struct Mesh {
    int M, m1, n, S;
    std::vector<double> A9, B9, AP, P, ufc, vec[12], rhs, out;
    std::vector<int> dkind;
    std::vector<unsigned long long> words;
    KrylovResult result{};
    CoarseDev c{};
    double *base(int v) { return vec[v].data(); }
    int pad(int k, int l) const { return (l + kCoarseHalo) * S + k + kCoarseHalo; }

    Mesh(int M_, double skew) : M(M_), m1(M_ + 1), n(m1 * m1), S(m1 + 2 * kCoarseHalo) {
        std::mt19937 gen(M);
        auto rnd = [&] { return gen() / 4294967296.0; };
        A9.assign(9 * (size_t)n, 0.0);
        B9 = A9;
        P.assign(25 * (size_t)n, 0.0);
        AP.assign(49 * (size_t)n, 0.0);
        dkind.assign(n, -1);
        auto in = [&](int k, int l) { return k >= 0 && l >= 0 && k < m1 && l < m1; };
        for (int l = 0; l < m1; ++l)
            for (int k = 0; k < m1; ++k) {
                const int node = l * m1 + k;
                const bool edge = k == 0 || l == 0 || k == M || l == M;
                const bool inner = M >= 8 && k == M / 2 && l == M / 2;
                if (edge) dkind[node] = -2;
                if (inner) dkind[node] = 0;
                for (int o = 0; o < 9; ++o) {
                    if (!in(k + o % 3 - 1, l + o / 3 - 1)) continue;
                    A9[(size_t)o * n + node] = o == 4 ? 1.0 + 0.5 * rnd() : edge || inner ? 0.0 : -0.1 * rnd() + (skew != 0.0 ? skew * (rnd() - 0.5) : 0.0);
                    B9[(size_t)o * n + node] = 0.2 * rnd();
                }
                for (int o = 0; o < 25; ++o)
                    if (in(k + o % 5 - 2, l + o / 5 - 2)) P[(size_t)o * n + node] = o == 12 ? 0.8 + 0.2 * rnd() : 0.02 * rnd();
            }
        for (int l = 0; l < m1; ++l)
            for (int k = 0; k < m1; ++k)
                for (int o = 0; o < 9; ++o) {
                    const int k2 = k + o % 3 - 1, l2 = l + o / 3 - 1;
                    if (!in(k2, l2)) continue;
                    for (int q = 0; q < 25; ++q)
                        AP[(size_t)(l * m1 + k) * 49 + (o / 3 - 1 + q / 5 - 2 + 3) * 7 + o % 3 - 1 + q % 5 - 2 + 3] +=
                            A9[(size_t)o * n + l * m1 + k] * P[(size_t)q * n + l2 * m1 + k2];
                }
        ufc.assign(1, 0.7);
        for (auto &v : vec) v.assign((size_t)S * S, 0.0);
        rhs.assign((size_t)S * S, 0.0);
        out.assign((size_t)S * S, 0.0);
        for (int l = 0; l < m1; ++l)
            for (int k = 0; k < m1; ++k) {
                vec[0][pad(k, l)] = rnd();
                vec[1][pad(k, l)] = rnd();
                vec[11][pad(k, l)] = rnd();
                rhs[pad(k, l)] = rnd() - 0.5;
            }
        words.assign(coarse_solve_words(n), 0ull);
        c.M = M;
        c.n = n;
        c.S = S;
        c.A9 = A9.data();
        c.B9 = B9.data();
        c.AP = AP.data();
        c.P = P.data();
        c.dkind = dkind.data();
        c.outer_value = 0.2;
        c.ufc = ufc.data();
        double **at[] = {&c.xn, &c.x1, &c.r, &c.rh, &c.p, &c.v, &c.s, &c.t, &c.y, &c.w, &c.z, &c.xprev};
        for (int v = 0; v < 12; ++v) *at[v] = vec[v].data();
        c.result = &result;
        c.words = words.data();
    }

    // ||b - A x1|| / ||b||, or that of (A P) out = rhs
    double residual(bool given) const {
        double rr = 0.0, bb = 0.0;
        for (int l = 0; l < m1; ++l)
            for (int k = 0; k < m1; ++k) {
                const int node = l * m1 + k, W = given ? 7 : 3;
                double b = 0.0, ax = 0.0;
                for (int o = 0; o < W * W; ++o) {
                    const int p = pad(k, l) + (o / W - W / 2) * S + o % W - W / 2;
                    if (given) {
                        ax += AP[(size_t)node * 49 + o] * out[p];
                    } else {
                        ax += A9[(size_t)o * n + node] * c.x1[p];
                        b += B9[(size_t)o * n + node] * c.xn[p];
                    }
                }
                if (given) b = rhs[pad(k, l)];
                else if (dkind[node] != -1) b = A9[(size_t)4 * n + node] * (dkind[node] == -2 ? c.outer_value : ufc[0]);
                rr += (b - ax) * (b - ax);
                bb += b * b;
            }
        return std::sqrt(rr / bb);
    }
};

static unsigned long long hash_of(const double *x, size_t n) {
    unsigned long long h = 1469598103934665603ull;
    for (size_t e = 0; e < n; ++e) {
        unsigned long long w;
        std::memcpy(&w, x + e, 8);
        h = (h ^ w) * 1099511628211ull;
    }
    return h;
}

int main(int argc, char **argv) {
    if (argc < 4) return 2;
    const int max_iter = argc > 4 ? std::atoi(argv[4]) : 200;
    const double tol = argc > 5 ? std::atof(argv[5]) : 1e-14, skew = argc > 6 ? std::atof(argv[6]) : 0.0;
    const int M = std::atoi(argv[1]), seeds = std::atoi(argv[2]), polls = std::atoi(argv[3]);
    const int side = (M + 1 + kSolveTile - 1) / kSolveTile, nb = side * side;
    struct Order {
        std::string name;
        std::function<size_t(const std::vector<emulated::Wave> &)> pick;
    };
    std::vector<Order> orders;
    size_t turn = 0;
    orders.push_back({"first", [](const std::vector<emulated::Wave> &) { return size_t(0); }});
    orders.push_back({"last", [](const std::vector<emulated::Wave> &w) { return w.size() - 1; }});
    // one workgroup goes on only when no other can
    for (int late = 0; late < nb && nb > 1; ++late)
        orders.push_back({"late" + std::to_string(late), [late, &turn](const std::vector<emulated::Wave> &w) {
                              for (size_t e = 0; e < w.size(); ++e) {
                                  const size_t at = (turn + e) % w.size();
                                  if (w[at].block != late) return turn = at;
                              }
                              return size_t(0);
                          }});
    // ... or one wavefront of each
    for (int late = 0; late < 6; ++late)
        orders.push_back({"latewave" + std::to_string(late), [late](const std::vector<emulated::Wave> &w) {
                              for (size_t e = 0; e < w.size(); ++e)
                                  if (w[e].wave != late) return e;
                              return size_t(0);
                          }});
    std::mt19937 gen(1);
    for (int s = 0; s < seeds; ++s) orders.push_back({"random" + std::to_string(s), [&gen](const std::vector<emulated::Wave> &w) { return gen() % w.size(); }});
    for (const Order &o : orders) {
        Mesh m(M, skew);
        m.c.polls = polls;
        emulated::policy = o.pick;
        for (int solve = 0; solve < 3; ++solve) {
            const bool given = solve == 2;
            m.result.lost = 0;
            if (given) launch_coarse_solve_given_one(m.c, m.rhs.data(), m.out.data(), max_iter, tol, nullptr);
            else launch_coarse_solve_one(m.c, solve == 0, max_iter, tol, nullptr);
            std::printf("%s %d %d %d %d %.3e %016llx %.17e\n", o.name.c_str(), solve, m.result.converged, m.result.lost,
                        m.result.iters, m.residual(given), hash_of(given ? m.out.data() : m.c.x1, m.out.size()),
                        m.result.relres);
        }
    }
    return 0;
}
