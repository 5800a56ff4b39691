// Runs the on-chip preconditioner's kernel on the CPU under chosen orders of its
// wavefronts.  onchip_kernel.inc is resident.hip with its device-only syntax
// replaced (test_onchip_protocol.py).  Usage: onchip_emulation <scenario> <seed>;
// prints "ok" or what went wrong.
#include <hip/hip_runtime.h>

#include <ucontext.h>

#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <memory>
#include <mutex>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "onchip_kernel.inc"

namespace emu {
constexpr int kLanes = 64;
struct Lane {
    Here at;
    ucontext_t ctx;
    std::unique_ptr<char[]> stack;
    bool over = false;
    int line = 0;   // of the barrier it waits at, 0: none
    Kind kind = kWave;
    uint64_t value = 0;
    int arg = 0;
};
struct Wave {
    Lane lanes[kLanes];
    bool over = false;
    int line = 0;
};
struct Group {
    std::vector<std::unique_ptr<Wave>> waves;
    std::vector<unsigned char> lds;
    ucontext_t home;
};
thread_local Group *t_group = nullptr;
thread_local Lane *t_lane = nullptr;
std::string g_error;

void fail(const std::string &what) {
    if (g_error.empty()) g_error = what;
}
Here &here() { return t_lane->at; }
unsigned char *dynamic_lds() { return t_group->lds.data(); }
void stop_lane() { swapcontext(&t_lane->ctx, &t_group->home); }
void barrier(int line) {
    t_lane->line = line;
    stop_lane();
}
uint64_t cross(Kind kind, uint64_t v, int q) {
    t_lane->kind = kind;
    t_lane->value = v;
    t_lane->arg = q;
    stop_lane();
    return t_lane->value;
}

std::function<void()> g_kernel;
void lane_main() {
    g_kernel();
    t_lane->over = true;
    stop_lane();
}

// One wavefront from where it stands to its next cross-lane operation, barrier or end.
void slice(Group &g, Wave &w) {
    t_group = &g;
    // (the lanes at a tile's x edges first: LDS writes come before the same
    // wavefront's later reads, as they do in lockstep)
    for (int q = 0; q < kLanes; ++q) {
        t_lane = &w.lanes[q == 0 ? 0 : q == 1 ? kLanes - 1 : q - 1];
        swapcontext(&g.home, &t_lane->ctx);
    }
    uint64_t v[kLanes];
    for (int q = 0; q < kLanes; ++q) {
        const Lane &l = w.lanes[q], &l0 = w.lanes[0];
        if (l.over != l0.over || l.line != l0.line || l.kind != l0.kind) fail("lanes of a wavefront part");
        v[q] = l.value;
    }
    w.over = w.lanes[0].over;
    w.line = w.lanes[0].line;
    if (w.over || w.line) return;
    uint64_t all = 1;
    for (uint64_t x : v) all &= x;
    for (int q = 0; q < kLanes; ++q) {
        Lane &l = w.lanes[q];
        switch (l.kind) {
        case kShiftUp: l.value = q > 0 ? v[q - 1] : 0; break;
        case kShiftDown: l.value = q + 1 < kLanes ? v[q + 1] : 0; break;
        case kLane: l.value = v[l.arg]; break;
        case kXor: l.value = v[q ^ l.arg]; break;
        case kAnd: l.value = all; break;
        case kWave: break;
        }
    }
}
// Barriers that every running wavefront of the group has reached.
void release(Group &g) {
    int line = 0;
    bool ended = false;
    for (auto &w : g.waves) {
        ended = ended || w->over;
        if (w->over) continue;
        if (!w->line) return;
        if (line && line != w->line) fail("wavefronts of a workgroup meet at different barriers");
        line = w->line;
    }
    if (line && ended) fail("a barrier without the workgroup's other wavefronts, which have left");
    for (auto &w : g.waves) {
        w->line = 0;
        for (Lane &l : w->lanes) l.line = 0;
    }
}

// Runs `groups` workgroups of `waves` wavefronts; pick(group, wave of it) says
// whether a wavefront may go on now (if none may, all may).
void run(int groups, int waves, size_t lds, std::mt19937 &rng, const std::function<bool(int, int)> &pick) {
    std::vector<std::unique_ptr<Group>> gs;
    for (int b = 0; b < groups; ++b) {
        gs.push_back(std::make_unique<Group>());
        Group &g = *gs.back();
        g.lds.resize(lds);
        for (int y = 0; y < waves; ++y) {
            g.waves.push_back(std::make_unique<Wave>());
            for (int q = 0; q < kLanes; ++q) {
                Lane &l = g.waves.back()->lanes[q];
                l.at = Here{dim3(q, y, 0), dim3(b, 0, 0), dim3(kLanes, waves), dim3(groups)};
                l.stack.reset(new char[1 << 16]);
                getcontext(&l.ctx);
                l.ctx.uc_stack.ss_sp = l.stack.get();
                l.ctx.uc_stack.ss_size = 1 << 16;
                l.ctx.uc_link = nullptr;
                makecontext(&l.ctx, lane_main, 0);
            }
        }
    }
    // a workgroup's slices run on its own thread, whose thread-local variables are its LDS
    std::mutex mu;
    std::condition_variable cv;
    int turn = -1, wave = 0;
    bool over = false;
    std::vector<std::thread> threads;
    for (int b = 0; b < groups; ++b)
        threads.emplace_back([&, b] {
            std::unique_lock<std::mutex> lock(mu);
            for (;;) {
                cv.wait(lock, [&] { return over || turn == b; });
                if (over) return;
                slice(*gs[b], *gs[b]->waves[wave]);
                release(*gs[b]);
                turn = -1;
                cv.notify_all();
            }
        });
    {
        std::unique_lock<std::mutex> lock(mu);
        while (g_error.empty()) {
            std::vector<std::pair<int, int>> can, may;
            for (int b = 0; b < groups; ++b)
                for (int y = 0; y < waves; ++y) {
                    const Wave &w = *gs[b]->waves[y];
                    if (w.over || w.line) continue;
                    can.emplace_back(b, y);
                    if (pick(b, y)) may.emplace_back(b, y);
                }
            if (can.empty()) break;
            const auto &from = may.empty() ? can : may;
            std::tie(turn, wave) = from[rng() % from.size()];
            cv.notify_all();
            cv.wait(lock, [&] { return turn == -1; });
        }
        for (auto &g : gs)
            for (auto &w : g->waves)
                if (!w->over) fail("wavefronts wait for each other for ever");
        over = true;
        cv.notify_all();
    }
    for (auto &t : threads) t.join();
}
}  // namespace emu

using namespace cuth;

// Problems of `ntx` x 1 tiles of 64 x 8 columns, two layers.
struct Set {
    static constexpr int nz = 2, ny = 8, k = 5;
    int ntx, nprob;
    std::vector<LayerCoef<float>> lc;
    std::vector<CgState<float>> st;
    std::vector<InnerProb<float>> probs;
    std::vector<std::vector<float>> r, z;
    std::vector<float> cheb, part_in, part_out;
    std::vector<ResGroup> groups;
    std::vector<unsigned long long> words;
    std::vector<unsigned> epoch;

    Set(int ntx_, int nprob_) : ntx(ntx_), nprob(nprob_) {
        for (int l = 0; l < nz; ++l) lc.push_back(LayerCoef<float>{0.5f, 0.25f, l ? 1.0f : 0.f, l ? 0.f : 1.0f, 0.1f * l, 0.f, 1.f});
        cheb.assign(1 + 2 * 8, 0.f);
        cheb[0] = 0.3f;
        for (int j = 1; j < k; ++j) {
            cheb[1 + j] = 0.4f;
            cheb[1 + 8 + j] = 0.2f;
        }
        const size_t n = (size_t)ntx * 64 * ny * nz;
        st.resize(nprob);
        part_in.assign((size_t)nprob * ntx, 1.f);
        part_out.assign((size_t)nprob * ntx, 0.f);
        for (int p = 0; p < nprob; ++p) {
            r.emplace_back(n);
            z.emplace_back(n, 0.f);
            for (size_t c = 0; c < n; ++c) r[p][c] = (float)((c * 37 + p) % 101) - 50.f;
        }
        for (int p = 0; p < nprob; ++p) {
            st[p] = CgState<float>{};
            st[p].iter = 6;
            st[p].tol2 = 1e-3f;
            InnerProb<float> d{};
            d.op.nx = ntx * 64;
            d.op.ny = ny;
            d.op.nz = nz;
            d.op.lc = lc.data();
            d.tile0 = p * ntx;
            d.ntiles = ntx;
            d.r = r[p].data();
            d.z[1] = z[p].data();
            d.st = &st[p];
            d.cheb = cheb.data();
            d.kcap = 8;
            d.r_ntx = d.r_ntiles = ntx;
            probs.push_back(d);
            groups.push_back(ResGroup{p * ntx, p, 0, 1, 0, 0, ny, 0});
        }
        words.assign((size_t)2 * nprob * ntx * res_tile_words<float>(8, 1, 8), 0);
        epoch.assign((size_t)nprob * ntx, 1u);
    }
    void launch(int width, int spin, std::mt19937 &rng, const std::function<bool(int, int)> &pick) {
        ResArgs ra;
        ra.groups = groups.data();
        ra.one = groups[0];
        ra.buf = words.data();
        ra.epoch = epoch.data();
        ra.ngroups = nprob;
        ra.tiles = nprob * ntx;
        ra.width = width;
        ra.spin = spin;
        emu::g_kernel = [&, ra] {
            k_cheb_res<float, false, false, 8, 1, 8>(probs.data(), k, 1, 1, part_in.data(), 0, part_out.data(), ra);
        };
        emu::run(width, 8, res_lds<float>(8, 1, 8), rng, pick);
    }
    static bool marked(const CgState<float> &st) { return st.gave_up != 0; }
    // z of problem p against the recurrence in 64 bits
    void check(int p) {
        const int nx = ntx * 64;
        auto at = [&](int i, int j, int l) { return (size_t)i + (size_t)nx * (j + (size_t)ny * l); };
        std::vector<double> a(r[p].size()), b(r[p].size(), 0.0);
        for (size_t c = 0; c < a.size(); ++c) a[c] = (double)r[p][c] * cheb[0];
        for (int s = 1; s < k; ++s) {
            std::vector<double> o(a.size());
            for (int l = 0; l < nz; ++l)
                for (int j = 0; j < ny; ++j)
                    for (int i = 0; i < nx; ++i) {
                        const double x = a[at(i, j, l)];
                        double y = lc[l].sink * x;
                        if (i > 0) y += lc[l].gx * (x - a[at(i - 1, j, l)]);
                        if (i + 1 < nx) y += lc[l].gx * (x - a[at(i + 1, j, l)]);
                        if (j > 0) y += lc[l].gy * (x - a[at(i, j - 1, l)]);
                        if (j + 1 < ny) y += lc[l].gy * (x - a[at(i, j + 1, l)]);
                        y += l ? lc[l].gzd * (x - a[at(i, j, l - 1)]) : lc[l].gzu * (x - a[at(i, j, l + 1)]);
                        const size_t c = at(i, j, l);
                        o[c] = x + cheb[1 + s] * (x - b[c]) + cheb[1 + 8 + s] * (r[p][c] - y);
                    }
            b.swap(a);
            a.swap(o);
        }
        for (size_t c = 0; c < a.size(); ++c)
            if (!(std::fabs(a[c] - z[p][c]) <= 1e-4)) return emu::fail("a wrong value of z");
    }
};

static void expect(bool ok, const char *what) {
    if (!ok) emu::fail(what);
}

int main(int argc, char **argv) {
    const std::string what = argv[1];
    std::mt19937 rng(std::atoi(argv[2]));
    (void)argc;
    const auto any = [](int, int) { return true; };
    if (what == "runs") {   // two tiles, and two problems of two tiles by two workgroups
        for (int n = 1; n <= 2; ++n) {
            Set s(2, n);
            s.launch(2, 1 << 20, rng, any);
            for (int p = 0; p < n; ++p) {
                s.check(p);
                expect(s.st[p].iter == 7 && s.st[p].done == 0, "a state after a sound application");
            }
        }
    } else if (what == "converged") {   // the lead tile sets the stop flag while others read it
        Set s(2, 2);
        s.st[0].tol2 = 1e3f;
        // (some wavefronts of the other tile start after it is set)
        const unsigned late = 1 + rng() % 254;
        s.launch(2, 1 << 20, rng, [&](int b, int y) { return b == 0 || !(late >> y & 1) || s.st[0].done; });
        expect(s.st[0].done == 1 && s.st[0].iter == 7, "the state of a converged problem");
        s.check(1);
    } else if (what == "gave_up") {   // a tile marks its problem while another tile's wavefronts start
        Set s(2, 2);
        const unsigned late = 1 + rng() % 254;
        bool alone = true;   // the first tile waits in vain
        s.launch(2, 300, rng, [&](int b, int y) {
            alone = alone && !Set::marked(s.st[0]);
            return !alone || b == 0 || !(late >> y & 1);
        });
        expect(Set::marked(s.st[0]), "the mark of a problem given up");
        expect(!Set::marked(s.st[1]) && s.st[1].iter == 7, "the problem after one given up");
        s.check(1);
    } else if (what == "late_lead") {   // the lead tile starts after the other one has given up
        Set s(2, 1);
        s.launch(2, 300, rng, [&](int b, int) { return b == 1 || Set::marked(s.st[0]); });
        expect(Set::marked(s.st[0]), "the mark of a problem given up");
        expect(s.st[0].iter == 7 && s.st[0].rr == 2.f, "the update before the application is not counted");
    } else if (what == "shapes") {   // <T, per cell, Jacobi>: which of the host's tile shapes have a kernel
        auto built = [](auto t, bool pc, bool jac) {
            using T = decltype(t);
            for (int nzc : {8, 12, 16, 20})
                for (int v : {18, 28, 27}) {
                    ResShape rs;
                    rs.nzc = nzc;
                    rs.vy = v / 10;
                    rs.nw = v % 10;
                    if (launch_cheb_res<T>(rs, nullptr, pc, jac, 2, 1, false, nullptr, false, nullptr, ResArgs{}, nullptr))
                        std::printf("%d:%d%d%d:%dx%d ", nzc, (int)sizeof(T), pc, jac, v / 10, v % 10);
                }
        };
        for (int q = 0; q < 4; ++q) {
            built(0.f, q & 1, q >> 1);
            built(0.0, q & 1, q >> 1);
        }
        expect(emu_launches == 0, "a launch without problems");
    }
    std::printf("%s\n", emu::g_error.empty() ? "ok" : emu::g_error.c_str());
    return 0;
}
