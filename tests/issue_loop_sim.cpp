// Host simulation of a solve's issue loop: IssueLoop decides, as in
// sph_visc_solve, on synthetic residual histories.  The device runs one
// iteration per tick, its p update first, which mails its outcome; the host
// looks at the mail every `period` ticks (a host that is kept away for longer
// than an iteration skips outcomes).  Histories from stdin instead, one r.r
// per line and component, with "stdin TAU2" as arguments.  Prints one line
// per run: name, poll_every, period, halting iteration H, iterations issued,
// most queued beyond the last one seen, ticks the device waited for the host.
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "issue_plan.hpp"

using sph::CtlPoll;
using sph::IssueLoop;

struct History {
    std::vector<std::array<double, 3>> rr;  // r.r after iteration j (j = 0: the start)
    double tau2;
};

static bool progressing(const History& h, int j, int c) { return !(h.rr[j][c] < h.tau2); }

// The p update of iteration it reads r.r of iteration it - 1 and halts when no
// component progresses, or at the end of the history (the iteration limit).
static int halt_iter(const History& h) {
    for (int it = 1; it <= (int)h.rr.size(); ++it) {
        bool any = false;
        for (int c = 0; c < 3; ++c) any |= progressing(h, it - 1, c);
        if (!any) return it;
    }
    return (int)h.rr.size();
}

static void run(const char* name, const History& h, int poll_every, int period) {
    const int H = halt_iter(h), last_it = (int)h.rr.size();
    IssueLoop loop(poll_every);
    int it = 1, seen = 0, done = 0, most = 0, idle = 0;  // done: p updates that have run
    bool halted = false;
    for (int tick = 0; !halted; ++tick) {
        if (tick % period == 0) {
            if (done > seen) {
                const int q = std::min(done, H);
                CtlPoll m{};
                m.iter = q;
                m.halt = q >= H;
                for (int c = 0; c < 3; ++c) {
                    m.rr[c] = h.rr[q - 1][c];
                    m.tau2[c] = h.tau2;
                    m.state[c] = progressing(h, q - 1, c) ? SPH_PROGRESSING : SPH_CONVERGED;
                }
                seen = q;
                loop.observe(m);
                halted = m.halt;
            }
            while (!halted && it <= last_it) {
                const int k = std::min(loop.queue(it, seen), last_it - it + 1);
                if (k <= 0) break;
                it += k;
                most = std::max(most, it - 1 - seen);
            }
        }
        if (done < it - 1) ++done;
        else if (!halted) ++idle;
        if (tick > 100 * last_it * period) {
            std::printf("%s: no halt\n", name);
            std::exit(1);
        }
    }
    std::printf("%s %d %d %d %d %d %d\n", name, poll_every, period, H, it - 1, most, idle);
}

static void runs(const char* name, const History& h) {
    for (int p : {0, 1, 2, 16, 1000})
        for (int period : {1, 2, 3, 12}) run(name, h, p, period);
}

static History decay(int n, double q, double tau2) {
    History h;
    for (int j = 0; j < n; ++j) h.rr.push_back({std::pow(q, j), std::pow(q * 0.98, j), std::pow(q * 0.9, j)});
    h.tau2 = tau2;
    return h;
}

int main(int argc, char** argv) {
    if (argc > 2 && std::string(argv[1]) == "stdin") {
        History h;
        h.tau2 = std::atof(argv[2]);
        std::array<double, 3> v;
        while (std::scanf("%lf %lf %lf", &v[0], &v[1], &v[2]) == 3) h.rr.push_back(v);
        runs("stdin", h);
        return 0;
    }
    runs("fast", decay(60, 0.1, 1e-12));
    runs("geometric", decay(400, 0.7, 1e-12));
    runs("slow", decay(2000, 0.97, 1e-12));
    for (int seed = 1; seed <= 5; ++seed) {  // noisy decays (BiCGSTAB's residual is not monotone)
        std::mt19937_64 rng(seed);
        std::normal_distribution<double> nd(0.0, 1.0);
        History h = decay(600, 0.85, 1e-12);
        for (auto& v : h.rr)
            for (double& r : v) r *= std::exp(1.5 * nd(rng));
        runs("noisy", h);
    }
    {  // a plateau of 30 iterations, then a geometric decay
        History h = decay(600, 0.7, 1e-12);
        h.rr.insert(h.rr.begin(), 30, {1.0, 1.0, 1.0});
        runs("plateau", h);
    }
    {  // a slow decay that ends at once: the worst forecast there is
        History h = decay(2000, 0.99, 1e-12);
        for (size_t j = 300; j < h.rr.size(); ++j) h.rr[j] = {1e-13, 1e-13, 1e-13};
        runs("collapse", h);
    }
    runs("converged_start", decay(10, 0.7, 10.0));
    runs("iteration_limit", decay(50, 0.999, 1e-12));
    return 0;
}
