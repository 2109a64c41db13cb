// Host-side planning of how many iterations of a solve are queued ahead of the
// device (no device code: the host unit tests compile it alone).
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "sph.h"

namespace sph {

// What the host knows of the solver's control block between iterations:
// residuals (bb: of b), tolerances, states, iteration and halt.
struct CtlPoll {
    double rr[3];
    double bb[3];
    double tau2[3];
    int32_t state[3];
    int32_t iter;
    int32_t halt;
};

// Forecast of a solve's halt from what p updates report, and the iterations to
// queue for it.  With nothing known 2 (at most kmax).  Two
// reports give each progressing component c a rate of decrease of ln(r.r) per
// iteration (the steeper of the latest interval's and the round's average,
// so that a noisy residual history errs towards an early halt; a round
// after a restart starts from the rates of the round before), and from it
// the iterations m_c left to reach its tolerance.  The iteration whose
// p-update halts is then predicted at H = iter + max_c m_c (iter: the last
// p-update seen), and each batch covers half of what is left up to H.
// When every issued iteration already reaches H the host queues nothing
// until the next report is read (unless none is in flight), so a solve that
// ends as predicted leaves no iteration issued past its halt.  The halting
// iteration itself is always issued (its p-update decides the halt), once
// per round of host-side residual checks.
class IssuePlan {
  public:
    explicit IssuePlan(int kmax) : kmax_(kmax) {}

    // a new round after a host-side residual check, whose control block is
    // `m` (restarted components progressing again from their true r.r): the
    // residuals start again, the rates are kept
    void restart(const CtlPoll& m) {
        npoll_ = 0;
        have_pred_ = false;
        observe(m);
    }

    void observe(const CtlPoll& m) {
        if (m.halt) return;
        double lrr[3];
        for (int c = 0; c < 3; ++c) lrr[c] = m.rr[c] > 0.0 ? std::log(m.rr[c]) : -HUGE_VAL;
        double horizon = 0.0;
        bool known = true;
        for (int c = 0; c < 3; ++c) {
            if (m.state[c] != SPH_PROGRESSING) continue;
            if (npoll_ >= 1 && m.iter > it_last_ && m.iter > it_first_ && std::isfinite(lrr[c]) &&
                std::isfinite(lrr_last_[c]) && std::isfinite(lrr_first_[c])) {
                const double r_last = (lrr[c] - lrr_last_[c]) / (double)(m.iter - it_last_);
                const double r_avg = (lrr[c] - lrr_first_[c]) / (double)(m.iter - it_first_);
                rate_[c] = std::min(r_last, r_avg);
            }
            if (!(rate_[c] < 0.0) || !(m.tau2[c] > 0.0) || !std::isfinite(lrr[c])) {
                known = false;
                continue;
            }
            horizon = std::max(horizon, (std::log(m.tau2[c]) - lrr[c]) / rate_[c]);
        }
        if (npoll_ == 0) {
            it_first_ = m.iter;
            for (int c = 0; c < 3; ++c) lrr_first_[c] = lrr[c];
        }
        it_last_ = m.iter;
        for (int c = 0; c < 3; ++c) lrr_last_[c] = lrr[c];
        ++npoll_;
        have_pred_ = known;
        if (known) halt_pred_ = m.iter + (int32_t)std::min(std::ceil(horizon), 1.0e6);
    }

    // iterations from the last one seen to the forecast halt, at most twice
    // those that the forecast rests on; 0: not known
    int32_t left() const {
        return have_pred_ ? std::max(std::min(halt_pred_ - it_last_, 2 * (it_last_ - it_first_)), 0) : 0;
    }

    // iterations to queue now, the first of them being `next`; 0 = wait for
    // the report in flight
    int batch(int32_t next, bool poll_in_flight) {
        if (!have_pred_) return std::min(2, kmax_);
        const int32_t reach = halt_pred_ - next + 1;  // iterations up to H
        if (reach <= 0) return poll_in_flight ? 0 : 1;
        // half the distance per batch, so that the reports close in on H; 0
        // (wait for the report in flight) once H is the next iteration
        const int32_t k = poll_in_flight ? reach / 2 : (reach + 1) / 2;
        return std::min(k, (int32_t)kmax_);
    }

  private:
    int kmax_;
    int npoll_ = 0;
    bool have_pred_ = false;
    int32_t halt_pred_ = 0;
    int32_t it_first_ = 0, it_last_ = 0;
    double lrr_first_[3] = {0.0, 0.0, 0.0}, lrr_last_[3] = {0.0, 0.0, 0.0};
    double rate_[3] = {0.0, 0.0, 0.0};  // 0: none known yet
};

// The issue loop's decision: how many iterations to queue beyond the last one
// whose p update the host has seen.  kAhead suffices for a device that never
// waits (the p update is the first kernel of its iteration, and the others run
// while the host queues the next), and one in later rounds, which are often
// short.  A host that is kept from this loop for longer can ask for more
// (poll_every): up to that many are queued while the forecast halt is at least
// four times as far, so that a forecast that is wrong by a factor of four still
// leaves nothing behind the halt, and the round twice as old.
class IssueLoop {
  public:
    static constexpr int32_t kAhead = 2;
    explicit IssueLoop(int32_t poll_every)
        : asked_(poll_every > 0 ? poll_every : kAhead), most_(std::min(asked_, kAhead)), plan_(asked_) {}
    void later_round(const CtlPoll& m) {
        most_ = 1;
        plan_.restart(m);
    }
    void observe(const CtlPoll& m) { plan_.observe(m); }
    // iterations to queue now, the first of them being `next`, when p updates
    // up to that of iteration `seen` are known
    int32_t queue(int32_t next, int32_t seen) {
        const int32_t ahead = next - 1 - seen;
        const int32_t most = std::max(most_, std::min(asked_, plan_.left() / 4));
        return ahead < most ? std::min(plan_.batch(next, ahead > 0), most - ahead) : 0;
    }

  private:
    int32_t asked_;  // most iterations ahead by the caller's wish
    int32_t most_;   // whatever the forecast
    IssuePlan plan_;
};

}  // namespace sph
