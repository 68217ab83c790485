// Copying field planes out of the read-back slots with several threads (host
// code only).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>

namespace lbm {

// Copies pieces of field planes out of the slots as they become ready: the
// caller and helper threads take parts of the ready pieces in order, so that
// any number of helpers, none included, does the work.  Helpers are started for
// planes of some size only (one for every 4 MiB) and end with the call.  It runs
// under a C entry point: it holds no memory of its own, and a helper that can't
// be started is done without.
class PlaneCopy {
public:
    static constexpr int kParts = 8, kMaxSlots = 4;
    PlaneCopy(double *const outs[6], const double *slots, int64_t slot_doubles, int nslots, int64_t piece, int64_t nodes)
        : outs_(outs), slots_(slots), slot_doubles_(slot_doubles), nslots_(nslots), piece_(piece), nodes_(nodes) {
        const int64_t mib = nodes * 6 * (int64_t)sizeof(double) >> 20;
        const int cpus = (int)std::thread::hardware_concurrency();
        const int helpers = (int)std::min<int64_t>({mib / 4, kParts - 1, cpus > 1 ? cpus - 1 : 0});
        try {
            for (; helpers_ < helpers; ++helpers_) threads_[helpers_] = std::thread([this] { serve(); });
        } catch (...) {  // fewer helpers, or none
        }
    }
    ~PlaneCopy() {
        {
            std::lock_guard<std::mutex> l(m_);
            quit_ = true;
        }
        ready_cv_.notify_all();
        for (int i = 0; i < helpers_; ++i) threads_[i].join();
    }
    // The slots of pieces before n are complete.
    void publish(int64_t n) {
        {
            std::lock_guard<std::mutex> l(m_);
            ready_ = n * kParts;
        }
        ready_cv_.notify_all();
    }
    // Returns when piece p is copied out; takes part in the copying.  Pieces are
    // finished in order, each before another takes its slot.
    void finish(int64_t p) {
        int &done = done_[p % nslots_];
        std::unique_lock<std::mutex> l(m_);
        while (done < kParts && take(l)) {
        }
        done_cv_.wait(l, [&] { return done == kParts; });
        done = 0;
    }

private:
    void serve() {
        std::unique_lock<std::mutex> l(m_);
        for (;;) {
            ready_cv_.wait(l, [this] { return quit_ || next_ < ready_; });
            if (quit_) return;
            while (take(l)) {
            }
        }
    }
    // Copies the next part, if one is ready.
    bool take(std::unique_lock<std::mutex> &l) {
        if (next_ >= ready_) return false;
        const int64_t p = next_ / kParts, part = next_ % kParts;
        ++next_;
        l.unlock();
        const int64_t o = p * piece_, n = std::min(piece_, nodes_ - o);
        const int64_t a = n * part / kParts, b = n * (part + 1) / kParts;
        const double *slot = slots_ + (p % nslots_) * slot_doubles_;
        for (int q = 0; q < 6; ++q)
            std::memcpy(outs_[q] + o + a, slot + q * n + a, (size_t)(b - a) * sizeof(double));
        l.lock();
        if (++done_[p % nslots_] == kParts) done_cv_.notify_one();
        return true;
    }

    double *const *outs_;
    const double *slots_;
    int64_t slot_doubles_, nslots_, piece_, nodes_;
    std::mutex m_;
    std::condition_variable ready_cv_, done_cv_;
    int64_t ready_ = 0, next_ = 0;  // parts that may be, that have been taken
    int done_[kMaxSlots] = {};      // parts copied of the piece in each slot
    bool quit_ = false;
    int helpers_ = 0;
    std::thread threads_[kParts - 1];
};

}  // namespace lbm
