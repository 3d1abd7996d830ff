// Threads that share the passes of one call (host only).
#pragma once

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <functional>
#include <mutex>
#include <thread>

namespace spmm {

// f(begin, end) over [0, n) in pieces of `piece`, by the calling thread and up to 7 others; `own`, where there is one, is run
// first by the calling thread.  Packing a model's weights is what its load waits for, in several passes over independent
// rows, and starting 7 threads for each of them took 50 to 100 us a pass.  They are started once, each by one started before, and
// wait for the next pass, as many as the first pass that is shared has pieces for (the others have as many: rows of a weight);
// nothing of it outlives the call that packs.  (1024x4096 at 80 %, onto the device: 0.99 ms with
// threads started for each pass and one form, 1.7 with both; now 0.91 with both.)
class Team {
public:
    Team() : most_((int)std::min<int64_t>(7, std::max<int64_t>(0, (int64_t)std::thread::hardware_concurrency() - 1))) {}
    ~Team()
    {
        {
            const std::lock_guard<std::mutex> lock(mutex_);
            end_ = true;
            pass_.fetch_add(1);
        }
        work_.notify_all();
        join();
    }
    Team(const Team&) = delete;
    Team& operator=(const Team&) = delete;

    template <typename F>
    void run(int64_t n, int64_t piece, const F& f) { run(n, piece, f, [] {}, false); }

    template <typename F, typename O>
    void run(int64_t n, int64_t piece, const F& f, const O& own) { run(n, piece, f, own, false); }

    // the last pass: the threads end when nothing is left of it, instead of being woken for that (a pass after it starts them anew:
    // where the device turns out to have no memory for what it was to pack, the host's passes follow; 4096x4096 at 70 %, 6.6 ms
    // instead of 39 by the calling thread alone)
    template <typename F>
    void finish(int64_t n, int64_t piece, const F& f) { run(n, piece, f, [] {}, true); }
    template <typename F, typename O>
    void finish(int64_t n, int64_t piece, const F& f, const O& own) { run(n, piece, f, own, true); }

private:
    template <typename F, typename O>
    void run(int64_t n, int64_t piece, const F& f, const O& own, bool last)
    {
        const int64_t pieces = (n + piece - 1) / piece;
        if (pieces <= 1 || !most_) {
            own();
            for (int64_t i = 0; i < pieces; ++i) f(i * piece, std::min(n, (i + 1) * piece));
            return;
        }
        if (over_) {
            join();
            started_ = false;
        }
        over_ = last;
        const std::function<void(int64_t)> call = [&](int64_t i) { f(i * piece, std::min(n, (i + 1) * piece)); };
        {
            const std::lock_guard<std::mutex> lock(mutex_);
            call_ = &call;
            next_ = 0;
            left_ = pieces_ = pieces;
            failed_ = nullptr;
            end_ = last;
            pass_.fetch_add(1);
        }
        work_.notify_all();
        if (!started_) {
            started_ = true;        // (300x300 is two pieces: 0.24 ms with 7 threads started, 0.15 with one)
            most_ = (int)std::min<int64_t>(most_, pieces - 1);
            start(0);
        }
        std::exception_ptr failed;
        try {
            own();
        } catch (...) {
            failed = std::current_exception();
        }
        while (work()) {}
        std::unique_lock<std::mutex> lock(mutex_);
        done_.wait(lock, [&] { return left_ == 0; });
        call_ = nullptr;
        if (!failed) failed = failed_;
        lock.unlock();
        if (failed) std::rethrow_exception(failed);
    }

    void join()
    {
        for (int i = 0; i < most_; ++i)         // (a thread starts two others before it can end)
            if (threads_[i].joinable()) threads_[i].join();
    }
    // a piece, if one is left
    bool work()
    {
        const std::function<void(int64_t)>* call;
        int64_t i;
        {
            const std::lock_guard<std::mutex> lock(mutex_);
            if (!call_ || next_ >= pieces_) return false;
            call = call_;
            i = next_++;
        }
        std::exception_ptr failed;
        try {
            (*call)(i);
        } catch (...) {
            failed = std::current_exception();
        }
        const std::lock_guard<std::mutex> lock(mutex_);
        if (failed && !failed_) failed_ = failed;
        if (--left_ == 0) done_.notify_one();
        return true;
    }
    // thread i, which starts 2 i + 1 and 2 i + 2
    void start(int i)
    {
        if (i >= most_) return;
        try {
            threads_[i] = std::thread([this, i] {
                start(2 * i + 1);
                start(2 * i + 2);
                for (;;) {
                    const unsigned seen = pass_.load();
                    while (work()) {}
                    if (end_) return;
                    for (int spin = 0; spin < 200 && pass_.load() == seen; ++spin) std::this_thread::yield();
                    std::unique_lock<std::mutex> lock(mutex_);
                    work_.wait(lock, [&] { return end_ || pass_.load() != seen; });
                }
            });
        } catch (...) {         // no more threads to be had: the others do the work
        }
    }

    int most_;                  // threads besides the caller's
    bool started_ = false, over_ = false;       // over_: by `finish`
    std::atomic<bool> end_{false};
    std::thread threads_[7];
    std::mutex mutex_;
    std::condition_variable work_, done_;
    std::atomic<unsigned> pass_{0};
    const std::function<void(int64_t)>* call_ = nullptr;
    int64_t next_ = 0, pieces_ = 0, left_ = 0;
    std::exception_ptr failed_;
};

}  // namespace spmm
