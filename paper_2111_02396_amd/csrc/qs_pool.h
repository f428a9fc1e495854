// Host worker threads for the planners' parallel loops.
#ifndef QS_POOL_H
#define QS_POOL_H

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstddef>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

namespace qs {

// The threads are started on first use and kept: starting them on every call
// cost more than the per-trajectory draws they share.  The calling thread
// takes part in its loop.  Several calls may have a loop open at once: the
// chunks of a concurrent call plan at the same time, and with one loop at a
// time they waited for one another (four states of two 11-qubit trajectories
// each 200 us a call, now 110; of two noisy 14-qubit ones 1.33 ms, now 0.82).
// A loop of up to three threads wakes only those it has room for (two
// noiseless trajectories of one qubit, planned by the caller alone: 55 us a
// call with fifteen threads woken, now 29); a longer one wakes all with one
// system call, and the first of them take its places.
class HostPool {
  public:
    static HostPool &get() {
        static HostPool *pool = new HostPool();  // never destroyed: workers may outlive statics
        return *pool;
    }
    unsigned size() const { return unsigned(workers_.size()) + 1; }
    // fn(lo, hi) over [0, n) in chunks of `chunk`, on at most `width` threads.
    void run(size_t n, size_t chunk, unsigned width, const std::function<void(size_t, size_t)> &fn) {
        if (n == 0) return;
        chunk = std::max<size_t>(chunk, 1);
        const size_t pieces = (n + chunk - 1) / chunk;
        width = unsigned(std::min<size_t>(pieces, std::max(1u, std::min(width, size()))));
        if (width == 1) {
            fn(0, n);
            return;
        }
        Loop loop;
        loop.fn = &fn;
        loop.n = n;
        loop.chunk = chunk;
        loop.helpers = width - 1;
        {
            std::lock_guard<std::mutex> lock(mu_);
            open_.push_back(&loop);
        }
        if (width >= 4) cv_.notify_all();  // the first to wake take the places
        else
            for (unsigned i = 1; i < width; ++i) cv_.notify_one();
        loop.drain();
        // helpers that have not started by now stay out of this loop
        std::unique_lock<std::mutex> lock(mu_);
        open_.erase(std::find(open_.begin(), open_.end(), &loop));
        loop.idle.wait(lock, [&] { return loop.busy == 0; });
    }

  private:
    // One call's loop, on its stack: helpers enter it only while it is in open_
    // and are counted in `busy`, both under mu_.
    struct Loop {
        const std::function<void(size_t, size_t)> *fn = nullptr;
        size_t n = 0, chunk = 1;
        std::atomic<size_t> next{0};
        unsigned helpers = 0, busy = 0;  // places left for helpers; helpers inside
        std::condition_variable idle;
        void drain() {
            for (;;) {
                const size_t lo = next.fetch_add(chunk);
                if (lo >= n) return;
                (*fn)(lo, std::min(n, lo + chunk));
            }
        }
    };
    HostPool() {
        const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
        const unsigned nw = std::min(15u, hw > 1 ? hw - 1 : 0u);
        for (unsigned i = 0; i < nw; ++i) workers_.emplace_back([this] { work(); });
        for (auto &w : workers_) w.detach();
    }
    // A loop with work and room for one more helper, or null (under mu_).
    Loop *pick() const {
        for (Loop *l : open_)
            if (l->helpers > 0 && l->next.load() < l->n) return l;
        return nullptr;
    }
    void work() {
        std::unique_lock<std::mutex> lock(mu_);
        for (;;) {
            Loop *l = nullptr;
            cv_.wait(lock, [&] { return (l = pick()) != nullptr; });
            --l->helpers;
            ++l->busy;
            lock.unlock();
            l->drain();
            lock.lock();
            if (--l->busy == 0) l->idle.notify_one();
        }
    }
    std::vector<std::thread> workers_;
    std::mutex mu_;
    std::condition_variable cv_;
    std::vector<Loop *> open_;
};

}  // namespace qs

#endif  // QS_POOL_H
