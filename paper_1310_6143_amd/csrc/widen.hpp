// Reading a large array back piece by piece: each piece is copied into one of
// two host buffers and widened to doubles by several threads while the next
// one arrives.
#pragma once

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <thread>
#include <vector>

namespace sllg {

// out[0, total) = (double) of the source's values.  fetch(first, len, to)
// copies values [first, first + len) to `to` and returns when they are there,
// or throws; buf holds two pieces.  spawn(f, w) starts a thread that runs
// f(w).  False, with no thread left, when the threads cannot be had (out may
// hold anything then).  Whatever is thrown, every thread is joined first.
template <typename R, typename Fetch, typename Spawn>
bool widen_pieces(R* buf, size_t piece, size_t total, double* out, size_t threads, Fetch&& fetch, Spawn&& spawn)
{
    const size_t pieces = (total + piece - 1) / piece;
    std::atomic<size_t> ready{0};                    // pieces that have arrived (pieces + 1: stop)
    std::vector<std::atomic<size_t>> done(pieces);   // threads that have widened each piece
    for (auto& d : done)
        d.store(0);
    auto widen = [&](size_t w) {
        for (size_t k = 0; k < pieces; ++k) {
            while (ready.load(std::memory_order_acquire) <= k)
                std::this_thread::yield();
            if (ready.load(std::memory_order_acquire) > pieces)
                return;
            const size_t len = std::min(piece, total - k * piece);
            const size_t lo = len * w / threads, hi = len * (w + 1) / threads;
            const R* from = buf + (k & 1) * piece;
            double* to = out + k * piece;
            for (size_t i = lo; i < hi; ++i)
                to[i] = (double)from[i];
            done[k].fetch_add(1, std::memory_order_release);
        }
    };
    struct Pool {
        std::atomic<size_t>& ready;
        size_t stop;
        std::vector<std::thread> all;
        ~Pool()   // on the way out of an exception: the threads stop at their next piece
        {
            if (!all.empty())
                ready.store(stop, std::memory_order_release);
            join();
        }
        void join()
        {
            for (auto& t : all)
                t.join();
            all.clear();
        }
    } pool{ready, pieces + 1, {}};
    try {
        pool.all.reserve(threads);
        for (size_t w = 0; w < threads; ++w)
            pool.all.push_back(spawn(widen, w));
    } catch (...) {   // no threads, or no memory for them
        return false;
    }
    for (size_t k = 0; k < pieces; ++k) {
        while (k >= 2 && done[k - 2].load(std::memory_order_acquire) < threads)
            std::this_thread::yield();
        const size_t len = std::min(piece, total - k * piece);
        fetch(k * piece, len, buf + (k & 1) * piece);
        ready.store(k + 1, std::memory_order_release);
    }
    pool.join();
    return true;
}

}  // namespace sllg
