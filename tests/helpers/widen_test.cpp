// Host test of the staged read-back: values, remainders, and threads or
// copies that fail.
#include <cstdio>
#include <new>
#include <stdexcept>
#include <system_error>
#include <thread>
#include <vector>

#include "widen.hpp"

#define CHECK(x)                                         \
    if (!(x)) {                                          \
        std::printf("line %d: %s\n", __LINE__, #x);      \
        return 1;                                        \
    }

template <typename R>
static int run(size_t total, size_t piece, size_t threads)
{
    std::vector<R> src(total), buf(2 * piece);
    for (size_t i = 0; i < total; ++i)
        src[i] = (R)(0.1 * (double)i);
    std::vector<double> out(total + 1, -7.0);
    auto fetch = [&](size_t first, size_t len, R* to) { std::copy(&src[first], &src[first] + len, to); };
    auto spawn = [](auto& f, size_t w) { return std::thread([&f, w] { f(w); }); };
    CHECK(sllg::widen_pieces(buf.data(), piece, total, out.data(), threads, fetch, spawn));
    for (size_t i = 0; i < total; ++i)
        CHECK(out[i] == (double)src[i]);
    CHECK(out[total] == -7.0);
    // the fourth thread cannot be had: no memory for it, or no thread
    for (int how = 0; how < 2; ++how) {
        size_t n = 0;
        auto scarce = [&](auto& f, size_t w) {
            if (++n == 4) {
                if (how == 0)
                    throw std::bad_alloc();
                throw std::system_error(std::make_error_code(std::errc::resource_unavailable_try_again));
            }
            return std::thread([&f, w] { f(w); });
        };
        const bool ok = sllg::widen_pieces(buf.data(), piece, total, out.data(), threads, fetch, scarce);
        CHECK(ok == (threads < 4));
    }
    // a copy that fails: its exception arrives here, after the threads have ended
    bool thrown = false;
    try {
        sllg::widen_pieces(
            buf.data(), piece, total, out.data(), threads,
            [&](size_t first, size_t len, R* to) {
                if (first + len == total)
                    throw std::runtime_error("copy");
                fetch(first, len, to);
            },
            spawn);
    } catch (const std::runtime_error&) {
        thrown = true;
    }
    CHECK(thrown);
    return 0;
}

int main()
{
    for (size_t threads : {1, 3, 8})
        for (size_t total : {1, 7, 64, 65, 128, 1000})
            if (run<float>(total, 64, threads) || run<double>(total, 64, threads))
                return 1;
    std::puts("ok");
    return 0;
}
