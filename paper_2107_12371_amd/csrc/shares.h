// Host work in equal shares on several threads.
#pragma once

#include <atomic>
#include <exception>
#include <new>
#include <thread>
#include <vector>

namespace spmvlib {

// Runs work(t) for t < n on up to n threads; a thread that cannot be started
// has its share run here.  std::bad_alloc where a share threw, once all ended.
template <typename F> void run_shares(int n, F &&work) {
    std::atomic<bool> failed{false};
    const auto share = [&](int t) {
        try {
            work(t);
        } catch (const std::exception &) {
            failed = true;
        }
    };
    std::vector<std::thread> th;
    int t = 1;
    try {
        th.reserve((size_t)n);
        for (; t < n; ++t) th.emplace_back(share, t);
    } catch (const std::exception &) {
    }
    share(0);
    for (; t < n; ++t) share(t);
    for (auto &x : th) x.join();
    if (failed) throw std::bad_alloc();
}

}  // namespace spmvlib
