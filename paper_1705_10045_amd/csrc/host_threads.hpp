// Host work over long arrays on a few threads that end with the call.
#pragma once

#include <algorithm>
#include <exception>
#include <thread>
#include <vector>

namespace lbm {

constexpr int kHostThreads = 8;

// Threads for `items` of host work, `grain` of them at least for each thread.
inline int host_threads(long long items, long long grain)
{
    const long long cores = (long long)std::thread::hardware_concurrency();
    return (int)std::max(1LL, std::min({(long long)kHostThreads, cores, items / grain}));
}

// work(t) for t = 0 .. threads - 1, t = 0 on the calling thread; work must not throw.  What no thread
// could be started for runs on the calling thread too.
template <class Work>
void on_threads(int threads, const Work& work)
{
    std::vector<std::thread> pool;
    int started = 1;
    try {
        pool.reserve(threads);
        for (; started < threads; ++started) pool.emplace_back([&work, t = started] { work(t); });
    } catch (const std::exception&) {
    }
    work(0);
    for (int t = started; t < threads; ++t) work(t);
    for (std::thread& t : pool) t.join();
}

}  // namespace lbm
