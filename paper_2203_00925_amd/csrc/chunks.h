// Row-parallel passes of the host setups (mesh.cpp, amg.cpp).
#pragma once
#include <algorithm>
#include <cstdint>
#include <exception>
#include <system_error>
#include <thread>
#include <vector>

namespace mifvm {

// Host threads for a setup's row-parallel passes: up to 16 for n rows of
// at least 65,536, else 1.
inline int setup_threads(int64_t n) {
    const unsigned h = std::thread::hardware_concurrency();
    return n < 65536 ? 1 : int(std::min<unsigned>(16, h ? h : 1));
}

// f(k, lo, hi) for the nt contiguous chunks [lo, hi) of [0, n), chunk k on
// its own thread (chunk 0 on the caller's, and those that get no thread);
// every row is handled by exactly one call, so results do not depend on nt.
// What a call throws is thrown here, once all have ended.
template <class F>
void for_chunks(int64_t n, int nt, F&& f) {
    std::vector<std::exception_ptr> thrown(size_t(nt), nullptr);
    auto run = [&f, &thrown, n, nt](int k) {
        try {
            f(k, n * k / nt, n * (k + 1) / nt);
        } catch (...) {
            thrown[k] = std::current_exception();
        }
    };
    std::vector<std::thread> th;
    th.reserve(size_t(nt));
    int k = 1;
    try {
        for (; k < nt; ++k) th.emplace_back(run, k);
    } catch (const std::system_error&) {
    }
    run(0);
    for (; k < nt; ++k) run(k);
    for (auto& t : th) t.join();
    for (auto& e : thrown)
        if (e) std::rethrow_exception(e);
}

}  // namespace mifvm
