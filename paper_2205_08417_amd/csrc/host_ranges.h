// Host loops over the cells of a large mesh on several threads.
#pragma once

#include <cstdint>
#include <exception>
#include <thread>
#include <vector>

namespace snrt {

constexpr int kHostParts = 8;
constexpr int64_t kHostAlone = 32768;      // below, threads cost more than they save (0.3 -> 3 ms)

// f(part, first, end) for up to kHostParts contiguous parts of [0, n), each on a thread of its own.
// The parts depend on n alone; a thread that cannot be had has its part done here, and the first
// exception of a part is thrown again when all have ended.
template <typename F>
void host_ranges(int64_t n, F&& f) {
    const int parts = n < kHostAlone ? 1 : kHostParts;
    std::exception_ptr error[kHostParts] = {};
    auto run = [&](int p) noexcept {
        try {
            f(p, n * p / parts, n * (p + 1) / parts);
        } catch (...) {
            error[p] = std::current_exception();
        }
    };
    std::thread threads[kHostParts];
    bool here[kHostParts] = {};
    for (int p = 1; p < parts; ++p) {
        try {
            threads[p] = std::thread(run, p);
        } catch (...) {
            here[p] = true;
        }
    }
    run(0);
    for (int p = 1; p < parts; ++p) {
        if (here[p]) run(p);
        else threads[p].join();
    }
    for (const std::exception_ptr& e : error)
        if (e) std::rethrow_exception(e);
}

}  // namespace snrt
