// Host tasks of the operator build, on threads.
#pragma once

#include <exception>
#include <functional>
#include <thread>
#include <vector>

namespace dm {

// Every task, each on a thread of its own if `threaded`; the first exception
// of a task is thrown again here, and a task that gets no thread runs on this
// one.
inline void run_tasks(bool threaded, const std::vector<std::function<void()>> &tasks) {
    std::vector<std::exception_ptr> errs(tasks.size());
    auto run = [&](size_t t) {
        try {
            tasks[t]();
        } catch (...) {
            errs[t] = std::current_exception();
        }
    };
    std::vector<std::thread> th;
    th.reserve(tasks.size());
    for (size_t t = 0; t < tasks.size(); ++t) {
        bool started = false;
        if (threaded && t + 1 < tasks.size()) {
            try {
                th.emplace_back(run, t);
                started = true;
            } catch (...) {   // no thread, or no memory for one
            }
        }
        if (!started) run(t);
    }
    for (auto &t : th) t.join();
    for (auto &e : errs)
        if (e) std::rethrow_exception(e);
}

}  // namespace dm
