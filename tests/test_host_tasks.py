"""The threads of the operator build (csrc/tasks.h), in a small C++ program:
an allocation that fails on the calling thread, at every place in turn, must
end in std::bad_alloc or in all tasks done -- never in std::terminate with
threads left running, which would abort the program that called the library."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1301_3794_amd", "csrc")

PROGRAM = r"""
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <stdexcept>
#include "tasks.h"

static thread_local long countdown = -1;   // allocations until the one that fails
void *operator new(std::size_t n) {
    if (countdown >= 0 && countdown-- == 0) throw std::bad_alloc();
    if (void *p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main() {
    std::atomic<int> done{0}, running{0};
    std::vector<std::function<void()>> tasks;
    for (int t = 0; t < 6; ++t)
        tasks.push_back([&] {
            ++running;
            std::this_thread::sleep_for(std::chrono::milliseconds(2));
            ++done;
            --running;
        });
    int failed = 0, whole = 0;
    for (long k = 0; k < 40; ++k) {
        done = 0;
        bool thrown = false;
        countdown = k;
        try {
            dm::run_tasks(true, tasks);
        } catch (const std::bad_alloc &) {
            thrown = true;
        }
        const bool hit = countdown < 0;
        countdown = -1;
        if (running != 0) return 2;              // a task outlives the call
        if (!thrown && done != 6) return 3;      // a task was lost
        failed += hit;
        whole += done == 6;
    }
    if (failed < 6) return 4;                    // the threads' own allocations were not reached
    // a task's exception comes back here, after the others have ended
    done = 0;
    std::vector<std::function<void()>> one = tasks;
    one[1] = [] { throw std::runtime_error("task"); };
    try {
        dm::run_tasks(true, one);
        return 5;
    } catch (const std::runtime_error &) {
    }
    if (done != 5) return 6;
    std::printf("%d failing allocations, %d calls whole\n", failed, whole);
    return 0;
}
"""


@pytest.mark.skipif(os.system("g++ --version > /dev/null 2>&1") != 0, reason="no host compiler")
def test_failing_allocations(tmp_path):
    src, exe = tmp_path / "tasks.cpp", tmp_path / "tasks"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stderr)
