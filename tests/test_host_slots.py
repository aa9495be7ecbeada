"""The pinned host slots of the contexts (csrc/host_slots.h), compiled here with an
allocator that counts its pages."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "host_slots.h"
#include <cstdio>
#include <cstdio>
#include <cstdlib>
#include <atomic>
#include <set>
#include <thread>
static std::atomic<int> live{0}, most{0};
static int fail = 0;
static int take_page(double** p, size_t bytes) {
    if (fail) return fail;
    *p = (double*)malloc(bytes);
    if (++live > most) most = live.load();
    return 0;
}
static void free_page(double* p) { free(p); --live; }
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main() {
    using namespace mg;
    HostSlots s(take_page, free_page);
    double* p[40];
    std::set<double*> seen;
    for (double*& q : p) {
        CHECK(s.take(&q) == 0 && seen.insert(q).second);
        for (size_t k = 0; k < kHostDoubles; ++k) q[k] = 1.0;  // in bounds of its page
    }
    CHECK(live == 5);
    // an error is passed on and takes no slot
    double* none = nullptr;
    fail = 7;
    CHECK(s.take(&none) == 7 && none == nullptr);
    fail = 0;
    // every other slot back: no page is free; a slot that is back is used again
    for (int i = 0; i < 40; i += 2) s.back(p[i]);
    CHECK(live == 5);
    double* again = nullptr;
    CHECK(s.take(&again) == 0 && live == 5 && seen.count(again));
    s.back(again);
    for (int i = 1; i < 40; i += 2) s.back(p[i]);
    CHECK(live == 1);  // one page kept
    for (int i = 0; i < 100; ++i) {  // and reused
        CHECK(s.take(&p[0]) == 0);
        s.back(p[0]);
        CHECK(live == 1);
    }
    auto work = [&] {
        double* q[6];
        for (int i = 0; i < 2000; ++i) {
            for (double*& r : q) s.take(&r);
            for (double*& r : q) r[0] = (double)(size_t)&r;
            for (double*& r : q)
                if (r[0] != (double)(size_t)&r) std::abort();
            for (double*& r : q) s.back(r);
        }
    };
    std::thread a(work), b(work), c(work);
    a.join(); b.join(); c.join();
    CHECK(live == 1 && most <= 6);
    return 0;
}
"""


def test_slots_are_unique_reused_and_given_back(tmp_path):
    src, exe = tmp_path / "slots.cpp", tmp_path / "slots"
    src.write_text(PROGRAM)
    inc = os.path.join(ROOT, "paper_2607_10983_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", inc, str(src), "-o", str(exe)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout
