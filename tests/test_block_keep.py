"""What the library keeps of a freed index's device memory, and when it gives it back: the pool's header knows
nothing of HIP, so a small C++ program drives it with a driver of its own that counts and can refuse."""
import shutil
import subprocess

import pytest

from tests.test_stage_pool import CSRC

_SRC = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include <thread>
#include <vector>
#include "st_block_keep.h"
static std::mutex mu;
static std::set<void*> held;
static int refuse = 0, idles = 0, idle_error = 0;   // the next `refuse` allocations fail
static int alloc_(void** out, int64_t)
{
    std::lock_guard<std::mutex> l(mu);
    if (refuse > 0) { --refuse; return 2; }
    held.insert(*out = malloc(1));
    return 0;
}
static int free_(void* p)
{
    std::lock_guard<std::mutex> l(mu);
    if (!held.erase(p)) abort();                     // freed twice, or never handed out
    free(p);
    return 0;
}
static int idle_() { ++idles; return idle_error; }
#define CHECK(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)
int main()
{
    st::BlockKeep k;
    void *a, *b, *c;
    auto index = [&](int64_t n, void** p) { return k.get_index(3, n, alloc_, free_, p); };
    auto gone = [&](void* p, int64_t n) { return k.put_index(3, p, n, free_, idle_); };
    // the last index of a device: all its memory goes back
    CHECK(index(100, &a) == 0 && gone(a, 100) == 0 && held.empty());
    // replaced by another: its block is kept (behind a wait for the device) and taken again
    CHECK(index(100, &a) == 0 && index(100, &b) == 0 && idles == 0 && gone(a, 100) == 0 && idles == 1 && held.size() == 2);
    CHECK(index(100, &c) == 0 && c == a && held.size() == 2);
    // one block at most, and none of another size
    CHECK(gone(b, 100) == 0 && held.size() == 2 && index(60, &b) == 0 && held.size() == 2);
    CHECK(gone(b, 60) == 0 && held.size() == 2 && gone(c, 100) == 0 && held.empty());
    // larger than the limit: not kept, and what was kept goes back as well
    CHECK(index(100, &a) == 0 && index(100, &b) == 0 && index(st::kKeepBytes + 1, &c) == 0 && gone(a, 100) == 0 && held.size() == 3);
    CHECK(gone(c, st::kKeepBytes + 1) == 0 && held.size() == 1 && gone(b, 100) == 0 && held.empty());
    // an allocation that fails is tried again without the kept block, and only then
    for (int which = 0; which < 2; ++which) {
        CHECK(index(100, &a) == 0 && index(100, &b) == 0 && gone(a, 100) == 0 && held.size() == 2);
        refuse = which;
        if (which) CHECK(k.get(3, 7, alloc_, free_, &c) == 0 && held.size() == 2 && free_(c) == 0);
        else CHECK(index(100, &c) == 0 && held.size() == 2 && gone(c, 100) == 0 && k.release(3, free_) == 0);
        CHECK(held.size() == 1 && gone(b, 100) == 0 && held.empty());
    }
    refuse = 1;
    CHECK(index(100, &a) == 2 && held.empty());
    CHECK(index(100, &a) == 0 && gone(a, 100) == 0 && held.empty());  // (the failed one was not counted)
    refuse = 2;
    CHECK(index(100, &a) == 2 && index(100, &a) == 2 && index(100, &a) == 0);
    // a failing wait leaves the index as it was
    CHECK(index(100, &b) == 0);
    idle_error = 5;
    CHECK(gone(a, 100) == 5 && held.size() == 2);
    idle_error = 0;
    CHECK(gone(a, 100) == 0 && held.size() == 2 && k.release(3, free_) == 0 && held.size() == 1 && gone(b, 100) == 0 && held.empty());
    // many threads: nothing is lost, freed twice or handed out twice
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; ++t)
        ts.emplace_back([&, t] {
            for (int i = 0; i < 5000; ++i) {
                void* p = nullptr;
                const int64_t n = 100 + (i + t) % 2;
                if (k.get_index(0, n, alloc_, free_, &p)) abort();
                if (k.put_index(0, p, n, free_, [] { return 0; })) abort();
            }
        });
    for (auto& t : ts) t.join();
    CHECK(held.empty());
    puts("ok");
    return 0;
}
"""


def test_kept_blocks_go_back(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "keep.cpp", str(tmp_path / "keep")
    src.write_text(_SRC)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Wextra", "-pthread", "-I", CSRC, str(src), "-o", exe],
                           capture_output=True, text=True)
    assert built.returncode == 0 and not built.stderr, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.strip() == "ok", (run.returncode, run.stdout, run.stderr)
