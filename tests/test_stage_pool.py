"""The staging-slot pool of the search entry points, exercised on the host alone: the pool's
header knows nothing of HIP, so a small C++ program drives it with fake events from many threads
and checks that no slot is ever held by two calls at once and that no slot is handed out while
the work recorded behind its last use is pending."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_14881_amd", "csrc")
SRC = os.path.join(ROOT, "tests", "stage_pool_host_test.cpp")


@pytest.mark.parametrize("sanitize", [False, True])
def test_slots_have_one_owner_and_wait_for_their_last_use(tmp_path, sanitize):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "stage_pool_host_test")
    cmd = [cxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, SRC, "-o", exe]
    if sanitize:
        cmd[1:1] = ["-fsanitize=thread"]
    built = subprocess.run(cmd, capture_output=True, text=True)
    if sanitize and built.returncode != 0:
        pytest.skip("ThreadSanitizer runtime not available: " + built.stderr[-200:])
    assert built.returncode == 0, built.stderr
    # more threads than slots, so that calls also meet a pool with every slot owned
    run = subprocess.run([exe, "24" if not sanitize else "12", "3000"], capture_output=True, text=True, timeout=240)
    assert run.returncode == 0, run.stdout + run.stderr
    words = run.stdout.split()
    assert words[0] == "ok" and int(words[1]) == (24 if not sanitize else 12) * 3000


_KEPT = r"""
#include <cstdio>
#include "st_stage_pool.h"
static int waits = 0;
static bool done(void*) { return false; }            // nothing on the device ever completes by itself
static int wait_for(void*) { ++waits; return 0; }
int main()
{
    st::StagePool pool;
    st::StageSlot* s = nullptr;
    if (pool.acquire(done, wait_for, &s) != 0) return 1;
    st::StageSlot* kept = s;
    pool.keep(kept);
    for (int i = 0; i < 5 * st::kStageSlots; ++i) {  // every other slot is pending: some have to be waited for
        if (pool.acquire(done, wait_for, &s) != 0) return 2;
        if (s == kept) return 3;
        pool.release(s, true);
    }
    if (waits == 0) return 4;
    for (int i = 1; i < st::kStageSlots; ++i) {
        if (pool.acquire(done, wait_for, &s) != 0) return 5;
        pool.keep(s);
    }
    if (pool.acquire(done, wait_for, &s) != st::StagePool::kNoSlot) return 6;
    st::StageSlot* back = pool.take_kept();
    if (!back) return 7;
    pool.release(back, false);
    if (pool.acquire(done, wait_for, &s) != 0 || s != back) return 8;
    puts("ok");
    return 0;
}
"""


def test_a_slot_that_a_graph_reads_is_not_handed_out(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "kept.cpp", str(tmp_path / "kept")
    src.write_text(_KEPT)
    built = subprocess.run([cxx, "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.strip() == "ok", (run.returncode, run.stderr)
