"""Knobs changed by one host thread while another one asks for launch shapes: what the other thread
remembers is dropped with the change, never kept from the moment before it."""
import os
import shutil
import subprocess

import pytest

SOURCE = r"""
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <atomic>
#include <thread>

typedef size_t (*size_fn)(int64_t, int64_t, int64_t, int);
typedef int (*tune_fn)(const char *, int64_t);

int main(int argc, char **argv) {
    void *h = argc > 1 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (h == nullptr) return 2;
    const size_fn size = (size_fn)dlsym(h, "nestedfp_gemm_workspace_size");
    const tune_fn tune = (tune_fn)dlsym(h, "nestedfp_tune");
    const int64_t M = 96, N = 5120, K = 32768;             // the table of timed shapes has another split than the cost model
    size_t want[2];
    for (int v = 0; v < 2; ++v) {
        tune("tuned_table", v - 1);
        want[v] = size(M, N, K, 0);
    }
    if (want[0] == want[1]) return 3;
    // the other thread asks all the time, and once more after each change
    std::atomic<int> asked{0}, answered{0};
    std::atomic<size_t> answer{0};
    std::atomic<bool> stop{false};
    std::thread other([&] {
        while (!stop.load()) {
            const int q = asked.load();
            const size_t s = size(M, N, K, 0);
            if (answered.load() != q) { answer.store(s);  answered.store(q); }
        }
    });
    int stale = 0;
    for (int i = 1; i <= 100000; ++i) {
        const int v = i & 1;
        tune("tuned_table", v - 1);
        asked.store(i);
        while (answered.load() != i) {}
        stale += answer.load() != want[v];
    }
    stop.store(true);
    other.join();
    printf("%d stale answers\n", stale);
    return stale ? 1 : 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a C++ compiler")
def test_a_changed_knob_reaches_threads_that_remember_launch_shapes(tmp_path):
    from paper_2506_02024_amd import binding, build

    if build.is_stale():
        build.build_library()
    binding.lib()                                          # (the library loads)
    src, exe = tmp_path / "knobs.cpp", tmp_path / "knobs"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", str(src), "-o", str(exe), "-ldl"], check=True)
    lib = os.environ.get("NESTEDFP_LIB") or build.lib_path()
    res = subprocess.run([str(exe), lib], capture_output=True, text=True, timeout=100)
    assert res.returncode == 0, res.stdout + res.stderr
