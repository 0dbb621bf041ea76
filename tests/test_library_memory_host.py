"""Host side of the library against a stand-in for the HIP runtime (two devices, kernels that run on the CPU when their
stream is waited for, calls that can be made to fail): memory of the library's own, and which kernels are launched.
Needs no GPU."""
import os
import shutil
import subprocess

import pytest

SOURCE = r"""
#include <dlfcn.h>
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <deque>
#include <functional>
#include <map>
#include <string>
#include <utility>

// ---- the stand-in: exported by the program, so the library binds to it ----------------------------------------------
struct Dim3 { uint32_t x, y, z; };
static const int kFail = 1;
static int current = 0;                                        // current device
static bool fail_wait, fail_pinned, fail_copy;
static int fail_launch;                                        // 1: refused; 2: an earlier error is reported, the kernel is queued
static int last_error, copies, launches, wrong_device, scratch_uses;
static uint64_t bad_weights;                                   // what a counting kernel finds
static std::deque<std::function<void()>> queued;
static std::map<const void *, std::string> kernels;
static std::map<const void *, size_t> variables;
static std::map<std::pair<int, const void *>, char *> images;  // a variable's copy on a device
static std::string last_gemm;                                  // name of the last GEMM kernel
static std::pair<void *, void *> last_copy;                    // where, from where

static void *stream_of(int dev) { return reinterpret_cast<void *>((intptr_t)0x1000 + dev); }
static int device_of(void *stream) { return stream == nullptr ? current : (int)(reinterpret_cast<intptr_t>(stream) - 0x1000); }
static int owner(const void *p) {                              // the device whose image holds p, -1: none
    for (auto &i : images)
        if ((const char *)p >= i.second && (const char *)p < i.second + variables[i.first.second]) return i.first.first;
    return -1;
}
static void run_queued() {
    while (!queued.empty()) { auto f = queued.front();  queued.pop_front();  f(); }
}
static bool on_stack(const void *p) {
    pthread_attr_t a;
    void *base = nullptr;
    size_t size = 0;
    pthread_getattr_np(pthread_self(), &a);
    pthread_attr_getstack(&a, &base, &size);
    pthread_attr_destroy(&a);
    return (const char *)p >= (char *)base && (const char *)p < (char *)base + size;
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *m;  return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[host] = name; }
void __hipRegisterVar(void **, void *var, char *, char *, int, size_t size, int, int) { variables[var] = size; }
static Dim3 grid_, block_;
static size_t shared_;
static void *stream_;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t s, void *st) { grid_ = g;  block_ = b;  shared_ = s;  stream_ = st;  return 0; }
int __hipPopCallConfiguration(Dim3 *g, Dim3 *b, size_t *s, void **st) { *g = grid_;  *b = block_;  *s = shared_;  *st = stream_;  return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *d) { *d = current;  return 0; }
int hipSetDevice(int d) { current = d;  return 0; }
int hipStreamGetDevice(void *s, int *d) { *d = device_of(s);  return 0; }
int hipGetLastError() { const int e = last_error;  last_error = 0;  return e; }
int hipGetSymbolAddress(void **p, const void *var) {
    char *&image = images[{current, var}];
    if (image == nullptr) image = (char *)calloc(1, variables[var]);
    *p = image;
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned) {
    if (fail_pinned) return last_error = kFail;
    *p = calloc(1, n);
    return 0;
}
int hipMemcpyAsync(void *to, const void *from, size_t n, int, void *) {
    if (fail_copy) return kFail;
    ++copies;
    last_copy = {to, const_cast<void *>(from)};
    queued.push_back([=] { memcpy(to, from, n); });
    return 0;
}
int hipStreamSynchronize(void *) {
    if (fail_wait) return kFail;
    run_queued();
    return 0;
}
int hipLaunchKernel(const void *f, Dim3, Dim3, void **args, size_t, void *stream) {
    if (fail_launch == 1) return last_error = kFail;
    if (fail_launch == 2) last_error = kFail;
    ++launches;
    const std::string &name = kernels[f];
    auto arg = [&](int i) { return *static_cast<uint64_t **>(args[i]); };
    auto look = [&](const void *p) { if (owner(p) >= 0 && owner(p) != device_of(stream)) ++wrong_device; };
    if (name.find("hand_on_count") != std::string::npos) {
        uint64_t *counter = arg(0), *dev = arg(1), *host = arg(2);
        look(counter);
        queued.push_back([=] { *dev = *host = *counter;  *counter = 0; });
    } else if (name.find("zero_u64") != std::string::npos) {
        uint64_t *p = arg(0);
        look(p);
        queued.push_back([=] { *p = 0; });
    } else if (name.find("zero_words") != std::string::npos) {
        look(arg(0));
    } else if (name.find("range_check") != std::string::npos || name.find("decompose") != std::string::npos) {
        uint64_t *counter = arg(name.find("range_check") != std::string::npos ? 3 : (name.find("decompose_rows") != std::string::npos ? 6 : 5));
        look(counter);
        const uint64_t n = bad_weights;
        if (counter) queued.push_back([=] { *counter += n; });
    } else if (name.find("quantize_act") != std::string::npos || name.find("splitk_reduce") != std::string::npos) {
        for (int i : {0, 3, 4, 5}) {
            if (i > 0 && name.find("splitk_reduce") != std::string::npos) break;
            look(arg(i));
        }
    } else if (name.find("gemm_kernel") != std::string::npos || name.find("bypass") != std::string::npos ||
               name.find("nested_rows") != std::string::npos) {
        last_gemm = name;
        for (int i = 0; i < 15; ++i) {                         // the pointers among the first 120 bytes of its parameters
            void *const p = static_cast<void **>(args[0])[i];
            look(p);
            scratch_uses += owner(p) >= 0;
        }
    } else {
        fprintf(stderr, "unknown kernel %s\n", name.c_str());
        exit(3);
    }
    return 0;
}
}

// ---- the calls --------------------------------------------------------------------------------------------------------
struct Layer { int64_t N, K; int32_t is_exception, layout; const void *upper, *lower, *W; int64_t ldw; uint64_t out_of_range; };
static int (*range_check)(const void *, int64_t, int64_t, int64_t, uint64_t *, uint64_t *, void *);
static int (*decompose)(const void *, int64_t, int64_t, int64_t, void *, void *, uint64_t *, uint64_t *, void *);
static int (*prepare)(const void *, int64_t, int64_t, int64_t, int, void *, void *, uint64_t *, Layer *, void *);
static int (*gemm_static)(const void *, int64_t, int64_t, int64_t, const void *, const void *, int64_t, int, const float *, void *, int64_t, void *);
static int (*gemm_packed)(const void *, int64_t, int64_t, int64_t, const void *, const void *, int64_t, int, const float *, void *, int64_t, void *, size_t, void *);
static int (*tune)(const char *, int64_t);
static char W[4096] __attribute__((aligned(16))), up[4096] __attribute__((aligned(16))), lo[4096] __attribute__((aligned(16)));

static int failures;
#define CHECK(x) do { if (!(x)) { ++failures;  printf("line %d: %s\n", __LINE__, #x); } } while (0)
enum { OK = 0, ERR_RANGE = 3, ERR_HIP = 5 };

// every entry point that waits for a count: right on the device, right on the host
static void all_right(void *stream) {
    for (uint64_t n : {(uint64_t)0, (uint64_t)7, (uint64_t)0, (uint64_t)3}) {
        bad_weights = n;
        uint64_t dev = 99, host = 99;
        const int want = n ? ERR_RANGE : OK;
        CHECK(range_check(W, 4, 32, 32, &dev, &host, stream) == want && dev == n && host == n);
        dev = host = 99;
        CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream) == want && dev == n && host == n);
        Layer layer;
        for (int layout : {0, 1}) {
            dev = 99;
            CHECK(prepare(W, 4, 32, 32, layout, up, lo, &dev, &layer, stream) == OK && dev == n);
            CHECK(layer.out_of_range == n && layer.is_exception == (n ? 1 : 0));
        }
        dev = host = 99;
        CHECK(decompose(nullptr, 0, 32, 32, nullptr, nullptr, &dev, &host, stream) == OK && dev == 0 && host == 0);
        dev = 99;
        CHECK(decompose(W, 4, 32, 32, up, lo, &dev, nullptr, stream) == OK);       // no wait: the caller's own
        run_queued();
        CHECK(dev == n);
    }
}

// a stream's device need not be the current one
static void streams_of_two_devices() {
    for (int dev : {1, 0, 1}) {
        all_right(stream_of(dev));
        CHECK(current == 0);
    }
    all_right(nullptr);
    current = 1;
    all_right(nullptr);
    all_right(stream_of(0));
    CHECK(current == 1 && wrong_device == 0 && copies == 0);
}

// no pinned memory: the count takes the way through the caller's device word; where the wait fails the copy may come later
static void without_pinned_words() {
    fail_pinned = true;
    for (int dev : {0, 1}) all_right(stream_of(dev));
    CHECK(copies > 0);
    uint64_t dev = 99, host = 98;
    Layer layer;
    bad_weights = 7;
    for (int call = 0; call < 3; ++call) {
        fail_wait = true;
        last_copy = {};
        CHECK((call == 0 ? decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) :
               call == 1 ? range_check(W, 4, 32, 32, &dev, &host, stream_of(0)) :
                           prepare(W, 4, 32, 32, 0, up, lo, &dev, &layer, stream_of(0))) == ERR_HIP);
        CHECK(last_copy.first != nullptr && !on_stack(last_copy.first));
        if (on_stack(last_copy.first)) queued.clear();
        fail_wait = false;
        run_queued();
    }
    fail_copy = true;
    CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) == ERR_HIP);
    fail_copy = false;
    all_right(stream_of(1));
}

// A launch that fails costs no word, however often: neither one that was refused nor one behind an earlier call's error, whose
// kernels run and leave a counter that is not zero.  A wait that fails keeps its word, to which a count may still come.
static void failing_calls() {
    uint64_t dev = 99, host = 99;
    Layer layer;
    for (int kind : {1, 2})
        for (int i = 0; i < 200; ++i) {
            bad_weights = 5;
            fail_launch = kind;
            void *const stream = stream_of(i % 2);
            CHECK((i % 3 == 0 ? decompose(W, 4, 32, 32, up, lo, &dev, &host, stream) :
                   i % 3 == 1 ? range_check(W, 4, 32, 32, &dev, &host, stream) :
                                prepare(W, 4, 32, 32, 1, up, lo, &dev, &layer, stream)) == ERR_HIP);
            fail_launch = 0;
            last_error = 0;
            if (i % 50 == 0) all_right(stream_of(i / 50 % 2));
        }
    all_right(stream_of(0));
    all_right(stream_of(1));
    CHECK(copies == 0);
    // (a launch behind an earlier error whose wait fails as well: its kernels are still to come)
    fail_wait = true;
    fail_launch = 2;
    CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) == ERR_HIP);
    fail_launch = last_error = 0;
    for (int i = 0; i < 20; ++i) CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) == ERR_HIP);
    fail_wait = false;
    auto late = queued;
    queued.clear();
    for (uint64_t n : {(uint64_t)3, (uint64_t)0}) {
        bad_weights = n;
        dev = host = 99;
        CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) == (n ? ERR_RANGE : OK) && dev == n && host == n);
        for (auto &f : late) f();
    }
    all_right(stream_of(0));
    CHECK(copies == 0);
    // ... until there is none left, and the counts take the other way
    fail_wait = true;
    for (int i = 0; i < 100; ++i) CHECK(decompose(W, 4, 32, 32, up, lo, &dev, &host, stream_of(0)) == ERR_HIP);
    fail_wait = false;
    CHECK(copies > 0);
    run_queued();
    all_right(stream_of(0));
    all_right(stream_of(1));
}

// the call without a workspace: its scratch is the stream's device's
static void fixed_scratch_on_two_devices() {
    static char X[1 << 20] __attribute__((aligned(16))), Y[1 << 20] __attribute__((aligned(16)));
    for (void *stream : {stream_of(1), stream_of(0), stream_of(1), (void *)nullptr})
        for (int mode : {0, 1})
            for (int64_t M : {1, 16, 40, 300}) {
                const int before = scratch_uses;
                CHECK(gemm_static(X, M, 14336, 14336, W, W, 4096, mode, nullptr, Y, 4096, stream) == OK);
                CHECK(scratch_uses > before || (mode == 0 && M != 40));
                CHECK(current == 0);
            }
    // a split that does not fit is not taken: the call is
    CHECK(gemm_static(X, 256, 5872, 5872, W, W, 17616, 0, nullptr, Y, 17616, stream_of(0)) == OK);
    CHECK(wrong_device == 0 && scratch_uses > 0);
}

// Packed weights on 64-token tiles: marked non-temporal with one token tile, on small layers, and where the weight tiles are a
// multiple of eight (FP16 mode: below 64 Mi weights).
static void non_temporal_weights() {
    static char ws[8 << 20] __attribute__((aligned(16))), X[16 << 20] __attribute__((aligned(16)));
    tune("small_max_m", 0);
    tune("large_bm", 64);
    tune("large_split", 1);
    struct { int64_t M, N, K;  bool fp16, fp8; } const cases[] = {
        {33, 5696, 5696, true, true}, {64, 5696, 5696, true, true}, {65, 5696, 5696, false, false}, {256, 5696, 5696, false, false},
        {200, 2000, 1024, true, true}, {200, 2944, 1536, false, false},       // 1.95 and 4.3 Mi weights in 16 and 23 tiles
        {200, 2049, 1024, true, true}, {256, 8192, 4096, true, true}, {256, 8192, 8192, false, true}};
    for (const auto &c : cases) {
        CHECK(gemm_packed(X, c.M, c.K, c.K, W, W, c.N, 0, nullptr, X, (c.N + 3) & ~3, ws, sizeof(ws), nullptr) == OK);
        CHECK(last_gemm.find(c.fp16 ? "nested_bypass_kernelILi64ELi128ELi1ELb0ELb1ELb0E" : "nested_bypass_kernelILi64ELi128ELi1ELb0ELb0ELb0E") != std::string::npos);
        CHECK(gemm_packed(X, c.M, c.K, c.K, W, W, c.N, 1, nullptr, X, (c.N + 3) & ~3, ws, sizeof(ws), nullptr) == OK);
        CHECK(last_gemm.find(c.fp8 ? "e4m3_bypass_kernelILi64ELi128ELb0ELb1E" : "e4m3_bypass_kernelILi64ELi128ELb0ELb0E") != std::string::npos);
    }
    tune("small_max_m", -1);
    tune("large_bm", -1);
    tune("large_split", -1);
}

int main(int argc, char **argv) {
    void *h = argc > 2 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (h == nullptr) { fprintf(stderr, "%s\n", dlerror());  return 2; }
    *(void **)&range_check = dlsym(h, "nestedfp_range_check");
    *(void **)&decompose = dlsym(h, "nestedfp_decompose");
    *(void **)&prepare = dlsym(h, "nestedfp_layer_prepare");
    *(void **)&gemm_static = dlsym(h, "nestedfp_gemm_static");
    *(void **)&gemm_packed = dlsym(h, "nestedfp_gemm_packed");
    *(void **)&tune = dlsym(h, "nestedfp_tune");
    const std::string what = argv[2];
    if (what == "streams_of_two_devices") streams_of_two_devices();
    else if (what == "without_pinned_words") without_pinned_words();
    else if (what == "failing_calls") failing_calls();
    else if (what == "fixed_scratch_on_two_devices") fixed_scratch_on_two_devices();
    else if (what == "non_temporal_weights") non_temporal_weights();
    else return 2;
    if (launches == 0) return 2;                               // (the library bound to the real runtime)
    return failures ? 1 : 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs a C++ compiler")
    from paper_2506_02024_amd import build

    if build.is_stale():
        build.build_library()
    folder = tmp_path_factory.mktemp("host")
    src, exe = folder / "host.cpp", folder / "host"
    src.write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", "-pthread", str(src), "-o", str(exe), "-ldl"], check=True)
    return [str(exe), os.environ.get("NESTEDFP_LIB") or build.lib_path()]


@pytest.mark.parametrize("what", ["streams_of_two_devices", "without_pinned_words", "failing_calls", "fixed_scratch_on_two_devices", "non_temporal_weights"])
def test_host_side(program, what):
    res = subprocess.run(program + [what], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0, res.stdout + res.stderr
