"""The pinned read-back stage (csrc/lhmm_stage.h) on the CPU, compiled against
a small model of the runtime calls it makes: copies and kernels on a stream
run as late as the runtime may run them (when an event or the stream is waited
for), events and streams belong to a device, a null stream is the current
device's, freed pinned memory must not be a pending operation's target.

* every part arrives whole, for one to five parts of any size around the
  stage's pieces, in the address range that was allocated;
* a read waits for the stream also where it copies nothing;
* a read gives the same with another device current, and leaves it current;
* an error of the runtime is returned, with nothing left that writes to the
  stage.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#pragma once
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidHandle = 400 };
enum { hipMemcpyDeviceToHost = 2, hipEventDisableTiming = 2 };
struct Op {
    std::function<void()> run;
    char* dst;
    size_t bytes;
};
struct Stream {
    int device = 0;
    std::deque<Op> ops;
    size_t finished = 0;
};
struct Event {
    int device = 0;
    Stream* s = nullptr;
    size_t upto = 0;
};
typedef Stream* hipStream_t;
typedef Event* hipEvent_t;
inline int g_device = 0, g_fail_copy = -1;
inline Stream g_null[2] = {{0, {}, 0}, {1, {}, 0}};
inline std::map<char*, size_t> g_pinned;
inline void check(bool ok, const char* what) {
    if (ok) return;
    printf("FAILED: %s\n", what);
    exit(1);
}
inline Stream* stream_of(hipStream_t s) { return s ? s : &g_null[g_device]; }
inline void drain(Stream* s, size_t upto) {
    while (s->finished < upto && !s->ops.empty()) {
        s->ops.front().run();
        s->ops.pop_front();
        s->finished += 1;
    }
}
inline hipError_t hipGetDevice(int* d) { return *d = g_device, hipSuccess; }
inline hipError_t hipSetDevice(int d) {
    if (d < 0 || d > 1) return hipErrorInvalidValue;
    return g_device = d, hipSuccess;
}
inline bool inside_pinned(const char* p, size_t n) {
    auto it = g_pinned.upper_bound((char*)p);
    return it != g_pinned.begin() && (--it, p + n <= it->first + it->second);
}
inline hipError_t enqueue(hipStream_t st, char* dst, size_t n, std::function<void()> run) {
    check(inside_pinned(dst, n), "an operation writes outside the pinned memory");
    stream_of(st)->ops.push_back({run, dst, n});
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, int, hipStream_t st) {
    if (g_fail_copy >= 0 && g_fail_copy-- == 0) return hipErrorInvalidValue;
    check(n > 0, "an empty copy");
    return enqueue(st, (char*)dst, n, [=] { memcpy(dst, src, n); });
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return *e = new Event{g_device, nullptr, 0}, hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t e) { return delete e, hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
    Stream* s = stream_of(st);
    if (e->device != s->device) return hipErrorInvalidHandle;
    e->s = s;
    e->upto = s->finished + s->ops.size();
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) { return drain(e->s, e->upto), hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t st) { return drain(stream_of(st), (size_t)-1), hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n) {
    *p = malloc(n);
    g_pinned[(char*)*p] = n;
    return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
    const size_t n = g_pinned.at((char*)p);
    for (Stream& s : g_null)
        for (Op& o : s.ops) check(o.dst + o.bytes <= (char*)p || o.dst >= (char*)p + n, "pinned memory freed under a pending operation");
    g_pinned.erase((char*)p);
    memset(p, 0xA5, n);
    free(p);
    return hipSuccess;
}
"""

PROGRAM = r"""
#include <random>
#include <string>
#include <vector>
#include "lhmm_stage.h"
using Bytes = std::vector<char>;
std::mt19937 rng(5);
Bytes random_bytes(size_t n) {
    Bytes b(n);
    for (char& x : b) x = (char)rng();
    return b;
}
void parts_arrive() {
    HostStage st;
    check(st.reserve(0) == hipSuccess, "reserve");
    const size_t H = HostStage::HALF;
    const size_t sizes[] = {4, 8, 12, 16, 100, H - 16, H - 4, H, H + 4, 2 * H - 8, 2 * H, 2 * H + 12, 3 * H + 20, 36000};
    for (int round = 0; round < 400; ++round) {
        const int n = 1 + (int)(rng() % 5);
        std::vector<Bytes> src, dst;
        HostStage::Part parts[5];
        for (int k = 0; k < n; ++k) {
            const size_t b = rng() % 2 ? sizes[rng() % 14] : 4 + 4 * (rng() % 90000);
            src.push_back(random_bytes(b));
            dst.push_back(Bytes(b));
        }
        for (int k = 0; k < n; ++k) parts[k] = {src[k].data(), src[k].size()};
        std::vector<size_t> got(n, 0);
        check(st.read(nullptr, parts, n, [&](int k, size_t at, size_t len, const char* x) {
            check(at == got[k] && at + len <= dst[k].size() && at % 16 == 0, "pieces of a part come in order");
            memcpy(dst[k].data() + at, x, len);
            got[k] += len;
        }) == hipSuccess, "read");
        for (int k = 0; k < n; ++k) check(got[k] == src[k].size() && dst[k] == src[k], "part differs");
    }
    // a kernel that fills the stage, as the surrogate's weights do
    for (size_t total : {(size_t)4, H, H + 4, 5 * H + 8}) {
        const Bytes src = random_bytes(total);
        Bytes dst(total);
        check(st.run(nullptr, total,
                     [&](size_t o, size_t len, char* pinned) {
                         return enqueue(nullptr, pinned, len, [&src, o, len, pinned] { memcpy(pinned, src.data() + o, len); });
                     },
                     [&](size_t o, size_t len, const char* x) { memcpy(dst.data() + o, x, len); }) == hipSuccess, "run");
        check(dst == src, "filled stage differs");
    }
    st.release();
    check(g_pinned.empty(), "pinned memory given back");
}
void empty_read_waits() {
    HostStage st;
    check(st.reserve(64) == hipSuccess, "reserve");
    char x[16] = {};
    bool done = false;
    g_null[0].ops.push_back({[&] { done = true; }, nullptr, 0});
    check(st.copy(nullptr, {{x, sizeof x}, {x, sizeof x}}, {nullptr, nullptr}) == hipSuccess && done, "an empty read waits");
    st.release();
}
void other_device() {
    for (size_t reserved : {(size_t)0, (size_t)256}) {
        HostStage st;
        g_device = 0;
        check(st.reserve(reserved) == hipSuccess, "reserve");
        const Bytes src = random_bytes(1000);
        Bytes dst(1000), late(1000);
        g_null[0].ops.push_back({[&] { late = src; }, nullptr, 0});  // the engine's work before the read
        g_device = 1;
        void* const to[1] = {dst.data()};
        check(st.copy(nullptr, {{late.data(), late.size()}}, to) == hipSuccess, "read with another device current");
        check(dst == src, "the engine's data");
        check(g_device == 1, "the caller's device stays current");
        bool done = false;
        g_null[0].ops.push_back({[&] { done = true; }, nullptr, 0});
        void* const none[1] = {nullptr};
        check(st.copy(nullptr, {{late.data(), late.size()}}, none) == hipSuccess && done && g_device == 1, "empty read");
        g_device = 0;
        st.release();
    }
}
void errors() {
    HostStage st;
    check(st.reserve(0) == hipSuccess, "reserve");
    const Bytes src = random_bytes(4 * HostStage::HALF);
    Bytes dst(src.size());
    void* const to[1] = {dst.data()};
    for (int at = 0; at < 4; ++at) {
        g_fail_copy = at;
        check(st.copy(nullptr, {{src.data(), src.size()}}, to) == hipErrorInvalidValue, "the error is returned");
        check(g_null[0].ops.empty(), "nothing is pending after an error");
        g_fail_copy = -1;
    }
    check(st.copy(nullptr, {{src.data(), src.size()}}, to) == hipSuccess && dst == src, "the stage serves again");
    st.release();
}
int main(int, char** a) {
    const std::string what = a[1];
    if (what == "parts") parts_arrive();
    if (what == "empty") empty_read_waits();
    if (what == "device") other_device();
    if (what == "errors") errors();
    printf("ok\n");
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("stage")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (d / "main.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-I", str(d), "-I", os.path.join(ROOT, "paper_2512_13267_amd", "csrc"),
                    "-o", str(d / "main"), str(d / "main.cpp"), "-pthread"], check=True)
    return str(d / "main")


@pytest.mark.parametrize("what", ["parts", "empty", "device", "errors"])
def test_read_back_stage(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout + res.stderr
