"""CPU: host-side units of the library, compiled with g++ into small programs."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1302_5010_amd", "csrc")


def _run(tmp_path, source, *flags):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "unit.cpp", tmp_path / "unit"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", *flags, "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr


def test_arena_list_updates_do_not_depend_on_the_host_list(tmp_path):
    """Chunks reach the device through the stream, after kernels that the host has enqueued already, while the host
    goes on and adds the next one.  A stream of deferred operations stands for the device: between any two of them its
    list holds whole entries only, those of the chunks taken over so far."""
    _run(tmp_path, r"""
#include <cstdio>
#include <functional>
#include <vector>
#include "arena_list.h"
using namespace bmpl;
int main()
{
    Arena host{}, dev{};
    std::vector<std::function<void()>> stream;
    static double mem[ARENA_CHUNKS];
    for (int k = 0; k < ARENA_CHUNKS; ++k) {
        const ArenaChunk c = arena_next(host, mem + k, 100 + k);
        arena_put(host, c);
        stream.push_back([c, &dev] { arena_put(dev, c); });
    }
    unsigned long long at = 0;
    for (int k = 0; k < ARENA_CHUNKS; ++k) {
        if (dev.nchunks != k || dev.base[k] != nullptr) { std::printf("chunk %d came early\n", k); return 1; }
        stream[k]();
        if (dev.nchunks != k + 1 || dev.base[k] != mem + k || dev.start[k] != at || dev.size[k] != 100ull + k) {
            std::printf("chunk %d is not whole\n", k);
            return 1;
        }
        at += dev.size[k];
    }
    return 0;
}
""")


def test_block_pool_bounds_and_no_allocation_of_its_own(tmp_path):
    """The pool of device blocks against stand-ins for hipMalloc and hipFree, with every C++ allocation failing (a
    context's destruction passes through it, and nothing may leave a C entry point as an exception): best fit within an
    eighth, the bounds in bytes and blocks with the oldest leaving first, ageing, dropping one device and all, and a
    failed device allocation tried again after a drop.  Every block is freed exactly once."""
    hip = tmp_path / "hip"
    hip.mkdir()
    (hip / "hip_runtime.h").write_text("""
#pragma once
#include <cstddef>
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
hipError_t hipMalloc(void**, size_t);
hipError_t hipFree(void*);
hipError_t hipGetLastError();
""")
    _run(tmp_path, r"""
#include <cstdio>
#include <cstdlib>
#include <new>
#include "block_pool.h"
static bool no_new = false;
void* operator new(size_t n) { if (no_new) throw std::bad_alloc(); return std::malloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
static char mem[4096];
static int at = 0, live = 0;
static bool state[4096], fail_once = false;
hipError_t hipMalloc(void** p, size_t)
{
    if (fail_once) { fail_once = false; return hipErrorOutOfMemory; }
    state[at] = true; ++live; *p = mem + at++;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    const int i = (int)((char*)p - mem);
    if (!state[i]) { std::printf("freed twice\n"); std::exit(1); }
    state[i] = false; --live;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
using namespace bmpl;
int main()
{
    BlockPool& pool = block_pool();
    no_new = true;
    void* p[200]; size_t got = 0;
    // best fit within an eighth, on its own device only
    const size_t sizes[3] = {800, 1000, 1100};
    for (int i = 0; i < 3; ++i) CHECK(pool.take(0, &p[i], sizes[i], &got) == hipSuccess && got == sizes[i]);
    for (int i = 0; i < 3; ++i) pool.put(0, p[i], sizes[i]);
    void* q = nullptr;
    CHECK(pool.take(1, &q, 1000, &got) == hipSuccess && q != p[1]);
    pool.put(1, q, got);
    CHECK(pool.take(0, &q, 990, &got) == hipSuccess && q == p[1] && got == 1000);
    CHECK(pool.take(0, &q, 990, &got) == hipSuccess && q == p[2] && got == 1100);
    CHECK(pool.take(0, &q, 600, &got) == hipSuccess && q != p[0]);
    CHECK(hipFree(q) == hipSuccess);
    pool.put(0, p[1], 1000);
    pool.put(0, p[2], 1100);
    CHECK(pool.kept(0) == 2900 && pool.kept(1) == 1000 && live == 4);
    // a failed allocation gives the device's blocks back and is tried again
    fail_once = true;
    CHECK(pool.take(0, &q, 5000, &got) == hipSuccess && pool.kept(0) == 0 && pool.kept(1) == 1000 && live == 2);
    pool.put(0, q, got);
    CHECK(pool.drop(-1) && !pool.drop(-1) && live == 0);
    // the bound in bytes: the oldest leave first; a block above it never stays
    const size_t third = POOL_BYTES / 3;
    for (int i = 0; i < 4; ++i) CHECK(pool.take(0, &p[i], third, &got) == hipSuccess);
    for (int i = 0; i < 4; ++i) pool.put(0, p[i], third);
    CHECK(pool.kept(0) == 3 * third && live == 3 && !state[(char*)p[0] - mem]);
    CHECK(pool.take(0, &q, POOL_BYTES + 1, &got) == hipSuccess);
    pool.put(0, q, POOL_BYTES + 1);
    CHECK(live == 3);
    // ageing, per device
    for (int i = 0; i < POOL_AGE; ++i) pool.age(0);
    CHECK(live == 3);
    pool.age(1);
    CHECK(live == 3);
    pool.age(0);
    CHECK(live == 0 && pool.kept(0) == 0);
    // the bound in blocks
    for (int i = 0; i < POOL_BLOCKS + 20; ++i) CHECK(pool.take(0, &p[i], 16, &got) == hipSuccess);
    for (int i = 0; i < POOL_BLOCKS + 20; ++i) pool.put(0, p[i], 16);
    CHECK(live == POOL_BLOCKS && !state[(char*)p[19] - mem] && state[(char*)p[20] - mem]);
    CHECK(pool.drop(0) && live == 0);
    return 0;
}
""", "-I", str(tmp_path))


def test_failed_allocation_leaves_no_error_behind(tmp_path):
    """dalloc and the pool against a device without memory, with a runtime that keeps the last error until it is asked
    for it: the status says that there was none, and the next launch check of any call must not find it."""
    hip = tmp_path / "hip"
    hip.mkdir()
    (hip / "hip_runtime.h").write_text("""
#pragma once
#include <cstddef>
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
inline hipError_t& last() { static hipError_t e = hipSuccess; return e; }
inline hipError_t hipMalloc(void**, size_t) { return last() = hipErrorOutOfMemory; }
inline hipError_t hipFree(void*) { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipGetLastError() { const hipError_t e = last(); last() = hipSuccess; return e; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
""")
    _run(tmp_path, r"""
#include "host_util.h"
int main()
{
    double* p = nullptr;
    if (bmpl::dalloc(&p, 10) != hipErrorOutOfMemory || hipGetLastError() != hipSuccess) return 1;
    void* q = nullptr;
    size_t got = 0;
    if (bmpl::block_pool().take(0, &q, 10, &got) != hipErrorOutOfMemory || hipGetLastError() != hipSuccess) return 2;
    return 0;
}
""", "-I", str(tmp_path), "-Wno-unused")
