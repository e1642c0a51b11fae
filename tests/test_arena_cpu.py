"""Device-memory arenas (csrc/arena.cpp) on the host: compiled with a device allocator of a
fixed size that hands out host memory, so that every request, refusal and free is seen.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2512_22215_amd", "csrc")
HIP = "/opt/rocm/include"

HEAD = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <map>
#include "arena.hpp"
#include "ldu.h"
using namespace ldu;
static size_t room = 0;                  // bytes the device has left
static std::map<void *, size_t> live;
extern "C" hipError_t hipMalloc(void **p, size_t n) {
    if (n > room) return hipErrorOutOfMemory;
    room -= n;
    *p = std::malloc(n);
    live[*p] = n;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *p) {
    if (!live.count(p)) { std::printf("free of unknown memory\n"); std::exit(2); }
    room += live[p];
    live.erase(p);
    std::free(p);
    return hipSuccess;
}
extern "C" hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
extern "C" hipError_t hipGetLastError(void) { return hipSuccess; }
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
constexpr size_t MiB = size_t(1) << 20;
static bool refused(Arena &a, size_t n) {
    try { a.alloc(n); } catch (const Error &e) { return e.code == LDU_ERR_NOMEM; }
    return false;
}
"""

PROGRAMS = {
    # a step that fails part way leaves the arena as it was
    "step": r"""
int main() {
    room = 100 * MiB;
    Arena a;
    a.alloc(10 * MiB);
    a.alloc(2 * MiB);                        // 2 of 5
    void *first = nullptr;
    const size_t left = room;
    for (int k = 0; k < 50; ++k) {
        try {
            Arena::Step step(a);
            void *p = a.alloc(1 * MiB);      // in the rest of a chunk
            if (!first) first = p;
            CHECK(p == first);
            a.alloc(40 * MiB);               // a chunk of its own
            a.alloc(80 * MiB);
            step.done();
        } catch (const Error &) {
        }
        CHECK(room == left);
    }
    Arena::Step step(a);
    CHECK(a.alloc(1 * MiB) == first);
    a.alloc(40 * MiB);
    step.done();
    CHECK(room < left - 39 * MiB);
    return 0;
}
""",
    # a temporary arena gives its chunks back without asking for host memory
    "put": r"""
#include <new>
static bool no_host = false;
void *operator new(size_t n) {
    void *p = no_host ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
int main() {
    room = 1000 * MiB;
    ChunkPool pool;
    {
        Arena a(&pool), b(&pool);
        for (int k = 1; k < 9; ++k) (k % 2 ? a : b).alloc(k * MiB);
        no_host = true;
    }
    no_host = false;
    CHECK(room < 1000 * MiB);
    pool.trim();
    CHECK(room == 1000 * MiB);
    return 0;
}
""",
    # a settled arena asks for no more than its requests need
    "settled": r"""
int main() {
    room = 1000 * MiB;
    Arena a;
    a.alloc(200 * MiB);
    a.settle();
    size_t left = room;
    a.reserve(24 * MiB);
    a.alloc(8 * MiB); a.alloc(8 * MiB); a.alloc(8 * MiB);
    CHECK(room == left - 24 * MiB);
    a.alloc(1 * MiB);
    CHECK(room == left - 25 * MiB);
    return 0;
}
""",
    # a request that opens a new chunk leaves the rest of the others usable
    "rest": r"""
int main() {
    room = 1000 * MiB;
    Arena a;
    a.alloc(80 * MiB);
    a.alloc(30 * MiB);                       // a chunk of 40 MiB (half of what is held)
    const size_t left = room;
    a.alloc(45 * MiB);                       // one of 60 MiB
    CHECK(room < left);
    const size_t after = room;
    char *q = static_cast<char *>(a.alloc(14 * MiB));  // in the third chunk
    char *p = static_cast<char *>(a.alloc(9 * MiB));   // in the second
    char *s = static_cast<char *>(a.alloc(1));
    CHECK(room == after && p && q && s);
    a.reserve(300);
    CHECK(room == after);
    char *last = nullptr;                    // arrays of every chunk stay apart
    for (int k = 0; k < 64; ++k) {
        char *t = static_cast<char *>(a.alloc(300));
        CHECK(reinterpret_cast<size_t>(t) % 16 == 0 && t != last);
        for (int i = 0; i < 300; ++i) t[i] = 1;
        last = t;
    }
    p[9 * MiB - 1] = q[14 * MiB - 1] = 1;
    a.release_all();
    CHECK(room == 1000 * MiB && live.empty());
    return 0;
}
""",
    # free chunks of the pool go back before a request is refused
    "pool-first": r"""
int main() {
    room = 100 * MiB;
    ChunkPool pool;
    {
        Arena a;
        a.use_pool(&pool);
        { Arena tmp(&a); tmp.alloc(60 * MiB); }
        CHECK(room == 40 * MiB);             // kept for the next temporary
        a.alloc(70 * MiB);
        CHECK(room == 30 * MiB);
        { Arena tmp(&a); tmp.alloc(20 * MiB); }
        a.alloc_own(25 * MiB);
        CHECK(room == 5 * MiB);
        CHECK(refused(a, 6 * MiB));
        a.alloc(5 * MiB);
    }
    CHECK(room == 100 * MiB);
    { Arena tmp(&pool); tmp.alloc(60 * MiB); }
    { Arena tmp(&pool); tmp.alloc(90 * MiB); }   // the larger chunk in place of the smaller
    pool.trim();
    CHECK(room == 100 * MiB && live.empty());
    return 0;
}
""",
}


@pytest.mark.skipif(not shutil.which("g++") or not os.path.isdir(os.path.join(HIP, "hip")),
                    reason="needs g++ and the HIP headers")
@pytest.mark.parametrize("name", list(PROGRAMS))
def test_arena(name, tmp_path):
    src, exe = tmp_path / "arena_test.cpp", tmp_path / "arena_test"
    src.write_text(HEAD + PROGRAMS[name])
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", HIP,
                    "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-o", str(exe), str(src),
                    os.path.join(CSRC, "arena.cpp")], check=True, timeout=300)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
