"""Memory kept between calls (csrc/pool.cpp) against a stand-in for the driver
that counts blocks and has a capacity."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2005_03070_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <new>
#include <unordered_map>
#include "pool.h"

static size_t capacity = (size_t)8 << 30, used = 0;
static std::unordered_map<char*, size_t> blocks;
static char* next_block = (char*)0x100000000;
static int wrong_frees = 0;
// (hip_runtime_api.h also has a hipMalloc template that calls this one)
extern "C" hipError_t hipMalloc(void** p, size_t n) {
    if (used + n > capacity) return hipErrorOutOfMemory;
    *p = next_block;
    blocks[next_block] = n;
    next_block += n;
    used += n;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void* p) {
    auto it = blocks.find((char*)p);
    if (it == blocks.end()) {
        ++wrong_frees;
        return hipErrorInvalidValue;
    }
    used -= it->second;
    blocks.erase(it);
    return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }

// host memory that runs out on request
static bool no_host_memory = false;
void* operator new(size_t n) {
    void* p = no_host_memory ? nullptr : malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

using namespace tgdk;
static const size_t MiB = (size_t)1 << 20;
#define CHECK(c)                                          \
    do {                                                  \
        if (!(c)) {                                       \
            printf("line %d: %s\n", __LINE__, #c);        \
            exit(1);                                      \
        }                                                 \
    } while (0)
static void keep(DevPool& p, size_t bytes) { p.put(p.get(bytes)); }

int main() {
    BODY
    CHECK(wrong_frees == 0);
    printf("ok\n");
    return 0;
}
"""


def _run(tmp_path, body):
    src, exe = tmp_path / "pool_test.cpp", tmp_path / "pool_test"
    src.write_text(DRIVER.replace("BODY", body))
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    str(src), os.path.join(CSRC, "pool.cpp"), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_a_failing_allocation_gets_what_is_held_free(tmp_path):
    """Every allocation of the library goes through dev_malloc: one that does
    not fit beside the blocks that pools of its device hold free takes theirs;
    another device's stay, and so do blocks in use."""
    _run(tmp_path, r"""
    capacity = 3000 * MiB;
    DevPool a(0), b(0), other(1);
    void* in_use = a.get(100 * MiB);
    keep(a, 600 * MiB);
    keep(b, 700 * MiB);
    keep(other, 800 * MiB);
    CHECK(used == 2200 * MiB);
    void* p = nullptr;
    CHECK(dev_malloc(0, &p, 1500 * MiB) == hipSuccess && p);
    CHECK(used == 2400 * MiB && blocks.size() == 3);  // in_use, the other device's, p
    CHECK(blocks.count((char*)in_use) == 1);
    void* q = p;
    CHECK(dev_malloc(0, &q, 5000 * MiB) == hipErrorOutOfMemory && !q);
    CHECK(a.get(5000 * MiB) == nullptr);
    hipFree(p);
    a.put(in_use);
    """)


def test_blocks_are_reused_bounded_and_age(tmp_path):
    _run(tmp_path, r"""
    capacity = (size_t)64 << 30;
    {
        DevPool a(0);
        void* p = a.get(800 * MiB);
        a.put(p);
        CHECK(a.get(700 * MiB) == p);             // an eighth less fits
        a.put(p);
        void* q = a.get(699 * MiB);               // less does not
        CHECK(q != p);
        a.put(q);
        keep(a, 900 * MiB);
        CHECK(used <= POOL_BYTES);
        keep(a, 3000 * MiB);                      // more than the bound goes back at once
        CHECK(used <= POOL_BYTES);
        for (unsigned i = 0; i < 2 * POOL_AGE; ++i) keep(a, 1 * MiB);
        CHECK(used <= 2 * MiB);
    }
    CHECK(used == 0);
    """)


def test_the_contexts_of_a_device_share_one_bound(tmp_path):
    """Eight pools of one device and one of another: together the eight hold at
    most the bound, the block that waits longest goes first, and flush() hands
    back one pool's."""
    _run(tmp_path, r"""
    capacity = (size_t)64 << 30;
    std::unique_ptr<DevPool> p[8];
    for (auto& q : p) q.reset(new DevPool(0));
    DevPool other(1);
    keep(other, 1024 * MiB);
    void* first = p[0]->get(512 * MiB);
    p[0]->put(first);
    for (int i = 1; i < 8; ++i) keep(*p[i], 512 * MiB);
    CHECK(used == POOL_BYTES + 1024 * MiB);
    CHECK(blocks.count((char*)first) == 0);
    void* last = p[7]->get(512 * MiB);
    CHECK(used == POOL_BYTES + 1024 * MiB);   // (it had stayed)
    p[7]->put(last);
    p[6]->flush();
    CHECK(used == POOL_BYTES + 512 * MiB);
    p[7].reset();
    CHECK(used == POOL_BYTES);
    """)


def test_without_host_memory_blocks_go_back_and_nothing_is_thrown(tmp_path):
    """get() and put() are called from C entry points (also from a garbage
    collector's thread): with no host memory for a block's record they return
    null and hand the block back."""
    _run(tmp_path, r"""
    DevPool a(0);
    void* p[3];
    for (void*& q : p) q = a.get(10 * MiB);
    a.put(p[0]);
    blocks.reserve(64);                   // (the stand-in's own table)
    const size_t before = used;
    no_host_memory = true;
    CHECK(a.get(10 * MiB) == nullptr);    // the kept block cannot be recorded as taken
    a.put(p[1]);
    a.put(p[2]);
    no_host_memory = false;
    CHECK(used <= before);
    for (int i = 0; i < 8; ++i) keep(a, 10 * MiB);
    CHECK(used == 10 * MiB || used == 20 * MiB || used == 30 * MiB);
    CHECK(a.get(10 * MiB) != nullptr);
    """)


def test_a_closed_pool_keeps_nothing(tmp_path):
    _run(tmp_path, r"""
    DevPool a(0);
    void *p = a.get(10 * MiB), *q = a.get(10 * MiB);
    a.put(p);
    a.close();
    CHECK(used == 10 * MiB);
    a.put(q);
    CHECK(used == 0);
    """)
