"""The library's pool of device memory, compiled for the CPU against stand-ins for the six HIP calls that it makes: what it
keeps, when it waits for the device, when it gives memory back, and that it holds no lock meanwhile."""
import os
import subprocess

import pytest

from conftest import ROOT

STAND_IN = r"""
#pragma once
#include <cstddef>
enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidDevice = 101, hipErrorStreamCaptureUnsupported = 900 };
hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipFree(void *p);
hipError_t hipDeviceSynchronize();
hipError_t hipGetDevice(int *dev);
hipError_t hipMemGetInfo(size_t *free_bytes, size_t *total);
hipError_t hipGetLastError();
"""

DRIVER = r"""
#include "groot_pool.hip"

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <future>
#include <thread>
#include <vector>

static std::mutex dm;
static std::unordered_map<void *, size_t> live;
static size_t live_bytes = 0, total_bytes = (size_t)128 << 20;
static std::atomic<int> syncs{0}, frees{0}, mallocs{0};
static hipError_t sync_result = hipSuccess;
static std::function<void()> on_sync, on_free;
static thread_local int device = 0;

hipError_t hipMalloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> lock(dm);
    if (live_bytes + bytes > total_bytes) return hipErrorOutOfMemory;
    ++mallocs;
    *p = malloc(bytes < 64 ? 64 : bytes);
    live[*p] = bytes;
    live_bytes += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (on_free) on_free();
    std::lock_guard<std::mutex> lock(dm);
    if (!live.count(p)) { printf("freed twice\n"); exit(1); }
    live_bytes -= live[p];
    live.erase(p);
    free(p);
    ++frees;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize()
{
    if (on_sync) on_sync();
    ++syncs;
    return sync_result;
}
hipError_t hipGetDevice(int *dev) { *dev = device; return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = total_bytes - live_bytes; *t = total_bytes; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); exit(1); } } while (0)
static void *get(size_t bytes) { void *p = nullptr; CHECK(groot::dev_alloc(&p, bytes) == 0 && p); return p; }
constexpr size_t KB = 1024;                                  // 128 MB of memory: 1 MB is kept, in blocks of up to 128 KB

static bool others_may_go_on()                               // an allocation and a free on this device and on another one
{
    auto f = std::async(std::launch::async, [] {
        for (int dev = 0; dev < 2; ++dev) {
            device = dev;
            void *p = get(5 * KB);
            groot::dev_free(p);
        }
    });
    if (f.wait_for(std::chrono::seconds(5)) == std::future_status::ready) return true;
    printf("another thread waits for the pool\n");
    fflush(stdout);
    _Exit(1);
}

int main(int, char **argv)
{
    const std::string what = argv[1];
    void *const first = get(KB);                             // an object that stays
    if (what == "reuse") {
        void *a = get(64 * KB), *b = get(100 * KB);
        groot::dev_free(a);
        groot::dev_free(b);
        CHECK(syncs == 0 && frees == 0);                     // freeing waits for nothing
        CHECK(get(64 * KB) == a && syncs == 1);              // handed out after one wait
        CHECK(get(90 * KB) == b && syncs == 1);              // which served both; at most a quarter larger
        groot::dev_free(a);
        void *c = get(40 * KB);
        CHECK(c != a && syncs == 1);                         // too large by more than a quarter: a new block
        CHECK(get(64 * KB) == a && syncs == 2);              // freed after the last wait: another one
    } else if (what == "give_back") {
        void *a = get(64 * KB), *big = get(200 * KB);
        const size_t before = live_bytes;
        groot::dev_free(a);
        CHECK(live_bytes == before);                         // kept while another object lives
        groot::dev_free(big);
        CHECK(live_bytes == before - 200 * KB);              // above an eighth of the bound: not kept
        groot::dev_free(first);
        CHECK(live_bytes == 0 && live.empty());
        return 0;
    } else if (what == "bound") {
        std::vector<void *> p;
        for (int i = 0; i < 40; ++i) p.push_back(get(100 * KB));
        for (void *q : p) groot::dev_free(q);
        CHECK(live_bytes <= 1024 * KB + 1 + KB && live_bytes >= 900 * KB);
    } else if (what == "out_of_memory") {
        std::vector<void *> p;
        for (int i = 0; i < 10; ++i) p.push_back(get(100 * KB));
        for (void *q : p) groot::dev_free(q);
        void *big = get(total_bytes - 100 * KB);             // fits only without what is kept
        CHECK(live_bytes <= total_bytes);
        void *more = first;
        CHECK(groot::dev_alloc(&more, 200 * KB) == hipErrorOutOfMemory && more == nullptr);
        groot::dev_free(big);
        CHECK(live_bytes == KB);
    } else if (what == "wait_fails") {                       // a stream is being captured, say
        void *a = get(64 * KB);
        groot::dev_free(a);
        sync_result = hipErrorStreamCaptureUnsupported;
        CHECK(get(64 * KB) != a);
        sync_result = hipSuccess;
        CHECK(get(64 * KB) == a);
    } else if (what == "no_lock") {
        bool ok = false;
        void *a = get(64 * KB);
        groot::dev_free(a);
        on_sync = [&] { on_sync = nullptr; ok = others_may_go_on(); };
        CHECK(get(64 * KB) == a && ok);
        ok = false;
        void *big = get(200 * KB);
        on_free = [&] { on_free = nullptr; ok = others_may_go_on(); };
        groot::dev_free(big);
        CHECK(ok);
    } else if (what == "threads") {
        std::vector<std::thread> t;
        for (int k = 0; k < 8; ++k)
            t.emplace_back([k] {
                device = k % 2;
                unsigned seed = k;
                std::vector<std::pair<unsigned char *, size_t>> mine;
                for (int i = 0; i < 4000; ++i) {
                    seed = seed * 1664525u + 1013904223u;
                    if (mine.size() < 8 && (seed >> 8) % 2) {
                        const size_t n = 256 + (seed >> 12) % (150 * KB);
                        mine.emplace_back((unsigned char *)get(n), n);
                        memset(mine.back().first, k + 1, n);
                    } else if (!mine.empty()) {
                        const auto b = mine[(seed >> 9) % mine.size()];
                        mine.erase(mine.begin() + (seed >> 9) % mine.size());
                        CHECK(b.first[0] == k + 1 && b.first[b.second - 1] == k + 1);   // nobody else had it
                        groot::dev_free(b.first);
                    }
                }
                for (auto &b : mine) groot::dev_free(b.first);
            });
        for (auto &th : t) th.join();
        groot::dev_free(first);
        CHECK(live_bytes == 0);
        return 0;
    } else {
        return 2;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("pool")
    (d / "hip").mkdir()
    (d / "hip" / "hip_runtime.h").write_text(STAND_IN)
    (d / "driver.cpp").write_text(DRIVER)
    csrc = os.path.join(ROOT, "paper_2511_18297_amd", "csrc")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-I", str(d), "-I", csrc, "-I", os.path.join(ROOT, "include"),
                    str(d / "driver.cpp"), "-o", str(d / "driver")], check=True)
    return str(d / "driver")


@pytest.mark.parametrize("what", ["reuse", "give_back", "bound", "out_of_memory", "wait_fails", "no_lock", "threads"])
def test_pool(driver, what):
    run = subprocess.run([driver, what], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0, run.stdout + run.stderr
