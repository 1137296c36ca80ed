"""What the library does when the host has no memory left, against a runtime that only counts (no GPU): the error comes back as a
status, nothing is thrown through the C entries, and nothing is left allocated on the device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include <new>
#include "srft_kv.h"

// the runtime the library sees
static int on_device = 0, launches = 0;
extern "C" {
int hipMalloc(void** p, size_t n) { ++on_device; *p = std::aligned_alloc(256, (n + 255) / 256 * 256); return 0; }
int hipFree(void* p) { --on_device; std::free(p); return 0; }
int hipMemcpy(void*, const void*, size_t, int) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }
struct three { unsigned x, y, z; };
int hipLaunchKernel(const void*, three, three, void**, size_t, void*) { ++launches; return 0; }
int hipGetLastError(void) { return 0; }
}

// the allocation that fails: number `left` from now on (0: none)
static long left = 0;
void* operator new(size_t n) {
    if (left > 0 && --left == 0) throw std::bad_alloc();
    void* p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

// call(), with every one of its allocations failing in turn; cleanup() after the one that succeeds
template <class F, class G>
static int every(const char* what, F call, G undo) {
    for (int k = 1;; ++k) {
        left = k;
        const int rc = call();
        const bool all = left > 0;                           // the one that fails was never reached
        left = 0;
        if (all) {
            CHECK(rc == SRFT_OK);
            std::printf("%s %d\n", what, k - 1);
            undo();
            return 0;
        }
        CHECK(rc == SRFT_ERR_HIP);
    }
}

int main() {
    srft_plan_t* p = nullptr;
    for (int d : {64, 128, 256})
        for (int transform : {0, 1}) {
            const int bad = every("plan", [&] {
                const int rc = srft_plan_create_ex(&p, d, 32, 4, transform, 7, nullptr);
                return rc == SRFT_OK ? rc : p || on_device ? 99 : rc;
            }, [&] { srft_plan_destroy(p); });
            if (bad) return bad;
            CHECK(on_device == 0);
        }
    // beside a plan that stays: its place is not touched
    srft_plan_t* keep = nullptr;
    CHECK(srft_plan_create(&keep, 128, 32, 1, nullptr) == SRFT_OK);
    const int held = on_device;
    if (every("second plan", [&] {
            const int rc = srft_plan_create(&p, 128, 32, 2, nullptr);
            return rc == SRFT_OK ? rc : p || on_device != held ? 99 : rc;
        }, [&] { srft_plan_destroy(p); }))
        return 1;
    CHECK(on_device == held);
    alignas(16) static unsigned char codes[64 * 64], view[64 * 256], fresh[64 * 256];
    alignas(16) static float scales[64 * 4];
    const srft_plan_t* plans[] = {keep};
    uint8_t* c[] = {codes};
    float* s[] = {scales};
    void* v[] = {view};
    const void* x[] = {fresh};
    srft_cache_t* cache = nullptr;
    if (every("cache", [&] {
            const int rc = srft_cache_create(&cache, plans, 1, 1, 64, 16, c, s, v);
            return rc == SRFT_OK || !cache ? rc : 99;
        }, [] {}))
        return 1;
    srft_cache_destroy(cache);
    for (int k = 1; k < 20; ++k) {                           // an append that fills a window, on a cache of its own
        CHECK(srft_cache_create(&cache, plans, 1, 1, 64, 16, c, s, v) == SRFT_OK);
        left = k;
        const int rc = srft_cache_append(cache, x, 16, nullptr);
        const bool all = left > 0;
        left = 0;
        CHECK(rc == (all ? SRFT_OK : SRFT_ERR_HIP));
        CHECK(srft_cache_quantized_tokens(cache) == (all ? 16 : 0));
        if (all) {
            left = 1;
            CHECK(srft_cache_rebuild_view(cache, nullptr) == SRFT_ERR_HIP);
            left = 0;
            CHECK(srft_cache_rebuild_view(cache, nullptr) == SRFT_OK);
        }
        srft_cache_destroy(cache);
        if (all) break;
    }
    srft_plan_destroy(keep);
    CHECK(on_device == 0 && launches > 0);
    std::printf("done\n");
    return 0;
}
"""


def test_no_host_memory_is_a_status(tmp_path):
    from paper_2605_05699_amd import binding, build
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    if not os.path.exists(binding.LIB_PATH):
        build.build()
    src, exe = tmp_path / "memory.cpp", tmp_path / "memory"
    src.write_text(SOURCE)
    lib = os.path.dirname(binding.LIB_PATH)
    subprocess.run([gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), str(src), binding.LIB_PATH, f"-Wl,-rpath,{lib}",
                    "-Wl,--allow-shlib-undefined", "-rdynamic", "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert out.returncode == 0 and out.stdout.endswith("done\n"), out.stdout + out.stderr
