"""The leave for large dynamic LDS (gd_grant.h) against a stand-in for the HIP calls: every GPU
of a process gets it for each kernel, once, also where several threads come at the same time;
a refusal is passed on and not remembered as a success."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2605_17879_amd", "csrc")

HIP = r"""
#include <atomic>
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize = 8 };
extern thread_local int current_device;
extern std::atomic<int> asked[128];
extern std::atomic<bool> refuse;
inline hipError_t hipGetDevice(int* d) { *d = current_device; return hipSuccess; }
inline hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) {
    asked[current_device]++;
    return refuse ? hipErrorInvalidValue : hipSuccess;
}
"""

MAIN = r"""
#include "gd_grant.h"
#include <stdio.h>
#include <thread>
#include <vector>
thread_local int current_device = 0;
std::atomic<int> asked[128];
std::atomic<bool> refuse{false};
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    std::atomic<uint64_t> one{0}, other{0};
    refuse = true;
    CHECK(gd_grant_lds(one, nullptr, 100000) == hipErrorInvalidValue);
    refuse = false;
    CHECK(gd_grant_lds(one, nullptr, 100000) == hipSuccess && asked[0] == 2);
    CHECK(gd_grant_lds(one, nullptr, 100000) == hipSuccess && asked[0] == 2);
    CHECK(gd_grant_lds(other, nullptr, 100000) == hipSuccess && asked[0] == 3);
    current_device = 1;                                  // the process's second GPU
    CHECK(gd_grant_lds(one, nullptr, 100000) == hipSuccess && asked[1] == 1);
    CHECK(gd_grant_lds(one, nullptr, 100000) == hipSuccess && asked[1] == 1);
    current_device = 100;                                // beyond what is remembered: asked every time
    CHECK(gd_grant_lds(one, nullptr, 1) == hipSuccess && gd_grant_lds(one, nullptr, 1) == hipSuccess && asked[100] == 2);
    std::atomic<uint64_t> shared{0};
    std::atomic<int> bad{0};
    std::vector<std::thread> threads;
    for (int i = 0; i < 8; ++i)
        threads.emplace_back([&, i] {
            current_device = 2 + i % 4;
            for (int k = 0; k < 1000; ++k)
                if (gd_grant_lds(shared, nullptr, 100000) != hipSuccess || !(shared.load() >> current_device & 1)) ++bad;
        });
    for (auto& t : threads) t.join();
    CHECK(bad == 0 && shared.load() == 0x3Cull);
    for (int d = 2; d < 6; ++d) CHECK(asked[d] >= 1 && asked[d] <= 2);
    printf("ok\n");
    return 0;
}
"""


def test_every_gpu_is_granted_once(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(HIP)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = tmp_path / "grant"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-Wall", "-Werror", f"-I{tmp_path}",
                    f"-I{CSRC}", str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0 and out.stdout.strip() == "ok", out.stdout + out.stderr


def test_kernels_with_large_lds_ask_for_it():
    """Every launch that asks for leave does so through it: no flag of its own that is one for
    the whole process."""
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        if name != "gd_grant.h":
            assert "hipFuncSetAttribute" not in text, name
        assert "static bool" not in text, name
