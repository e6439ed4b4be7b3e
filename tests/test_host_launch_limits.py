"""KernelLimits (launch.h) settles a kernel's limits once on each device, whichever comes first and from whichever thread, and not at
all where that fails; the device runtime is played by the program."""
import subprocess

PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "launch.h"
using namespace d2ft;
thread_local int current = 0;
std::atomic<int> allowed[64], asked[64];
int refuse = -1;
extern "C" {
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
    if (current == refuse) return hipErrorInvalidValue;
    if (bytes == 163840) ++allowed[current];
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int d) { ++asked[d]; *v = 256 - d; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = current == 3 ? 0 : 2; return hipSuccess; }
}
int main() {
    KernelLimits limits;
    auto get = [&](int dev, int want) {
        current = dev;
        int n = -1;
        return limits.get(nullptr, 256, 163840, &n) == hipSuccess && n == want;
    };
    bool ok = true;
    for (int round = 0; round < 2; ++round) ok = ok && get(0, 512) && get(1, 510) && get(3, 253) && get(40, 432);
    refuse = 2;
    current = 2;
    int n = 0;
    ok = ok && limits.get(nullptr, 256, 163840, &n) != hipSuccess;
    refuse = -1;
    ok = ok && get(2, 508);
    for (int d : {0, 1, 2, 3}) ok = ok && allowed[d] == 1 && asked[d] == 1;
    ok = ok && allowed[40] == 2;   // more devices than are remembered
    std::vector<std::thread> threads;
    std::atomic<int> bad{0};
    for (int t = 0; t < 16; ++t) threads.emplace_back([&, t] { for (int k = 0; k < 1000; ++k) if (!get(4 + (t + k) % 4, 2 * (252 - (t + k) % 4))) ++bad; });
    for (auto& t : threads) t.join();
    for (int d = 4; d < 8; ++d) ok = ok && allowed[d] >= 1;
    ok = ok && in_eights(512) == 512 && in_eights(253) == 248 && in_eights(3) == 8;
    return ok && bad == 0 ? 0 : 1;
}
"""


def test_limits_per_device_and_thread(tmp_path):
    from paper_2504_12471_amd import build
    src, exe = tmp_path / "limits.hip", tmp_path / "limits"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-host-only", "-std=c++17", "-O1", "-w", "-pthread",
                    "-I", build.CSRC, str(src), "-o", str(exe)], check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
