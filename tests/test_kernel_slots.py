"""The kept occupancies (csrc/kernel_slots.h), in a host program with made-up kernels of one signature."""
import os
import subprocess

from paper_2609_26300_amd import build as lib_build

PROGRAM = r"""
#include "kernel_slots.h"
#include <cstdio>
#include <thread>
#include <utility>
#include <vector>

template <int I> void kernel(float*) {}
static std::atomic<int> queries{0}, wrong{0}, go{0};
constexpr int kKernels = 150;  // more than a small table would hold

template <int I> int slots(int dev, bool answers = true) {
    const compkv::Occupancy o = compkv::kernel_occupancy<kernel<I>>(dev, [&](compkv::Occupancy& q) {
        ++queries;
        std::this_thread::yield();
        q = {I + 1, 256 + dev};
        return answers;
    });
    return answers && (o.per_cu != I + 1 || o.cus != 256 + dev) ? -1 : o.per_cu * o.cus;
}

template <int... I> void all(int first, int dev, std::integer_sequence<int, I...>) {
    int (*const f[])(int, bool) = {slots<I>...};
    for (int k = 0; k < kKernels; ++k)
        if (f[(first + k) % kKernels](dev, true) < 0) ++wrong;
}

int main() {
    const auto kernels = std::make_integer_sequence<int, kKernels>();
    if (slots<0>(3, false) != 1 || slots<0>(3, false) != 1 || queries != 2) return 1;  // a failed query is not kept
    std::vector<std::thread> t;
    for (int i = 0; i < 8; ++i)
        t.emplace_back([=] {
            ++go;
            while (go < 8) {}
            all(i % 2, 0, kernels);  // threads meet at the same kernels for the first time
            all(i * 11, 1, kernels);
        });
    for (auto& x : t) x.join();
    const int first = queries;
    all(0, 0, kernels);
    all(0, 1, kernels);
    if (queries != first) return 2;  // every kernel's answer is kept
    slots<5>(99);
    slots<5>(99);
    if (queries != first + 2) return 3;
    return wrong == 0 ? 0 : 4;
}
"""


def test_each_kernel_keeps_its_own_occupancy(tmp_path):
    """Eight threads that ask for 150 kernels of one signature at once: each gets every kernel's own answer,
    later calls ask for none again, and a failed query is not kept."""
    (tmp_path / "slots.cpp").write_text(PROGRAM)
    exe = os.path.join(tmp_path, "slots")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", lib_build.CSRC, str(tmp_path / "slots.cpp"), "-o", exe],
                   check=True)
    for _ in range(5):
        assert subprocess.run([exe], timeout=60).returncode == 0
