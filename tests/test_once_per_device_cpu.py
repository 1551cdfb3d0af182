"""The one-time preparation of a launch runs once on every device, also when threads launch together: compiled here."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2505_07203_amd", "csrc")

PROGRAM = r"""
#include "once_per_device.h"
#include <cstdio>
#include <thread>
#include <vector>
int main() {
    static po::OncePerDevice once;
    int runs[8] = {};
    for (int pass = 0; pass < 3; ++pass)
        for (int device = 0; device < 8; ++device) once.run(device, [&] { ++runs[device]; });
    for (int device = 0; device < 8; ++device)
        if (runs[device] != 1) return std::printf("device %d: %d runs\n", device, runs[device]), 1;
    static po::OncePerDevice shared;
    std::atomic<int> prepared[8] = {};
    std::atomic<int> early{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < 8; ++t)
        threads.emplace_back([&, t] {
            for (int i = 0; i < 64; ++i) {
                const int device = (t + i) % 8;
                shared.run(device, [&] { prepared[device].fetch_add(1); });
                if (prepared[device].load() == 0) early.fetch_add(1);      // came past before anybody had prepared it
            }
        });
    for (auto& t : threads) t.join();
    return early.load();
}
"""


def test_every_device_is_prepared_before_a_launch_goes_past(tmp_path):
    src, exe = tmp_path / "once.cpp", tmp_path / "once"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
