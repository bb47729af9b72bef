"""The gate of the resident launches (csrc/resgate.h) on the CPU: devices do
not wait for each other, calls that fit one device hold it together, the others
come in in the order of their calls."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>
#include "resgate.h"
using namespace lsrtm;

static void pause() { std::this_thread::sleep_for(std::chrono::milliseconds(100)); }
#define CHECK(x) do { if (!(x)) { printf("failed: %s (line %d)\n", #x, __LINE__); return 1; } } while (0)

int main() {
    std::atomic<int> in{0};
    {   // another device, and what fits beside, do not wait
        ResRoom a(0, 240, 256);
        std::thread other([&] { ResRoom b(1, 240, 256); in += 1; });
        other.join();
        CHECK(in == 1);
        std::thread beside([&] { ResRoom b(0, 16, 256); in += 1; });
        beside.join();
        CHECK(in == 2);
    }
    {   // every XCD takes an eighth, rounded up: 30 and 226 are 33 on the first ones
        in = 0;
        ResGate& g = res_gate(2);
        g.acquire(30, 256);
        std::thread t([&] { ResRoom b(2, 226, 256); in += 1; });
        pause();
        CHECK(in == 0);
        g.release(30);
        t.join();
        CHECK(in == 1);
    }
    {   // in the order of the calls: the small one does not overtake the large one
        in = 0;
        std::atomic<int> order{0}, large{0}, small{0};
        ResGate& g = res_gate(3);
        g.acquire(128, 256);
        std::thread t1([&] { ResRoom b(3, 200, 256); large = ++order; pause(); });
        pause();
        std::thread t2([&] { ResRoom b(3, 64, 256); small = ++order; });
        pause();
        CHECK(order == 0);
        g.release(128);
        t1.join();
        t2.join();
        CHECK(large == 1 && small == 2);
    }
    {   // never more than there is room, everyone gets in
        std::atomic<int> now{0}, most{0}, done{0};
        std::vector<std::thread> ts;
        for (int i = 0; i < 16; ++i)
            ts.emplace_back([&, i] {
                for (int k = 0; k < 50; ++k) {
                    const int n = 8 * (1 + (i * 7 + k) % 32);
                    ResRoom b(4, n, 256);
                    const int v = now += n;
                    int m = most;
                    while (v > m && !most.compare_exchange_weak(m, v)) {}
                    std::this_thread::yield();
                    now -= n;
                    done += 1;
                }
            });
        for (auto& t : ts) t.join();
        CHECK(done == 800 && most <= 256);
    }
    printf("ok\n");
    return 0;
}
'''


def test_gate(tmp_path):
    if not shutil.which("g++"):
        pytest.fail("the native toolchain is missing")
    src = tmp_path / "gate.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "gate"
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", os.path.join(ROOT, "paper_2508_10405_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
