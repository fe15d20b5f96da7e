"""What the library's host side remembers between calls, where it could be remembered wrongly: small programs around its host
headers, built with the host compiler."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_06786_amd", "csrc")


def run_program(tmp_path, text):
    src, exe = tmp_path / "program.cpp", tmp_path / "program"
    src.write_text(text)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr


def test_two_threads_ask_for_two_lds_sizes(tmp_path):
    """A thread that asks for less, while the runtime is granting more to another one, must not leave the smaller size in
    force: what was recorded as allowed has to be allowed."""
    run_program(tmp_path, r'''
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <thread>
#include "mq_lds.h"

int main() {
    mq::LdsGrants grants;
    std::mutex m;
    std::condition_variable cv;
    int in_force = 0, calls = 0;
    // the runtime: the last size set is in force; the first caller is held until a second one has come, or half a second
    auto set = [&](int bytes) {
        std::unique_lock<std::mutex> lock(m);
        in_force = bytes;
        ++calls;
        cv.notify_all();
        if (calls == 1) cv.wait_for(lock, std::chrono::milliseconds(500), [&] { return calls > 1; });
        return true;
    };
    std::thread large([&] { grants.ensure(0, 100000, set); });
    {
        std::unique_lock<std::mutex> lock(m);
        cv.wait(lock, [&] { return calls == 1; });
    }
    std::thread small([&] { grants.ensure(0, 80000, set); });
    large.join();
    small.join();
    if (!grants.ensure(0, 100000, set) || in_force < 100000) return std::printf("100000 recorded, %d in force\n", in_force), 1;
    // a refusal is not recorded, another device has its own size
    if (grants.ensure(0, 150000, [](int) { return false; })) return std::printf("a refusal was taken for a grant\n"), 1;
    if (!grants.ensure(0, 150000, set) || in_force != 150000) return std::printf("not asked again after a refusal\n"), 1;
    calls = 1;
    if (!grants.ensure(1, 90000, set) || in_force != 90000) return std::printf("device 1 was not asked\n"), 1;
    if (grants.ensure(-1, 1, set)) return std::printf("no device\n"), 1;
    return 0;
}
''')


def test_remembered_workspace_sizes_refuse_what_the_call_refuses():
    """16.0 equals 16 and hashes alike, but it is no size."""
    from paper_2502_06786_amd import binding
    assert binding.mq_workspace_bytes(0, 16, 256, 256, 3) > 0
    with pytest.raises(ctypes.ArgumentError):
        binding.mq_workspace_bytes(0, 16.0, 256, 256, 3)
