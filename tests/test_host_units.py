"""CPU: host-side units of the library, compiled with g++ into small programs."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1302_5010_amd", "csrc")


def _run(tmp_path, source, *flags):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "unit.cpp", tmp_path / "unit"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", *flags, "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr


def test_arena_list_updates_do_not_depend_on_the_host_list(tmp_path):
    """Chunks reach the device through the stream, after kernels that the host has enqueued already, while the host
    goes on and adds the next one.  A stream of deferred operations stands for the device: between any two of them its
    list holds whole entries only, those of the chunks taken over so far."""
    _run(tmp_path, r"""
#include <cstdio>
#include <functional>
#include <vector>
#include "arena_list.h"
using namespace bmpl;
int main()
{
    Arena host{}, dev{};
    std::vector<std::function<void()>> stream;
    static double mem[ARENA_CHUNKS];
    for (int k = 0; k < ARENA_CHUNKS; ++k) {
        const ArenaChunk c = arena_next(host, mem + k, 100 + k);
        arena_put(host, c);
        stream.push_back([c, &dev] { arena_put(dev, c); });
    }
    unsigned long long at = 0;
    for (int k = 0; k < ARENA_CHUNKS; ++k) {
        if (dev.nchunks != k || dev.base[k] != nullptr) { std::printf("chunk %d came early\n", k); return 1; }
        stream[k]();
        if (dev.nchunks != k + 1 || dev.base[k] != mem + k || dev.start[k] != at || dev.size[k] != 100ull + k) {
            std::printf("chunk %d is not whole\n", k);
            return 1;
        }
        at += dev.size[k];
    }
    return 0;
}
""")
