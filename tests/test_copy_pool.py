"""The copies of several threads (csrc/copy_pool.h) on the CPU: sizes around a
part and the smallest shared copy, from several callers at once, under the
thread sanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>
#include "copy_pool.h"
int main() {
    const size_t part = (size_t)128 << 10;
    for (int round = 0; round < 3; ++round) {
        ssj::CopyPool pool;
        std::vector<std::thread> callers;
        for (unsigned c = 0; c < 3; ++c)
            callers.emplace_back([&pool, c, part] {
                for (size_t n : {(size_t)0, (size_t)1, part, 4 * part - 1, 4 * part, 4 * part + 1, 9 * part + 7, 5 * part}) {
                    std::vector<unsigned char> a(n + 16, 7), b(n + 16, 9);
                    for (size_t k = 0; k < n; ++k) a[k] = (unsigned char)(k * 31u + c);
                    pool.copy(b.data() + 3, a.data(), n);
                    for (size_t k = 0; k < b.size(); ++k)
                        if (b[k] != (k < 3 || k >= n + 3 ? 9 : a[k - 3])) { std::printf("byte %zu of %zu\n", k, n); std::exit(1); }
                }
            });
        for (auto& t : callers) t.join();
    }
    return 0;
}
"""


@pytest.mark.parametrize("flags", [["-O2"], ["-O1", "-g", "-fsanitize=thread"]])
def test_copies_of_several_threads(tmp_path, flags):
    src = tmp_path / "pool.cpp"
    src.write_text(MAIN)
    exe = tmp_path / "pool"
    csrc = os.path.join(ROOT, "paper_1812_09141_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", csrc, *flags, str(src), "-o", str(exe)], check=True)
    subprocess.run([str(exe)], check=True, timeout=120)
