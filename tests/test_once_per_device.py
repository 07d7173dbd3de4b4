"""A kernel's LDS beyond 64 KB is asked for once on every device of the process
(two contexts on two devices share the kernels), and again where asking failed.
The counting is host code, run here with asks that only count."""
import os
import re
import subprocess

CODE = r"""
#include "once_per_device.h"
#include <cstdio>
#include <stdexcept>
int main() {
    morap::OncePerDevice once, other;
    int asked[100] = {0}, failed = 0;
    auto ask = [&](int d) { once(d, [&] { ++asked[d]; }); };
    for (int d : {0, 1, 0, 1, 63, 63, 0, 64, 64}) ask(d);
    for (int i = 0; i < 2; ++i)
        try {
            once(5, [&] { ++asked[5]; if (i == 0) throw std::runtime_error("no"); });
        } catch (const std::exception&) { ++failed; }
    ask(5);
    int second = 0;
    other(0, [&] { ++second; });   // another kernel
    std::printf("%d %d %d %d %d %d %d\n", asked[0], asked[1], asked[63], asked[64], asked[5], failed, second);
}
"""


def test_asked_once_on_every_device(root, tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text(CODE)
    exe = tmp_path / "t"
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(root, "paper_2305_04397_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    assert out.split() == ["1", "1", "1", "2", "2", "1", "1"]


def test_no_kernel_keeps_one_answer_for_all_devices(root):
    csrc = os.path.join(root, "paper_2305_04397_amd", "csrc")
    for f in os.listdir(csrc):
        with open(os.path.join(csrc, f)) as h:
            assert not re.search(r"static[^;{}]*=\s*hipFuncSetAttribute", h.read()), f
