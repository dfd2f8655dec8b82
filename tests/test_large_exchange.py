"""Host checks of the large-grid kernel's exchange (csrc/evolve_big.hip), on its source as
it stands; no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


def source(pattern):
    src = open(os.path.join(ROOT, "paper_1706_07413_amd", "csrc", "evolve_big.hip")).read()
    m = re.search(pattern, src, re.S)
    assert m, pattern
    return m.group(0)


def run(tmp_path, cxx, code):
    c, exe = tmp_path / "check.cpp", tmp_path / "check"
    c.write_text("#include <cstdint>\n#include <cstdio>\n#include <cstring>\n#include <initializer_list>\n#define __device__\n"
                 "#define __forceinline__ inline\ntypedef unsigned long long u64;\n" + code)
    subprocess.run([cxx, "-O2", "-std=c++17", "-o", str(exe), str(c)], check=True)
    return subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split()


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_a_wait_lasts_as_long_whatever_a_poll_takes(tmp_path):
    """Ticks of 10 ns: longer than any launch that may hold the compute units (the library's
    longest take 9 s), and an end in less than half a minute, with polls of 50 ns to 20 us."""
    code = source(r"struct Wait \{.*?\n\};\n") + r"""
int main()
{
    for (u64 poll : {5ull, 30ull, 70ull, 300ull, 2000ull}) {
        u64 now = 123456789;
        const u64 start = now;
        Wait w;
        for (;;) {
            now += poll;
            if (w.look() && w.over(now)) break;
        }
        std::printf("%llu\n", now - start);
    }
    return 0;
}
"""
    for t in run(tmp_path, "g++", code):
        assert 10e8 < int(t) < 30e8, t


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang++")
def test_no_value_is_sent_as_the_empty_word(tmp_path):
    """The pattern of an empty word, as data, goes out as a quiet NaN; every other value as
    it is.  (Through the library such data never reach the exchange: the constraint solve
    after adscl_init marks the instance non-finite, and the kernel skips it.)"""
    code = source(r"constexpr u64 kEmpty = [^\n]*\n") + r"""
static long long __double_as_longlong(double v)
{
    long long b;
    std::memcpy(&b, &v, 8);
    return b;
}
""" + source(r"__device__ __forceinline__ u64 word_of\(double v\) \{[^\n]*\n") + r"""
static double value(u64 b)
{
    double v;
    std::memcpy(&v, &b, 8);
    return v;
}
int main()
{
    std::printf("%llx\n", (u64)(kEmpty ^ word_of(value(kEmpty))));
    // zeros, the smallest and largest numbers, infinities, quiet NaNs
    for (u64 b : {0ull, 1ull << 63, 1ull, (1ull << 63) | 1, 0x000fffffffffffffull, 0x7fefffffffffffffull,
                  0x3ff0000000000001ull, 0x7ff0000000000000ull, 0xfff0000000000000ull, 0x7ff8000000000000ull,
                  0xfff8000000000123ull})
        std::printf("%llx\n", (u64)(b ^ word_of(value(b))));
    return 0;
}
"""
    out = run(tmp_path, CLANG, code)
    assert int(out[0], 16) == 1 << 51  # the quiet bit
    assert set(out[1:]) == {"0"}
