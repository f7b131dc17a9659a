"""The divisions of the kernels' index arithmetic (div_by() of csrc/kvcomm_device.h), on the CPU: every quotient of 31-bit numbers,
at the multiples of the divisor and next to them, where a multiplication in place of a division goes wrong first."""
import subprocess

from paper_2510_12872_amd import build

MAIN = r"""
#include <cstdio>
#include <vector>
#include "attn_common.h"
int main()
{
    const int64_t top = 2147483647;
    std::vector<int64_t> ds, ns = {0, 1, 2, top - 1, top};
    for (int64_t d = 1; d <= 1100; ++d) ds.push_back(d);
    for (int b = 11; b < 31; ++b)
        for (int64_t d = ((int64_t)1 << b) - 1; d <= ((int64_t)1 << b) + 1; ++d) ds.push_back(d);
    ds.push_back(top);
    for (int64_t d : ds) {
        const kvc::divisor_t m = kvc::make_divisor((uint32_t)d);
        std::vector<int64_t> at = ns;
        for (int64_t q : {(int64_t)1, (int64_t)2, (int64_t)3, (int64_t)1000, top / d / 2, top / d - 1, top / d})
            for (int64_t n = q * d - 1; n <= q * d + 1; ++n)
                if (n >= 0 && n <= top) at.push_back(n);
        for (int64_t n : at)
            if (kvc::div_by((int)n, m) != n / d) return printf("%ld / %ld gave %d\n", (long)n, (long)d, kvc::div_by((int)n, m)), 1;
    }
    puts("ok");
}
"""


def test_quotients(tmp_path):
    src, exe = tmp_path / "div.hip", tmp_path / "div"
    src.write_text(MAIN)
    subprocess.run([build.hipcc_path(), "--offload-arch=gfx950", "--offload-host-only", "-O1", "-std=c++17", "-I", build.CSRC, "-I",
                    build.ROOT + "/include", "-o", str(exe), str(src)], check=True, capture_output=True, timeout=120)
    ran = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert ran.returncode == 0 and ran.stdout == "ok\n", ran.stdout
