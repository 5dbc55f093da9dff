"""The device exponential (zeus_device.h) compiled for the host: over its range,
infinities and NaN, under the compiler's check of conversions to integers,
against the C library's."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# the HIP names that the header uses, for a host compiler
STUB = """#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#define __device__
#define __host__
#define __forceinline__ inline
static inline uint64_t __umul64hi(uint64_t a, uint64_t b) { return (uint64_t)(((unsigned __int128)a * b) >> 64); }
#define __sincosf(a, s, c) (*(s) = sinf(a), *(c) = cosf(a))
#define __expf(a) expf(a)
"""

PROG = """#include "zeus_device.h"
#include <stdio.h>
int main() {
  const double inf = __builtin_huge_val(), nan = __builtin_nan("");
  // argument, value
  const double edge[][2] = {{nan, nan}, {-nan, nan}, {inf, inf}, {-inf, 0.0}, {1e300, inf}, {-1e300, 0.0},
                            {1e19, inf}, {-1e19, 0.0}, {710.5, inf}, {-746.5, 0.0}, {0.0, 1.0},
                            {-0.0, 1.0}, {5e-324, 1.0}};
  int bad = 0;
  for (auto &p : edge) {
    volatile double x = p[0];  // not a constant to the compiler
    const double e = zeus::zm::exp(x);
    if (!(e == p[1] || (e != e && p[1] != p[1]))) { printf("exp(%g) = %g\\n", p[0], e); bad = 1; }
  }
  for (int i = -7000; i <= 7000; ++i) {
    const double x = i * 0.1, e = zeus::zm::exp(x), r = ::exp(x);
    if (!(e / r - 1.0 < 4e-16 && 1.0 - e / r < 4e-16)) { printf("exp(%g)\\n", x); bad = 1; }
  }
  return bad;
}
"""


def test_exp_is_defined_for_every_argument(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(PROG)
    exe = tmp_path / "main"
    csrc = os.path.join(ROOT, "paper_2603_28770_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-fsanitize=float-cast-overflow",
                    "-fno-sanitize-recover=all", "-I", str(tmp_path), "-I", csrc,
                    str(tmp_path / "main.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
