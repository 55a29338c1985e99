"""The selections' key arithmetic (csrc/order_keys.h), compiled for the host: where a threshold key with
its low 16 bits cleared may stand in for scores as a float, and that a threshold taken as the wave
selection takes it never loses the top-k, whatever share of the scores is -inf."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_12364_amd", "csrc")

SOURCE = r"""
#include <math.h>
#include <stdio.h>
#include <float.h>
#include <initializer_list>
#include <vector>
#include "order_keys.h"
using namespace umem;

static int bad(const char* what, uint32_t a, uint32_t b) {
  printf("%s: %08x %08x\n", what, a, b);
  return 1;
}

// The largest prefix of 16 bits that at least k of the maxima reach, ending early at exactly k.
static uint32_t kth16(const std::vector<uint32_t>& v, int k) {
  uint32_t p = 0;
  for (int b = 31; b >= 16; --b) {
    const uint32_t c = p | (1u << b);
    int n = 0;
    for (uint32_t x : v) n += x >= c;
    if (n >= k) p = c;
    if (n == k) break;
  }
  return p;
}

int main() {
  // every limit: the float compare says what the keys' compare says, at each float next to a prefix
  for (uint32_t hi = 0; hi < 65536; ++hi) {
    const uint32_t L = hi << 16;
    if (!key32_is_limit(L) || L > order_key(INFINITY)) continue;
    const float lim = key32_value(L);
    if (lim != lim) return bad("a limit without a value", L, 0);
    const uint32_t own = __builtin_bit_cast(uint32_t, lim) >> 16;
    for (uint32_t i = 0; i < 263; ++i) {                  // the float's neighbours, and floats all over
      const uint32_t h2 = i < 7 ? (own + i - 3) & 0xFFFFu : (i - 7) * 257;
      for (uint32_t lo : {0x0000u, 0x0001u, 0xFFFFu}) {
        const float x = __builtin_bit_cast(float, (h2 << 16) | lo);
        if ((x >= lim) != (order_key(x) >= L)) return bad("compare", L, (h2 << 16) | lo);
      }
    }
  }
  if (!key32_is_limit(order_key(-FLT_MAX))) return bad("the lowest number is a limit", 0, 0);
  if (key32_is_limit(order_key(-INFINITY)) || key32_is_limit(0)) return bad("-inf is none", 0, 0);
  // scores dealt to groups as to a wave's lanes: a piece of four to a lane, `groups` maxima
  const float fill[] = {-INFINITY, -FLT_MAX, NAN};
  for (int n : {256, 512, 1024, 1792, 2048})
    for (int k : {1, 7, 32, 33, 42, 64})
      for (float rest : fill)
        for (int live : {0, 1, k / 2, k - 1, k, 64, 100, 4 * k, n}) {
          if (8 * k > n || live > n) continue;
          std::vector<float> x(n, rest);
          for (int i = 0; i < live; ++i) x[i] = sinf(static_cast<float>(i));
          const int groups = k <= 32 || n <= 768 ? 2 : 4;
          std::vector<uint32_t> mx(64 * groups, 0u);
          int numbers = 0;
          for (int i = 0; i < n; ++i) {
            uint32_t& m = mx[i / 4 % 64 + 64 * (i / 256 % groups)];
            const uint32_t key = order_key(x[i]);
            m = key > m ? key : m;
            numbers += key != 0;
          }
          const uint32_t L = kth16(mx, k);
          if (!key32_is_limit(L)) continue;                // the exact search over all scores
          int survivors = 0;
          for (float v : x) survivors += v >= key32_value(L);
          if (survivors < k) return bad("survivors", L, survivors);
        }
  // a Tucker grid of 64 x 64 fp64 scores, 512 maxima over eight rows of a column, rounded to fp32
  for (double rest : {-1e300, -1e39, -static_cast<double>(INFINITY), static_cast<double>(NAN)})
    for (double best : {1e300, 1.0, -1e38, -1e300})
      for (int cols : {0, 1, 7, 8, 9, 64})
        for (int m : {1, 8, 64}) {
          std::vector<uint32_t> mx(512);
          for (int i = 0; i < 512; ++i) mx[i] = order_key(static_cast<float>(i % 64 < cols ? best : rest));
          const uint32_t L = kth16(mx, m);
          if (!key32_is_limit(L)) continue;
          int survivors = 0;
          for (int i = 0; i < 4096; ++i)
            survivors += static_cast<float>(i % 64 < cols ? best : rest) >= key32_value(L);
          if (survivors < m) return bad("grid survivors", L, survivors);
        }
  puts("ok");
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("order_keys")
    (d / "t.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", f"-I{CSRC}", str(d / "t.cpp"), "-o", str(d / "t")], check=True)
    return str(d / "t")


def test_threshold_keys(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
