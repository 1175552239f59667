"""CPU test: the bounds by which a wave of the kernels tells hidden, partly and wholly visible blocks apart, compiled for the host, against
classify_block() on every block of small calls, and against the mask itself at the ends of the range of positions."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2511_02043_amd", "csrc")

SOURCE = r"""
#include <cstdio>
#include <random>
#include "fl_bwd_bf16.hpp"
using namespace fl;

static const uint32_t kMasks[] = {0, kMaskCausal, kMaskWindow | kMaskCausal, kMaskPrefix};

// rows at the positions [q_lo, q_hi] x keys [k_lo, k_hi]
static bool block(uint32_t mask, int q_lo, int q_hi, int k_lo, int k_hi, int Sk, int window, int prefix) {
  const int cls = classify_block(mask, q_lo, q_hi, k_lo, k_hi, Sk, window, prefix, make_int2(0, 0), make_int2(0, 0));
  const KeyBounds kb = key_bounds(mask, q_lo, q_hi, Sk, window, prefix);
  const RowBounds rb = row_bounds(mask, k_lo, k_hi, Sk, window, prefix);
  int lo, hi;
  query_range(mask, k_lo, k_hi < Sk ? k_hi : Sk - 1, q_hi + 1, window, prefix, lo, hi);
  const bool in_range = q_lo < hi && q_hi >= lo;
  bool ok = kb.whole(k_lo, k_hi) == (cls == kFull) && rb.whole(q_lo, q_hi) == (cls == kFull);
  ok = ok && rb.hidden(q_lo, q_hi) == (cls == kSkip);
  // a block past the last key may count as partly visible: its scores are hidden one by one
  ok = ok && (k_hi < Sk ? kb.hidden(k_lo, k_hi) == (cls == kSkip) : !kb.hidden(k_lo, k_hi) || cls == kSkip);
  ok = ok && (k_lo >= Sk || in_range || cls == kSkip);
  if (!ok)
    std::printf("mask %u rows %d..%d keys %d..%d of %d window %d prefix %d: class %d, by keys %d %d, by rows %d %d, rows in range %d\n", mask, q_lo, q_hi, k_lo,
                k_hi, Sk, window, prefix, cls, kb.hidden(k_lo, k_hi), kb.whole(k_lo, k_hi), rb.hidden(q_lo, q_hi), rb.whole(q_lo, q_hi), in_range);
  return ok;
}

// the tiles of 64 keys that the forward kernel takes as whole, and as visible at all
static bool tiles(uint32_t mask, int q_lo, int q_hi, int Sk, int window, int prefix) {
  int lo, hi, f_lo, f_hi;
  key_range(mask, q_lo, q_hi, Sk, window, prefix, lo, hi);
  full_tile_range(mask, q_lo, q_hi, Sk, window, prefix, 64, f_lo, f_hi);
  for (int t = 0; t <= Sk / 64; ++t) {
    const int cls = classify_block(mask, q_lo, q_hi, t * 64, t * 64 + 63, Sk, window, prefix, make_int2(0, 0), make_int2(0, 0));
    if ((cls == kFull) != (t >= f_lo && t < f_hi) || (cls != kSkip && !(t >= lo / 64 && t < (hi + 63) / 64))) {
      std::printf("mask %u rows %d..%d tile %d of %d keys window %d prefix %d\n", mask, q_lo, q_hi, t, Sk, window, prefix);
      return false;
    }
  }
  return true;
}

int main() {
  for (uint32_t mask : kMasks)
    for (int Sk : {1, 31, 32, 33, 64, 100, 129, 192})
      for (int at : {0, 1, 31, 32, 70, 96})        // window, or prefix
        for (int off : {0, 1, 40, 300})
          for (int q = 0; q < 224; q += 32) {
            for (int k = 0; k < 256; k += 32)
              for (int n : {32, 64})
                if (!block(mask, q + off, q + off + n - 1, k, k + 31, Sk, at, at) || !block(mask, q + off, q + off + 31, k, k + n - 1, Sk, at, at)) return 1;
            if (!tiles(mask, q + off, q + off + 31, Sk, at, at)) return 1;
          }
  // positions, keys and windows up to the largest that a call may have
  std::mt19937_64 rng(1);
  const int top = 0x7fffff00;
  auto any = [&](int n) { return (int)(rng() % ((uint64_t)n / 32)) * 32; };
  for (int i = 0; i < 2000000; ++i) {
    const int Sk = i % 2 ? top : top - (int)(rng() % 64), window = i % 3 ? top - any(1 << 20) : (int)(rng() % (unsigned)top), q = any(top - 64), k = any(top - 64);
    const int near = i % 5 == 0 ? (q > (1 << 20) ? q - any(1 << 20) : q) : k;
    if (!block(kMasks[i % 4], q, q + 31, near, near + 31, Sk, window, window)) return 1;
  }
  return 0;
}
"""


def test_bounds_agree_with_the_classes(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    src = tmp_path / "bounds.hip"
    src.write_text(SOURCE)
    exe = str(tmp_path / "bounds")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", exe], check=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
