"""The bins of token selection (csrc/token_bins.h), on the host: bins are ordered
as their keys are, a key lies in its bin's range and in no other's (up to the
ends 0 and 2^64 - 1, with repeated and neighbouring splitters), and the sampled
tokens do not fall in step with video frames."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_23743_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>
#include "token_bins.h"

using namespace sva;
typedef unsigned long long u64;

int main(int argc, char** argv) {
  if (argc > 1) {                                  // the sampled indices of n tokens
    for (int i = 0; i < kSamples; ++i) std::printf("%d ", sample_index(i, std::atoi(argv[1])));
    return 0;
  }
  std::mt19937_64 rng(1);
  long bad = 0;
  const u64 top = ~0ull, one = 0xBFF0000000000000ull, nan = 0xFFFFE00000000000ull, zero = 0x8000000000000000ull;
  const int share[] = {1, 100, 10000, 50000, 63240, 63239, 33333};
  for (int kind = 0; kind < 9; ++kind)
    for (int rep = 0; rep < 210; ++rep) {
      std::vector<u64> s(kSamples);
      for (auto& x : s) {
        const u64 r = rng();
        switch (kind) {
          case 0: x = r; break;                                  // anywhere
          case 1: x = one + (r >> 12); break;                    // scores within a factor of two
          case 2: x = r % 3 ? one + (r >> 20) : zero; break;     // with zero rows
          case 3: x = r % 2 ? nan : one + (r >> 12); break;      // with wide NaNs
          case 4: x = one + r % 40; break;                       // neighbours
          case 5: x = one; break;                                // one score
          case 6: x = r % 2 ? top - r % 3 : r % 3; break;        // both ends
          case 7: x = top - (r >> 8); break;                     // near 2^64
          default: x = r >> (r % 64); break;
        }
      }
      std::sort(s.begin(), s.end());
      const KeyBins bins = make_bins(s.data(), 63240, share[rep % 7]);
      bad += bins.from < 0 || bins.to > 64 || bins.from > bins.to || bins.per < 60;
      std::vector<u64> keys = {0, 1, 2, zero - 1, zero, zero + 1, nan, top - 1, top};
      for (u64 x : s)
        for (int d = -2; d <= 2; ++d) keys.push_back(x + (u64)(long long)d);
      for (int i = 0; i < 64; ++i) {
        const u64 x = s[rng() % 64], y = s[rng() % 64];
        keys.push_back(rng());
        keys.push_back(std::min(x, y) + rng() % std::max<u64>(1, std::max(x, y) - std::min(x, y)));
      }
      std::sort(keys.begin(), keys.end());
      int before = 0;
      for (u64 key : keys) {
        const int b = key_bin(bins, key);
        bad += b < before || b >= kKeyBins;
        before = b;
        uint64_t lo, hi;
        bin_range(bins, b, lo, hi);
        bad += key < lo || key > hi || key_bin(bins, lo) != b || key_bin(bins, hi) != b;
        bad += lo > 0 && key_bin(bins, lo - 1) >= b;
        bad += hi < top && key_bin(bins, hi + 1) <= b;
      }
      for (u64 x : s) {                            // a splitter has a bin of its own
        uint64_t lo, hi;
        bin_range(bins, key_bin(bins, x), lo, hi);
        bad += lo != x || hi != x;
      }
    }
  for (int n : {1, 2, 63, 64, 65, 1000, 63240, 111600, 2147483647}) {
    int last = -1;
    for (int i = 0; i < kSamples; ++i) {
      const int at = sample_index(i, n);
      bad += at < 0 || at >= n || at < last || at < (long long)i * n / 64;
      last = at;
    }
  }
  std::printf("bad=%ld\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    d = tmp_path_factory.mktemp("bins")
    (d / "bins.hip").write_text(PROGRAM)
    subprocess.run([hipcc, "-O2", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-w", "-I", CSRC, str(d / "bins.hip"), "-o", str(d / "bins")],
                   check=True, capture_output=True)
    return str(d / "bins")


def test_bins_follow_the_keys(exe):
    res = subprocess.run([exe], capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.strip() == "bad=0", res.stdout + res.stderr


@pytest.mark.parametrize("frames", [8, 16, 21, 31, 32, 64])
@pytest.mark.parametrize("frame", [30 * 52, 34 * 60, 45 * 80])
def test_samples_spread_over_the_frame(exe, frames, frame):
    """64 random places of a frame leave gaps of up to about ln(64) / 64 of it; the
    first token of every 64th of 32 frames is at one of two places."""
    res = subprocess.run([exe, str(frames * frame)], capture_output=True, text=True, check=True)
    at = np.sort(np.array([int(x) for x in res.stdout.split()]) % frame)
    gaps = np.diff(np.concatenate([at, at[:1] + frame]))
    assert len(at) == 64 and len(np.unique(at)) >= 48
    assert gaps.max() <= 0.15 * frame, gaps.max() / frame
