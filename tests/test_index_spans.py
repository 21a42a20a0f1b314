"""Index arithmetic of the set-up and row kernels (csrc/span.h) at the top of the
accepted sizes, on the CPU: the header is compiled for the host and every walk is
compared with one in 64 bits.  A walk in plain int steps from an end near 2^31 - 1
to a negative index that passes the end test again."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "span.h"
typedef long long i64;
const i64 TOP = 2147483647;

static int entries(i64 e0, i64 e1) {
  for (int lane = 0; lane < 64; ++lane) {
    rpk::LaneEntries it((int)e0, (int)e1, lane);
    for (i64 e = e0 + lane; e < e1; e += 64, it.next())
      if (!it.more() || it.at() != e) return std::printf("entries %lld %lld lane %d: not at %lld\n", e0, e1, lane, e);
    if (it.more()) return std::printf("entries %lld %lld lane %d: goes on at %d\n", e0, e1, lane, it.at());
  }
  return 0;
}

static int rows(i64 lo, i64 hi, int block) {
  for (int w = 0; w < block; w += 64) {
    unsigned at = (unsigned)(lo + w);
    for (i64 r = lo + w; r < hi; r += block, at += (unsigned)block)
      if (!rpk::row_below(at, (int)hi) || (i64)at != r) return std::printf("rows %lld %lld: not at %lld\n", lo, hi, r);
    if (rpk::row_below(at, (int)hi)) return std::printf("rows %lld %lld block %d: goes on at %u\n", lo, hi, block, at);
  }
  return 0;
}

int main() {
  int bad = 0;
  for (i64 end : {(i64)0, (i64)1, (i64)63, (i64)64, (i64)65, (i64)1000, TOP - 200, TOP - 64, TOP - 63, TOP - 62, TOP - 1, TOP})
    for (i64 cnt : {(i64)0, (i64)1, (i64)62, (i64)63, (i64)64, (i64)65, (i64)127, (i64)128, (i64)700})
      if (cnt <= end) bad += entries(end - cnt, end) != 0;
  // one slice that holds every entry: the walk's last steps
  for (i64 cnt : {TOP, TOP - 1, TOP - 62, TOP - 63, TOP - 64})
    for (int lane = 0; lane < 64; ++lane) {
      rpk::LaneEntries it(0, (int)cnt, lane);
      it.k += (unsigned)((cnt - 1 - lane) / 64 * 64);
      bad += !it.more() || it.at() >= cnt;
      it.next();
      bad += it.more();
    }
  for (i64 n : {(i64)1, (i64)63, (i64)64, (i64)65, (i64)128, (i64)1000, TOP - 200, TOP - 64, TOP - 63, TOP - 1, TOP})
    for (i64 s = (n - 1) / 64; s >= 0 && s > (n - 1) / 64 - 3; --s) {
      const i64 want = 64 * s + 64 < n ? 64 * s + 64 : n;
      if (rpk::slice_end((int)n, (int)s) != want) bad += std::printf("slice %lld of %lld rows\n", s, n) > 0;
    }
  for (i64 hi : {(i64)1, (i64)64, (i64)4097, TOP - 2000, TOP - 1023, TOP - 64, TOP - 1, TOP})
    for (int block : {64, 256, 1024}) bad += rows((hi > 4000 ? hi - 4000 : 0) & ~63ll, hi, block) != 0;
  std::printf("bad %d\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("span")
    src, exe = d / "span.cpp", d / "span"
    src.write_text(PROGRAM)
    subprocess.check_call(["hipcc", "-x", "hip", "--offload-host-only", "-std=c++17", "-O1",
                           "-I" + os.path.join(ROOT, "paper_2302_04180_amd", "csrc"), str(src), "-o", str(exe)])
    return exe


def test_walks_end_where_64_bit_ones_do(program):
    out = subprocess.run([str(program)], stdout=subprocess.PIPE, timeout=60)
    assert out.returncode == 0 and b"bad 0" in out.stdout, out.stdout.decode()
