"""The block order of the causal kernels is a bijection: every (block, head, row) is taken once, whatever the grid,
also where the products in it need 64 bits.  The function is cut out of the header and compiled for the host."""
import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2301_08984_amd", "csrc", "mfma_common.h")

DRIVER = r"""
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <vector>
using std::min;
struct Dim { int x, y, z; };
static Dim gridDim, blockIdx;
struct BlockId { int x, y, z; };
#define __device__
%s
static bool bijection(int gx, int gy, int gz, bool pairs) {
  gridDim = {gx, gy, gz};
  std::vector<char> seen((size_t)gx * gy * gz, 0);
  for (blockIdx.z = 0; blockIdx.z < gz; ++blockIdx.z)
    for (blockIdx.y = 0; blockIdx.y < gy; ++blockIdx.y)
      for (blockIdx.x = 0; blockIdx.x < gx; ++blockIdx.x) {
        const BlockId b = causal_block_id(pairs);
        if (b.x < 0 || b.x >= gx || b.y < 0 || b.y >= gy || b.z < 0 || b.z >= gz) return false;
        char& s = seen[b.x + (size_t)gx * (b.y + (size_t)gy * b.z)];
        if (s) return false;
        s = 1;
      }
  return true;
}
int main() {
  int bad = 0;
  for (int pairs = 0; pairs < 2; ++pairs) {
    for (int gx = 1; gx <= 70; ++gx)
      for (int units = 1; units <= 40; ++units) bad += !bijection(gx, units, 1, pairs);
    bad += !bijection(13, 5, 7, pairs);
    bad += !bijection(60000, 7, 2, pairs);   // 105 000 blocks an XCD, 45 000 of them dealt: past 31 bits
    bad += !bijection(46339, 9, 1, pairs);
  }
  std::printf("%%d\n", bad);
  return bad != 0;
}
"""


def test_causal_block_order_is_a_bijection(tmp_path):
    text = open(HEADER).read()
    body = re.search(r"__device__ inline BlockId causal_block_id\(bool pairs\) \{\n.*?\n\}\n", text, re.S).group(0)
    src, exe = tmp_path / "order.cpp", str(tmp_path / "order")
    src.write_text(DRIVER % body)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-fsanitize=undefined", "-fno-sanitize-recover=undefined", "-o", exe, str(src)])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout, r.stderr[-2000:])
