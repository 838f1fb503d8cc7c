"""The list of values a call reads back (csrc/common.hpp, ReadBack) holds kReadMost of them and
never writes past its arrays; one too many is counted, for the call to refuse."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
COMMON = os.path.join(os.path.dirname(HERE), "paper_2509_26193_amd", "csrc", "common.hpp")

HARNESS = r"""
#include <stdint.h>
#include <stdio.h>
%s
struct Guarded {
  ReadBack r;
  uint64_t after = 0x5EED5EED5EED5EEDull;
};
int main() {
  Guarded g;
  int32_t a[3 * kReadMost];
  int64_t b[3 * kReadMost];
  for (int k = 0; k < 3 * kReadMost; ++k) {
    if (k & 1) g.r.add(&b[k]);
    else g.r.add(&a[k]);
    if (g.r.count != k + 1) return 1;
    for (int q = 0; q <= k && q < kReadMost; ++q)
      if (g.r.from[q] != (q & 1 ? (const void*)&b[q] : (const void*)&a[q]) ||
          g.r.wide[q] != (q & 1)) return 2;
  }
  return g.after != 0x5EED5EED5EED5EEDull ? 3 : 0;
}
"""


def test_room_of_the_list(tmp_path):
    src = open(COMMON).read()
    code = re.search(r"^constexpr int kReadMost = \d+;", src, re.M).group(0) + "\n" + \
        re.search(r"^struct ReadBack \{.*?^\};", src, re.S | re.M).group(0)
    cpp = tmp_path / "r.cpp"
    cpp.write_text(HARNESS % code)
    exe = tmp_path / "r"
    subprocess.check_call(["g++", "-O1", "-std=c++17", str(cpp), "-o", str(exe)])
    assert subprocess.run([str(exe)]).returncode == 0
    body = re.search(r"inline hipError_t read_back\(.*?\{(.*?)ReadLease", src, re.S).group(1)
    assert "R.count > kReadMost" in body
