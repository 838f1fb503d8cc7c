"""The order of a simulation's sources, and with it the tiles and the cuts of their walks,
does not depend on the batch the simulation is searched in (csrc/batch.hpp: hilbert_bits,
source_key). The library's own functions, compiled for the host: the keys of a simulation's
sources in an ensemble order them, ties included, as its keys alone do, stay below the
next group's, and fit the bits the sort takes."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
BATCH = os.path.join(os.path.dirname(HERE), "paper_2509_26193_amd", "csrc", "batch.hpp")

HARNESS = r"""
#include <stdint.h>
#include <stdio.h>
#include <algorithm>
#include <random>
#include <vector>
%s
int main() {
  std::mt19937_64 rng(5);
  const int64_t sizes[] = {1, 4096, 16384, 16385, 131072, 262145, 1 << 23, 1 << 25};
  const int nsims[] = {1, 2, 64, 256, 257, 2048, 100000};
  for (int64_t n : sizes)
    for (int64_t largest : sizes)
      for (int ns : nsims) {
        if (largest < n || (ns == 1 && largest != n)) continue;
        const int own = hilbert_bits(n), bits = hilbert_bits(largest);
        int gb = 1;
        while ((1ll << gb) < 2ll * ns) ++gb;
        // indices all over the cube, and close together in one place of it
        std::vector<uint64_t> h(400);
        for (int k = 0; k < 400; ++k) h[k] = (k < 200 ? rng() : (rng() >> (1 + k %% 60))) >> 1;
        for (uint64_t group : {(uint64_t)0, (uint64_t)(2 * ns - 1)})
          for (uint64_t a : h) {
            const uint64_t ka = source_key(group, a, own, bits);
            if (gb + bits < 64 && ka >> (gb + bits)) return printf("bits\n"), 1;
            if (ka >> bits != group) return printf("group\n"), 1;
            for (uint64_t b : h) {
              const uint64_t kb = source_key(group, b, own, bits);
              const uint64_t sa = source_key(0, a, own, own), sb = source_key(0, b, own, own);
              if ((ka < kb) != (sa < sb) || (ka == kb) != (sa == sb)) return printf("order\n"), 1;
            }
          }
      }
  printf("ok\n");
  return 0;
}
"""


def test_order_of_a_simulation_is_its_own(tmp_path):
    src = open(BATCH).read()
    code = ""
    for f in ("int hilbert_bits", "uint64_t source_key"):
        one = re.search(r"^__host__ __device__ (inline %s\([^{]*\{(?:[^\n]*\}$|.*?^\}))" % f, src,
                        re.S | re.M)
        assert one, f
        code += one.group(1) + "\n"
    cpp = tmp_path / "order.cpp"
    cpp.write_text(HARNESS % code)
    exe = tmp_path / "order"
    subprocess.check_call(["g++", "-O2", "-std=c++17", str(cpp), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
