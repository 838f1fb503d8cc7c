"""Every part of a search's tiles has at least two checkpoint slots inside the array that
holds them (csrc/batch.hpp: parts_log, slots_log, max_parts_for, search_size_in). The
library's own sizing functions, compiled for the host, are evaluated over ensembles from
one simulation to many thousands, of one size and of mixed sizes, with few and with all
neurons searching, on devices from 16 to 288 GB: the tiles' parts stay within their bound,
and the slots that the preparation hands out, halved as it halves them, within the array."""
import os
import re
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2509_26193_amd", "csrc")

HARNESS = r"""
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <algorithm>
#include <vector>
%s
int main() {
  // no round of fitting without checkpoints, and after the last one two slots for each part
  if (slot_cuts(0) != 0) return printf("rounds without checkpoints\n"), 1;
  for (int ck : {kCkptMin, kCkptMax})
    for (int p = 0; p <= kPartLogMax; ++p)
      if (slots_log(p, ck, slot_cuts(ck)) != 1) return printf("slots at the end\n"), 1;
  const double shares[] = {0.02, 0.3, 0.7, 1.0};
  const int64_t sizes[] = {1, 64, 1000, 2500, 4000, 4096, 5000, 8192, 20000, 65536, 262144,
                           1 << 20, 1 << 23, 1 << 25};
  const int sims[] = {1, 2, 7, 64, 500, 2048, 4096, 6500, 8192, 9000, 30000};
  const double gbs[] = {16, 64, 192, 288};
  long checked = 0, tight = 0;
  for (int64_t n : sizes)
    for (int ns : sims) {
      if (n * ns >= ((int64_t)1 << 31) - 4096) continue;
      for (int mixed = 0; mixed < 2; ++mixed)
        for (double share : shares)
          for (double gb : gbs)
            for (int force = -1; force <= (ns == 1 ? 3 : -1); ++force) {
              std::vector<int64_t> own(ns, n);
              if (mixed)                            // sizes spread below n
                for (int k = 0; k < ns; ++k) own[k] = 1 + (n * ((k * 7919ll) %% 97 + 1)) / 97;
              int64_t total = 0;
              for (int64_t v : own) total += std::min(v, n);
              const SearchSize q = search_size_in((size_t)(gb * 1e9), total, ns, force, false);
              int64_t parts = 0, least = 0;
              std::vector<int64_t> ts(ns);
              for (int k = 0; k < ns; ++k) {
                const int64_t s = (int64_t)(share * std::min(own[k], n)), e = s * 4 / 5;
                ts[k] = (e + kWave - 1) / kWave + (s - e + kWave - 1) / kWave;
                parts += ts[k] << parts_log(ts[k], force);
              }
              if (parts > max_parts_for(total, ns, force)) return printf("parts\n"), 1;
              for (int ck : {q.slots, kCkptMin}) {  // (a tuned plan may aim at fewer)
                int64_t sum = 0;
                for (int cut = 0; cut <= slot_cuts(ck); ++cut) {
                  sum = 0;
                  for (int k = 0; k < ns; ++k) {
                    const int p = parts_log(ts[k], force);
                    sum += (ts[k] << p) << slots_log(p, ck, cut);
                  }
                  if (sum <= q.ck_cap) break;
                }
                if (sum > q.ck_cap) {
                  printf("%%d simulations of %%ld, %%g searching, %%g GB: %%ld slots of %%ld\n",
                         ns, (long)n, share, gb, (long)sum, (long)q.ck_cap);
                  return 1;
                }
                ++checked;
                tight += sum == 2 * parts;
              }
            }
    }
  printf("ok %%ld %%ld\n", checked, tight);
  return 0;
}
"""


def _text(src, pattern):
    m = re.search(pattern, src, re.S | re.M)
    assert m, pattern
    return m.group(0)


def test_every_part_has_its_slots(tmp_path):
    wave = open(os.path.join(CSRC, "search_wave.hpp")).read()
    batch = open(os.path.join(CSRC, "batch.hpp")).read()
    code = "constexpr int kWave = 64;\n"
    for c in ("kCkptMax", "kCkptMin", "kPartLogMax", "kPartsFine", "kPartsMax", "kMinSlots"):
        code += _text(wave, r"^constexpr int %s = \d+;" % c) + "\n"
    code += _text(batch, r"^constexpr size_t kCkptSlotBytes =.*?;") + "\n"
    code += _text(batch, r"^struct SearchSize \{.*?^\};") + "\n"
    for f in ("int parts_log", "int slots_log", "int slot_cuts", "int64_t max_tiles_for", "int64_t max_parts_for",
              "SearchSize search_size_in"):
        one = _text(batch, r"^(?:__host__ __device__ )?inline %s\([^{]*\{(?:[^\n]*\}$|.*?^\})" % f)
        code += one.replace("__host__ __device__ ", "") + "\n"
    cpp = tmp_path / "room.cpp"
    cpp.write_text(HARNESS % code)
    exe = tmp_path / "room"
    subprocess.check_call(["g++", "-O2", "-std=c++17", str(cpp), "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    ok, checked, tight = r.stdout.split()
    assert ok == "ok" and int(checked) > 5000 and int(tight) > 0
