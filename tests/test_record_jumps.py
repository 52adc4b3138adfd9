"""The split decoder's lane for every bit finds where a word is left by three doublings of a jump of one
look-up: eight jumps have to leave a word from any of its bits.  The compiler evaluates the table's own
constructor, from the source, over every entry."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(ROOT, "paper_1610_02132_amd", "csrc")

CHECK = """
#include "qsgd_decode_split.hip"
namespace qsgd {
constexpr Records<QSGD_CODE_SPARSE> kRecords;
// the fewest bits that a jump of two records passes, and that a jump of one record and the jump behind
// it pass: the second record does not fit in what the first one leaves of the kBits bits
constexpr uint32_t fewest(bool two) {
  uint32_t least = 64;
  for (uint32_t i = 0; i < kEntries; ++i) {
    const uint32_t e = kRecords.e[i], n = e & 15u, both = (e >> 4) & 15u;
    if (n == 0 || (both != n) != two) continue;
    if (two) { least = both < least ? both : least; continue; }
    for (uint32_t f = 0; f < (1u << n); ++f) {   // whatever the bits behind the kBits are
      const uint32_t next = kRecords.e[((i << n) & (kEntries - 1u)) | f] & 15u;
      const uint32_t sum = n + (next ? next : kBits + 1u);
      least = sum < least ? sum : least;
    }
  }
  return least;
}
// a lone record that is the last jump passes 3 bits: the worst of eight jumps
constexpr uint32_t kTwo = fewest(true), kPair = fewest(false);
constexpr uint32_t passed(uint32_t jumps) {
  uint32_t best[9] = {0};
  for (uint32_t j = 1; j <= jumps; ++j) {
    const uint32_t last = j == jumps ? 3u : 64u;
    best[j] = best[j - 1] + (kTwo < last ? kTwo : last);
    if (j >= 2 && best[j - 2] + kPair < best[j]) best[j] = best[j - 2] + kPair;
  }
  return best[jumps];
}
static_assert(kTwo == 6, "two records");
static_assert(kPair == %d, "one record, and the one behind it");
static_assert(passed(8) >= 32, "eight jumps leave a word");
}
"""


def compiles(tmp_path, text):
    src = tmp_path / "check.hip"
    src.write_text(text)
    r = subprocess.run([HIPCC, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-std=c++17",
                        "-fsyntax-only", "-fconstexpr-steps=2000000000", "-Wno-unused-function",
                        "-I", os.path.join(ROOT, "include"), "-I", CSRC, str(src)],
                       capture_output=True, text=True, timeout=300)
    return r.returncode == 0, r.stderr


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no hipcc")
def test_eight_jumps_leave_a_word(tmp_path):
    ok, said = compiles(tmp_path, CHECK % 11)
    assert ok, said[-2000:]
    ok, said = compiles(tmp_path, CHECK % 12)      # (the check looks)
    assert not ok and "one record, and the one behind it" in said
