"""Which decoder of short buckets a step takes, asked of the library's own rule on the host, for steps
that were timed with all of them (us, from an MI355X; normal and heavy-tailed values, messages cut to
their length): the one that was the fastest, or one within a tenth of it.  And what is known of the
strings' length: a message in a whole buffer says nothing, and does not hide what the others say."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
PKG = os.path.join(ROOT, "paper_1610_02132_amd")
LIB = os.path.join(PKG, "libqsgd.so")
pytestmark = pytest.mark.skipif(not shutil.which(HIPCC) or not os.path.exists(LIB), reason="needs hipcc and the library")

ASK = r"""
#include "qsgd_capi.hip"
#include <cstdio>
int main() {   // n d s code norm K, words of a string, messages in whole buffers
  unsigned long long n, d; unsigned s, code, norm, K, whole; double words;
  while (std::scanf("%llu %llu %u %u %u %u %lf %u", &n, &d, &s, &code, &norm, &K, &words, &whole) == 8) {
    qsgd_params p; std::memset(&p, 0, sizeof p);
    p.n = n; p.d = d; p.s = s; p.code = code; p.norm = norm;
    Geometry g;
    if (make_geometry(&p, g)) return 1;
    DecodeArgs a; std::memset(&a, 0, sizeof a);
    a.K = K; a.n = g.n; a.d = (uint32_t)g.d; a.nb = (uint32_t)g.nb; a.s = s; a.code = code;
    size_t bytes[QSGD_MAX_PEERS];
    for (unsigned k = 0; k < K; ++k)
      bytes[k] = k < whole ? qsgd_max_encoded_bytes(&p)
                           : 4 * (size_t)(H_WORDS + g.table_words + words * (double)g.nb);
    const StringLength w = string_length(g, nullptr, bytes, K);
    const SplitPlan split = plan_decode_split(a, 256, w.planned(), 0);
    std::printf("%d %.3f %.3f %d\n", g.d > kEntryMinD ? 2 : (int)choose_decoder(g, a, w, 256).which, w.words,
                w.guess, split.bits ? 0 : (int)split.waves);
  }
}
"""
SPARSE, DENSE, L2, MAX = 0, 1, 0, 1
RING, TILE, SPLIT = 0, 1, 2

# n, d, s, code, norm, K, words of a string, (ring, tile, split) us
STEPS = [
    (41086512, 2796, 1, SPARSE, L2, 1, 18.8, (107, 125, 180)),
    (23576477, 684, 1, SPARSE, L2, 2, 8.3, (82, 96, 147)),
    (43002281, 2380, 2, SPARSE, L2, 1, 29.1, (132, 164, 256)),
    (12382431, 1464, 1, SPARSE, L2, 6, 8.8, (58, 78, 100)),
    (1586796, 2892, 1, SPARSE, MAX, 1, 81.9, (207, 88, 22)),
    (140783, 3280, 38, DENSE, L2, 16, 306.7, (None, 196, 115)),
    (121594, 516, 3, SPARSE, MAX, 19, 30.7, (360, 48, 37)),
    (3631300, 3424, 8, SPARSE, MAX, 4, 434.8, (2368, 269, 202)),
    (45873, 3380, 36, SPARSE, L2, 23, 196.8, (1669, 175, 148)),
    (114579, 548, 17, DENSE, MAX, 27, 95.9, (None, 98, 80)),
    (555644, 3880, 59, DENSE, L2, 23, 366.4, (None, 327, 204)),
    (5916, 1488, 25, DENSE, MAX, 31, 193.0, (None, 195, 133)),
    (574453, 292, 16, SPARSE, L2, 1, 22.9, (138, 25, 19)),
    (14859789, 3500, 34, DENSE, MAX, 2, 782.0, (None, 828, 655)),
    (12469531, 228, 3, SPARSE, L2, 4, 8.5, (120, 57, 218)),
    (48254841, 96, 9, DENSE, L2, 8, 10.9, (None, 264, 3579)),
    (24756319, 3572, 2, SPARSE, L2, 5, 36.6, (210, 144, 296)),
    (36678, 88, 1, SPARSE, MAX, 9, 4.9, (28, 16, 18)),
    (42785835, 7408, 3, SPARSE, L2, 3, 76.8, (356, 267, 355)),
    (9360, 100, 7, DENSE, L2, 3, 10.2, (None, 16, 20)),
    (98864, 236, 13, DENSE, L2, 14, 24.9, (None, 23, 29)),
    (356618, 231, 10, DENSE, L2, 5, 21.7, (None, 21, 30)),
    (141298, 176, 1, SPARSE, L2, 9, 4.4, (22, 17, 25)),
    (27777, 304, 12, DENSE, L2, 30, 28.1, (None, 27, 51)),
    (67_000_000, 8192, 4, SPARSE, L2, 16, 102.4, (583, 394, None)),
    (67_000_000, 4096, 3, SPARSE, L2, 16, 27.0, (206, 362, None)),
    (67_000_000, 2048, 2, SPARSE, L2, 16, 26.7, (285, 349, None)),
    (268_000_000, 8192, 7, SPARSE, L2, 16, 154.5, (2194, 1447, None)),
    (268_000_000, 8192, 4, SPARSE, L2, 16, 102.4, (1061, 1299, None)),
    (268_000_000, 1024, 1, SPARSE, L2, 16, 11.0, (639, 1197, None)),
    (1_000_000_000, 8192, 4, SPARSE, L2, 16, 46.0, (1780, 3678, 21400)),
]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    path = tmp_path_factory.mktemp("ask")
    (path / "ask.hip").write_text(ASK)
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-Wno-unused-function",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc"), str(path / "ask.hip"),
                    "-o", str(path / "ask"), "-L", PKG, "-lqsgd", "-Wl,-rpath," + PKG], check=True, capture_output=True)

    def answers(rows):
        text = "".join(" ".join(map(str, r)) + "\n" for r in rows)
        out = subprocess.run([str(path / "ask")], input=text, capture_output=True, text=True, check=True).stdout
        return [(int(a), float(b), float(c), int(d)) for a, b, c, d in (line.split() for line in out.splitlines())]
    return answers


def test_the_fastest_decoder_or_nearly(ask):
    for step, (which, _, _, _) in zip(STEPS, ask([s[:7] + (0,) for s in STEPS])):
        times = step[7]
        assert times[which] is not None and times[which] <= 1.1 * min(t for t in times if t), (step, which)


def test_a_whole_buffer_does_not_hide_the_others(ask):
    n, d, s, K, words = 20_000_000, 8192, 4, 16, 38.0       # outliers: strings of a third of the guess
    cut, one, all_ = ask([(n, d, s, SPARSE, L2, K, words, w) for w in (0, 1, K)])
    guess = cut[2]
    assert words < 0.5 * guess
    assert abs(cut[1] - (words + 0.5)) < 0.01
    assert abs(one[1] - ((K - 1) * (words + 0.5) + guess) / K) < 0.01
    assert abs(all_[1] - guess) < 0.01
    assert one[0] == cut[0] != all_[0]


def test_strings_longer_than_the_guess_count(ask):
    """... up to twice of it: a buffer of another size than the worst case is no length."""
    shape = (1_000_000, 512, 4, SPARSE, L2, 4)
    guess = ask([shape + (1.0, 4)])[0][2]
    assert abs(ask([shape + (1.5 * guess, 0)])[0][1] - (1.5 * guess + 0.5)) < 0.05
    assert ask([shape + (3.0 * guess, 0)])[0][1] == pytest.approx(2.0 * guess, abs=0.01)


@pytest.mark.parametrize("n,d,s,K,waves", [
    (43_649, 15_102, 58, 16, 16), (20_162, 20_162, 122, 8, 16), (520_000, 520_000, 80, 8, 16),   # one for a compute unit
    (530_000, 530_000, 80, 4, 12), (3_400_000, 3_400_000, 80, 6, 8), (4_000_000, 100_000, 80, 16, 8),
    (4_000_000, 100_000, 80, 8, 4), (16_000_000, 9770, 85, 4, 2),
    (16_000_000, 9770, 85, 16, 4), (9_000, 9_000, 80, 1, 3),                                       # (no more words than that)
])
def test_wavefronts_of_a_segment(ask, n, d, s, K, waves):
    """The fewer segments a compute unit has, the more wavefronts share one."""
    assert ask([(n, d, s, DENSE, L2, K, 0, K)])[0][3] == waves


def test_the_ring_decoder_is_kept_to_what_it_reads(ask):
    """Code_s under the L2 scale, 32 messages at most (a bit each in a word), loads of four values, and no
    shorter buckets than it was ever taken for."""
    rows = [(n, d, s, code, norm, K, w, 0)
            for n in (4_000, 500_000, 60_000_000) for d in (4, 20, 60, 64, 254, 1024, 8190, 8192) for s in (1, 3, 40)
            for code in (SPARSE, DENSE) for norm in (L2, MAX) for K in (1, 8, 33, 64) for w in (1.2, 9.0, 200.0)]
    chosen = [r for r, a in zip(rows, ask(rows)) if a[0] == RING]
    assert chosen
    for n, d, s, code, norm, K, _, _ in chosen:
        assert code == SPARSE and norm == L2 and K <= 32 and d % 4 == 0 and d >= 64
