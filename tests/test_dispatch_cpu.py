"""The rules that choose kernels (csrc/internal.hpp), compiled for the host:
each takes the faster side at points measured on an MI355X (256 CUs, us per
call, calls back to back), and both sides of each line occur."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256
MAIN = r"""
#include <cstdio>
#include <cstring>
#include "internal.hpp"
using namespace rosetta;
int main() {
  char what[16];
  unsigned n, N, l, beta;
  unsigned long long batch, cus;
  while (scanf("%15s %u %u %u %u %llu %llu", what, &n, &N, &l, &beta, &batch, &cus) == 7) {
    rosetta_params p{};
    p.n = n; p.k = 1; p.N = N; p.ks_level = p.pbs_level = l; p.ks_base_log = p.pbs_base_log = beta;
    if (!strcmp(what, "ks"))
      printf("%d\n", (int)ks_route(p, batch, cus));
    else if (!strcmp(what, "br"))
      printf("%d\n", fft_pieces(p));
    else
      printf("%d\n", trace_pieces(N, l, beta, batch, cus));
  }
}
"""


def build_rule(d):
    """Compile the rules in directory d; returns ask(rows), which runs them."""
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2609_16915_amd/csrc", "main.cpp", "-o", "main"],
                   cwd=d, check=True)

    def ask(rows):
        text = "".join(" ".join(map(str, r)) + "\n" for r in rows)
        out = subprocess.run([str(d / "main")], input=text, capture_output=True, text=True, check=True)
        return [int(x) for x in out.stdout.split()]
    return ask


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    return build_rule(tmp_path_factory.mktemp("dispatch"))


VALU, SPLIT, DIGITS, MFMA = range(4)
# (n, N, level, base, batch): k_keyswitch_mfma, digits made once
KS_MEASURED = [
    ((16, 256, 1, 4, 4097), 19, 29), ((31, 256, 1, 4, 65536), 36, 93), ((64, 256, 1, 4, 1361), 18, 29),
    ((95, 256, 1, 4, 32768), 52, 65), ((128, 256, 1, 4, 16384), 45, 39), ((200, 256, 1, 4, 577), 18, 30),
    ((1024, 256, 1, 4, 896), 21, 30), ((2048, 256, 1, 4, 49), 15, 30), ((2048, 256, 1, 4, 1152), 43, 31),
    ((1024, 256, 2, 4, 113), 25, 29), ((2048, 256, 2, 4, 98), 24, 29), ((1024, 256, 2, 4, 896), 32, 29),
    ((31, 256, 3, 4, 9000), 33, 31), ((20, 256, 3, 4, 12288), 35, 34), ((16, 256, 3, 4, 32768), 39, 62),
    ((20, 512, 2, 4, 16384), 57, 61), ((20, 512, 2, 4, 131072), 186, 390), ((50, 512, 1, 4, 12288), 40, 50),
    ((20, 1024, 2, 4, 12288), 109, 88), ((20, 1024, 2, 4, 20480), 110, 130), ((742, 256, 1, 4, 3328), 43, 30),
    ((80, 512, 2, 4, 16384), 72, 66), ((80, 512, 2, 4, 20480), 70, 80), ((80, 512, 2, 4, 22528), 118, 95),
    ((20, 1024, 5, 3, 16384), 184, 147), ((20, 1024, 5, 3, 24576), 185, 217), ((50, 1024, 5, 3, 131072), 1014, 1183),
    ((20, 2048, 6, 3, 20480), 431, 413), ((20, 2048, 6, 3, 28672), 437, 508), ((50, 2048, 6, 3, 131072), 2179, 2722),
    ((63, 4096, 6, 3, 32768), 956, 1436), ((1, 4096, 6, 3, 65536), 1093, 2718), ((64, 4096, 6, 3, 32768), 1990, 1435),
    ((80, 2048, 6, 3, 131072), 3251, 2784), ((742, 1024, 1, 7, 161), 57, 30), ((742, 2048, 5, 3, 3000), 732, 272),
    ((1024, 2048, 6, 3, 113), 398, 130), ((1024, 2048, 6, 3, 9000), 2390, 959), ((2048, 4096, 6, 3, 49), 735, 323),
]


def test_key_switch_takes_the_faster_kernel(rule):
    got = rule([("ks", *c, CUS) for c, _, _ in KS_MEASURED])
    for (c, mfma, digits), route in zip(KS_MEASURED, got):
        assert route in (MFMA, DIGITS), c
        chosen, other = (mfma, digits) if route == MFMA else (digits, mfma)
        assert chosen <= 1.1 * other, (c, mfma, digits)
    assert set(got) == {MFMA, DIGITS}


def test_key_switch_split_and_valu(rule):
    """16 ciphertexts x 32 columns per CU split the contraction; digits wider
    than a byte take the VALU kernel."""
    rows = [("ks", 1024, 2048, 6, 3, 112, CUS), ("ks", 1024, 2048, 6, 3, 113, CUS), ("ks", 31, 256, 3, 4, 4096, CUS),
            ("ks", 31, 256, 3, 4, 4097, CUS), ("ks", 64, 1024, 2, 9, 5, CUS)]
    assert rule(rows) == [SPLIT, DIGITS, SPLIT, DIGITS, VALU]


# (N, level, base, batch): modular trace, double precision
TRACE_MEASURED = [
    ((2048, 1, 13, 1), 130, 118), ((2048, 1, 13, 256), 132, 123), ((2048, 1, 13, 512), 174, 178),
    ((2048, 1, 13, 513), 229, 250), ((2048, 1, 13, 4096), 1077, 1157), ((2048, 1, 18, 1), 134, 117),
    ((2048, 1, 18, 512), 183, 179), ((2048, 1, 18, 8192), 2188, 2276), ((4096, 1, 12, 1), 206, 219),
    ((4096, 1, 12, 256), 215, 233), ((4096, 1, 12, 300), 424, 429), ((4096, 1, 12, 14336), 11989, 11301),
    ((4096, 1, 17, 64), 220, 227), ((4096, 1, 17, 513), 656, 628), ((4096, 1, 17, 14336), 12324, 11320),
    ((2048, 2, 17, 4096), 1557, 1304), ((4096, 2, 16, 1), 294, 239), ((2048, 4, 12, 14336), 7470, 5850),
]


def test_trace_takes_the_faster_kernel(rule):
    got = rule([("tr", 1, *c, CUS) for c, _, _ in TRACE_MEASURED])
    for (c, modular, double), pieces in zip(TRACE_MEASURED, got):
        chosen, other = (double, modular) if pieces else (modular, double)
        assert chosen <= 1.03 * other, (c, pieces)
    assert set(got) == {0, 4}


def test_trace_pieces_elsewhere_follow_the_bound(rule):
    """Other levels, digit widths and rings keep what exactness allows, at any
    batch."""
    def bound(N, l, b):
        holds = lambda bits: b + bits - 2 < 40 and l * N * 160 << (b + bits - 2) <= 1 << 51
        return 0 if N < 2048 else 3 if holds(22) else 4 if holds(16) else 0
    rows = [(N, l, b, batch) for N in (256, 1024, 2048, 4096) for l in (1, 2, 3, 4) for b in range(1, 31)
            for batch in (1, 256, 257, 512, 513, 14336) if l * b <= 62]
    for (N, l, b, batch), got in zip(rows, rule([("tr", 1, *r, CUS) for r in rows])):
        want = bound(N, l, b)
        assert got == want or (got, l, want) == (0, 1, 4), (N, l, b, batch)


def test_benchmark_names_the_kernels_of_these_rules(rule):
    """bench.py states the rules again, for its rooflines."""
    import bench
    assert bench.CU == CUS
    names = ["k_keyswitch", "k_keyswitch_small", "k_keyswitch_gemm", "k_keyswitch_mfma"]
    ks = [(n, N, l, b, batch) for n in (1, 31, 32, 63, 64, 95, 96, 742, 1024, 2048) for N in (256, 512, 1024, 2048, 4096)
          for l, b in ((1, 4), (1, 7), (2, 5), (3, 4), (6, 3), (3, 9))
          for batch in (1, 16, 100, 257, 900, 2000, 5000, 10300, 14400, 18000, 21000, 70000)]
    for c, got in zip(ks, rule([("ks", *c, CUS) for c in ks])):
        assert bench.keyswitch_kernel(*c) == names[got], c
    br = [(N, l, b, batch) for N in (256, 1024, 2048, 4096) for l in (1, 2, 3, 4) for b in range(1, 31)
          for batch in (1, 256, 257, 512, 513) if l * b <= 62]
    for c, pieces, tr in zip(br, rule([("br", 1, *c, CUS) for c in br]), rule([("tr", 1, *c, CUS) for c in br])):
        assert bench.key_pieces(*c[:3]) == pieces and bench.trace_pieces(*c) == tr, c
