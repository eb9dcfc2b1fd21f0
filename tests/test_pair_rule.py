"""Which whole-site LDS launches take the pair form, on the host: the rule of the launcher against the one
bench.py names kernels by, over every format, tile count and lattice size where either changes, and
the shipped launch table, whose entries were timed with the pair form."""
import itertools
import os
import subprocess

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FORMATS = [(16, 18)] + [(e, r) for e in (8, 4) for r in (18, 14, 13, 9)]
LATTICES = [(4, 4, 4, 4), (16, 16, 16, 8), (20, 10, 18, 10), (16, 16, 16, 16), (24, 16, 16, 16), (28, 20, 24, 14),
            (24, 32, 16, 16), (32, 32, 32, 8)]

PROGRAM = r"""
#include "dslash_kernel.hpp"
#include <cstdio>
int main() {
  int elem, nr, rt, wpb, epi, nt, nb;
  while (std::scanf("%d %d %d %d %d %d %d", &elem, &nr, &rt, &wpb, &epi, &nt, &nb) == 7)
    std::printf("%d\n", int(dslash::pair_form_pays(elem, nr, rt, wpb, epi != 0, nt, nb)));
}
"""


def test_launch_rule_and_kernel_names_agree(tmp_path):
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text(PROGRAM)
    res = subprocess.run(["/opt/rocm/bin/hipcc", "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1409_1510_amd", "csrc"),
                          str(src), "-o", str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    cases = [(f, d, rt, lds, fused, n) for f, d, rt, lds, fused, n in
             itertools.product(FORMATS, LATTICES, (1, 2, 4), (1, 2, 3), (False, True), range(1, 65))
             if not (rt == 4 and lds == 3)]
    lines = []
    for (elem, nr), d, rt, lds, fused, n in cases:
        nb = -(-(d[0] * d[1] * d[2] * d[3] // 2) // 64)
        lines.append(f"{elem} {nr} {rt} {4 << (lds - 1)} {int(fused)} {-(-n // rt)} {nb}")
    res = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, timeout=300)
    got = [v == "1" for v in res.stdout.split()]
    assert len(got) == len(cases) and any(got) and not all(got)
    for ((elem, nr), d, rt, lds, fused, n), pays in zip(cases, got):
        name = bench.dslash_kernel_name((rt, 64, 0, lds, 0), d, n, elem, nr, fused)
        assert (name == "k_dslash_pair") == pays, (elem, nr, d, rt, lds, fused, n)


def test_shipped_entries_keep_the_pair_form():
    path = os.path.join(ROOT, "paper_1409_1510_amd", "tuning", "gfx950.txt")
    seen = 0
    for line in open(path):
        f = line.split()
        if not f or f[0].startswith("#"):
            continue
        lx, ly, lz, lt, prec, recon, n, fused, rt, spb, nt, lds, xm = map(int, f[:13])
        if spb == 64 and 1 <= lds <= 3 and (rt <= 2 if prec == 0 else rt >= 2):
            name = bench.dslash_kernel_name((rt, spb, nt, lds, xm), (lx, ly, lz, lt), n, (16, 8, 4)[prec], recon, bool(fused))
            assert name == "k_dslash_pair", line
            seen += 1
    assert seen > 30
