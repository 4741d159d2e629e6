"""The launch rules (csrc/mala_dispatch.h) on the sizes of calls, on the CPU: a small C++
program compiled against the header answers for the shapes below."""
import os
import shutil
import subprocess

import pytest

from paper_2609_32712_amd import build as libbuild

CXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")

PROGRAM = r"""
#include <cstdio>
#include "mala_dispatch.h"
using namespace mala;
struct P {
  const void* cu;
  const void* counters;
  int B, Hq, Hkv, Nq, Nk, max_len, max_len_k, nkblk, psize, nparts;
  float log2tau;
};
int main() {
  // kind (0 fixed, 1 packed), B (sequences), Hq, Hkv, Nq, Nk (totals), longest q, longest k, D, tau
  int kind, D;
  double tau;
  P p;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %lf", &kind, &p.B, &p.Hq, &p.Hkv, &p.Nq, &p.Nk,
                    &p.max_len, &p.max_len_k, &D, &tau) == 10) {
    p.cu = kind ? &p : nullptr;
    p.counters = nullptr;
    p.nkblk = (p.max_len_k + kBwdKeys - 1) / kBwdKeys;
    p.log2tau = std::log2(tau);
    if (kind)
      dkdv_split_packed(p.B, p.max_len, p.Nk, p.Hq, p.Hkv, &p.psize, &p.nparts);
    else
      dkdv_split(p.B, p.Hq, p.Hkv, p.Nq, p.Nk, &p.psize, &p.nparts);
    std::printf("%s\n", answer(p, D));
  }
}
"""


def _ask(tmp_path, answer, lines):
    """Answers of the C++ function body `answer` (const char* from P p, int D)."""
    src, exe = str(tmp_path / "ask.cpp"), str(tmp_path / "ask")
    head, main = PROGRAM.split("int main")
    with open(src, "w") as f:
        f.write(head + "const char* answer(const P& p, int D) {\n" + answer + "}\nint main" + main)
    subprocess.run([CXX, "-std=c++17", "-Wall", "-Werror", "-I" + libbuild.CSRC, src, "-o", exe],
                   check=True)
    text = "\n".join(" ".join(map(str, x)) for x in lines)
    return subprocess.run([exe], input=text, check=True, capture_output=True, text=True).stdout.split()


def _fixed(B, Hq, Hkv, Nq, Nk, D, tau):
    return (0, B, Hq, Hkv, Nq, Nk, Nq, Nk, D, tau)


DKDV = """  switch (dkdv_plan(p, D).rule) {
    case DkdvRule::kPairs: return "pairs";
    case DkdvRule::kBlocks: return "blocks";
    case DkdvRule::kBySequence: return "sequence";
  }
  return "";
"""


def test_dkdv_kernel_of_fixed_length_calls(tmp_path):
    # the faster kernel by measurement (backwards at tau = 1e-3, all tiles retained)
    want = {(1, 8, 2, 1024, 1024): "pairs", (1, 8, 2, 4096, 4096): "pairs",
            (4, 8, 2, 4096, 4096): "pairs", (16, 8, 2, 700, 700): "pairs",
            (1, 8, 8, 4096, 4096): "pairs", (1, 32, 8, 1024, 1024): "pairs",
            (1, 32, 8, 256, 2048): "pairs", (1, 8, 1, 4096, 4096): "pairs",
            (8, 8, 2, 4096, 4096): "blocks", (1, 8, 2, 131072, 131072): "blocks",
            # sweeps alike: the pairs' work and not the chain of one sweep sets the time
            (2, 8, 2, 2048, 8192): "blocks", (8, 16, 16, 32, 256): "blocks",
            (4, 8, 8, 64, 1024): "blocks", (1, 32, 8, 512, 4096): "blocks",
            (2, 16, 4, 1024, 4096): "blocks", (1, 4, 4, 2048, 8192): "blocks",
            (1, 8, 2, 512, 16384): "blocks", (1, 16, 2, 1000, 9000): "blocks",
            (2, 4, 4, 500, 3000): "blocks", (16, 8, 8, 256, 256): "blocks",
            (1, 32, 32, 1024, 1024): "blocks", (1, 8, 1, 8192, 8192): "blocks"}
    got = _ask(tmp_path, DKDV, [_fixed(*x, 128, 1e-3) for x in want])
    assert dict(zip(want, got)) == want
    # tolerances that may skip: by sequence where the blocks kernel would have long sweeps,
    # and at D = 128 pairs where they are short and few, but not of an iteration or two
    skip = {(8, 8, 2, 4096, 4096): "sequence", (1, 8, 2, 131072, 131072): "sequence",
            (2, 8, 2, 2048, 8192): "sequence", (1, 8, 2, 4096, 4096): "pairs",
            (1, 32, 32, 1024, 1024): "pairs", (1, 32, 8, 512, 4096): "pairs",
            (8, 16, 16, 32, 256): "blocks", (4, 8, 8, 64, 1024): "blocks",
            (16, 8, 8, 256, 256): "blocks"}
    got = _ask(tmp_path, DKDV, [_fixed(*x, 128, 1.0) for x in skip])
    assert dict(zip(skip, got)) == skip
    got = _ask(tmp_path, DKDV, [_fixed(*x, 64, 1.0) for x in want])
    assert all(g == want[x] or g == "sequence" and x[3] * x[1] // x[2] >= 512 * 32
               for x, g in zip(want, got))


def _packed(lens, Hq, Hkv, D, tau):
    return (1, len(lens), Hq, Hkv, sum(lens), sum(lens), max(lens), max(lens), D, tau)


PACKED = """  static char s[64];
  const DkdvPlan q = dkdv_plan(p, D);
  std::snprintf(s, sizeof(s), "%s%s%s",
                q.rule == DkdvRule::kPairs ? "pairs" : q.rule == DkdvRule::kBlocks ? "blocks" : "sequence",
                q.parts ? "+parts" : "", q.rule == DkdvRule::kBySequence && q.block_parts ? "+both" : "");
  return s;
"""


def test_dkdv_plan_of_packed_batches(tmp_path):
    # the faster plan by measurement (backwards at tau = 1e-3); unless stated, another kernel
    # or the other choice of parts took 5-40% longer
    one_long, rest = [8192] + [64] * 23, [8192, 1000, 1000, 1000]
    want = [
        # the longest sequence's workgroups fall to a share of the chip: pairs' work and the
        # parts' sums make it worse
        (_packed(one_long, 2, 2, 64, 1e-3), "blocks"), (_packed(one_long, 4, 1, 128, 1e-3), "blocks"),
        (_packed([16384, 64, 64, 64], 8, 1, 64, 1e-3), "blocks"),
        (_packed(rest, 2, 2, 128, 1e-3), "blocks"), (_packed(rest, 8, 2, 128, 1e-3), "blocks"),
        # equal sequences fill the chip whole
        (_packed([8192] * 2, 16, 4, 128, 1e-3), "blocks"), (_packed([16384] * 2, 8, 2, 128, 1e-3), "blocks"),
        (_packed([9000] * 7, 8, 1, 128, 1e-3), "blocks"), (_packed([6000] * 5, 16, 2, 128, 1e-3), "blocks"),
        (_packed([8192, 100], 32, 8, 128, 1e-3), "blocks"),
        (_packed([6000, 3000, 1500, 700, 350], 32, 8, 64, 1e-3), "blocks"),
        (_packed([130] * 16, 32, 8, 64, 1e-3), "blocks"),    # a tie
        # few blocks: parts, or pairs
        (_packed([8192, 4096, 2048, 1024, 512], 8, 2, 128, 1e-3), "blocks+parts"),
        (_packed([6000, 3000, 1500, 700, 350], 16, 4, 128, 1e-3), "blocks+parts"),
        (_packed([16384, 8192, 4096, 1500, 1024, 1000, 500, 68, 4], 4, 1, 128, 1e-3), "blocks+parts"),
        (_packed([9000] * 5, 8, 1, 128, 1e-3), "blocks+parts"),
        (_packed([8192, 4096, 2048, 1024, 512], 4, 1, 128, 1e-3), "pairs"),
        (_packed([6000, 3000, 1500, 700, 350], 4, 1, 128, 1e-3), "pairs+parts"),
        (_packed([3000] + [700] * 9, 2, 2, 64, 1e-3), "pairs"),
        # by sequence: the sparse ones in parts, the others by the same rule as above
        (_packed([16384, 8192, 4096, 1500, 1024, 1000, 500, 68, 4], 8, 2, 128, 1.0), "sequence+parts"),
        (_packed([6000, 3000, 1500, 700, 350], 16, 4, 128, 1.0), "sequence+parts+both"),
        (_packed([16384] * 4, 32, 8, 128, 1.0), "sequence"),
        (_packed([8192, 100], 4, 1, 128, 1.0), "pairs+parts")]
    got = _ask(tmp_path, PACKED, [x for x, _ in want])
    assert got == [a for _, a in want]


ROWS = """  static char s[8];
  std::snprintf(s, sizeof(s), "%d%d", fwd_takes_rows(p, D), dq_takes_rows(p, D));
  return s;
"""


def test_kernels_of_few_row_blocks(tmp_path):
    # forward and dQ pass by 32 rows per workgroup ("1") or 256 ("0"), by measurement; unless
    # stated, the other kernel took 3-150% longer
    fixed = lambda *x: _fixed(x[0], x[1], x[1], *x[2:])
    packed = lambda lens, H, *x: _packed(lens, H, H, *x)
    want = [
        (fixed(1, 32, 256, 256, 128, 1e-3), "11"), (fixed(1, 32, 512, 512, 128, 1e-3), "11"),
        (fixed(1, 32, 2048, 2048, 128, 1e-3), "00"), (fixed(1, 8, 2048, 2048, 128, 1e-3), "11"),
        (fixed(1, 8, 4096, 4096, 128, 1e-3), "11"), (fixed(1, 8, 8192, 8192, 128, 1e-3), "00"),
        (fixed(1, 8, 512, 16384, 128, 1e-3), "11"), (fixed(1, 8, 64, 64, 128, 1e-3), "01"),
        (fixed(1, 1, 1024, 1024, 64, 1e-3), "11"), (fixed(1, 8, 2048, 2048, 128, 1.0), "11"),
        # more row blocks than one round of the chip, of few steps
        (fixed(4, 16, 134, 134, 64, 1.0), "00"),    # dQ pass: a tie
        (fixed(12, 2, 1172, 1172, 64, 1e-3), "01"),
        (fixed(6, 4, 1135, 1376, 128, 1.0), "00"), (fixed(3, 8, 771, 13015, 128, 1.0), "00"),
        (fixed(2, 4, 3177, 10541, 64, 1.0), "01"),
        # the longest sequence's workgroups fall to a share of the chip
        (packed([38, 139, 389, 4298], 4, 64, 1e-3), "00"),
        # sequences of few rows in a grid that the longest one sizes
        (packed([300, 1, 64, 513, 37], 4, 128, 1e-3), "11"), (packed([1000, 7, 256], 2, 64, 1.0), "11"),
        (packed([56, 24, 3052], 8, 64, 1e-3), "11"),
        # (dQ pass: 4% behind the other kernel)
        (packed([21, 55, 31, 19, 164, 85, 133, 72, 491, 1610], 8, 128, 1e-3), "01")]
    got = _ask(tmp_path, ROWS, [x for x, _ in want])
    assert got == [a for _, a in want]
