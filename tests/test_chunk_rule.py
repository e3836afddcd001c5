"""The rule that splits full tiles over workgroups (csrc/pmp_chunks.h), compiled
for the host.  No GPU needed."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <random>
#include <vector>
#include "pmp_chunks.h"

// Slots claimed by the split tiles of one deposit, in chunks of at most cc / cs
// entries (1 << 24: on account of the shares alone).
static long long claimed(const std::vector<long long>& c, const std::vector<long long>& s, int cu,
                         int cc, int cs) {
  long long nct = 0, nst = 0, sum = 0;
  for (long long v : c) nct += v;
  for (long long v : s) nst += v;
  for (size_t t = 0; t < c.size(); ++t) {
    const int k = pmp::tile_chunks(c[t], s[t], cc, cs, nct, nst, pmp::kSharesPerCu * cu);
    if (k < 1 || (long long)k < (c[t] + cc - 1) / cc || (long long)k < (s[t] + cs - 1) / cs)
      return -1;  // chunks longer than asked for
    if (k > 1) sum += k;
  }
  return sum;
}

int main() {
  std::mt19937_64 rng(5);
  const int cu = 256;
  long long worst = 0;
  auto look = [&](const std::vector<long long>& c, const std::vector<long long>& s) {
    const long long k = claimed(c, s, cu, 1 << 24, 1 << 24);
    if (k < 0) { std::puts("chunks too long"); std::exit(1); }
    if (k > worst) worst = k;
    if (claimed(c, s, cu, 64, 16) < 0) { std::puts("chunks too long"); std::exit(1); }
  };
  // 400 tiles with a little more than a share of each kind, and one heavy tile
  std::vector<long long> c(4000, 0), s(4000, 0);
  for (int t = 0; t < 400; ++t) { c[t] = 3200; s[1000 + t] = 250; }
  c[3999] = 200000;
  look(c, s);
  for (int q = 0; q < 400; ++q) {
    const int nt = 1 + (int)(rng() % 6000), full = 1 + (int)(rng() % nt);
    const long long mc = 1 + (long long)(rng() % 20000), ms = 1 + (long long)(rng() % 2000);
    std::vector<long long> a(nt, 0), b(nt, 0);
    for (int t = 0; t < full; ++t) {
      a[rng() % nt] += mc + (long long)(rng() % (mc / 8 + 1));
      b[rng() % nt] += ms + (long long)(rng() % (ms / 8 + 1));
    }
    look(a, b);
  }
  std::printf("%lld %d\n", worst, pmp::kSlotsPerCu * cu);
  return worst <= pmp::kSlotsPerCu * cu ? 0 : 2;
}
"""


def test_shares_never_claim_more_slots_than_there_are(tmp_path):
    """Whatever the tiles hold, the chunks claimed on account of a workgroup's
    share fit the slots, so no order of claims leaves a heavy tile without."""
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-include", "cstdlib", "-I",
                    os.path.join(ROOT, "paper_2509_18261_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
