// Rule that splits a full tile's entries over several workgroups.  Plain C++:
// the host tests compile it too (constexpr functions run on the device as well).
#pragma once

namespace pmp {

// Workgroups per compute unit a deposit's entries are shared over, and chunk
// slots per compute unit.
constexpr int kSharesPerCu = 2, kSlotsPerCu = 4;
constexpr int kChunkMinCic = 1024, kChunkMinSn = 128, kChunksMost = 32;

// Chunks a tile's nc CIC and ns supernova entries are split into: at most cc
// CIC and cs supernova entries per chunk; and one for each whole workgroup's
// share of the deposit's nct and nst entries it holds (total / share, but at
// least kChunkMin entries; up to kChunksMost chunks on that account), so that a
// cluster's core, which may hold a fifth of all particles in one tile, is
// spread over the chip.  Whole shares: the tiles of a deposit hold at most
// `share` of each kind, so the chunks claimed on account of shares fit the
// 2 share = kSlotsPerCu num_cu slots whatever the tiles' order; counting begun
// shares too, moderately full tiles could claim them all before the heaviest
// tile (256^3 FP64, 400 tiles of 3200 CIC particles, 400 of 250 supernovae and
// one of 200000 particles: 257 us in some runs, 212 in others; now 210).
// 1e6 Plummer particles at 256^3 FP64 on 16 x 8 x 8 tiles with cc = 16384: the
// step with 256 sinks takes 270 us with whole chunks of cc behind device-scope
// fences, 230 us without the fences (see the partial sums in the tile pass),
// 202 us with the share; shares of one, two or four workgroups per compute
// unit differ by 3%.
constexpr int tile_chunks(long long nc, long long ns, int cc, int cs, long long nct,
                          long long nst, int share) {
  if (share <= 0) return 1;  // never split
  const long long ec = nct / share > kChunkMinCic ? nct / share : kChunkMinCic;
  const long long es = nst / share > kChunkMinSn ? nst / share : kChunkMinSn;
  const long long want_c = nc / ec, want_s = ns / es;
  const long long need_c = (nc + cc - 1) / cc, need_s = (ns + cs - 1) / cs;
  long long n = want_c > want_s ? want_c : want_s;
  if (n > kChunksMost) n = kChunksMost;
  if (need_c > n) n = need_c;
  if (need_s > n) n = need_s;
  return n > 1 ? (int)n : 1;
}

}  // namespace pmp
