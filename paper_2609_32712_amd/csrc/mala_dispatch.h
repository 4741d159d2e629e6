// Host-side rules of the launches: which kernel a call takes and how its sweeps are split.
// Plain C++ on the sizes of a call (P: FwdParams, BwdParams, or a test's stand-in for them).
#pragma once
#include <algorithm>
#include <cmath>
#include <numeric>

namespace mala {

// Decision geometry (shared by forward and backward so that the backward
// support nests inside the forward support; decode uses 1 x kDecBk).
constexpr int kBq = 32;      // query rows per decision tile = rows of one wavefront
constexpr int kBk = 32;      // keys per decision tile
constexpr int kBwdKeys = 128;                // keys per block of the dK/dV pass (4 key groups x kBk)
constexpr int kNumCus = 256;                 // compute units of an MI355X
// Below kDkdvSplitGroups key-block workgroups (batch x KV heads x key blocks) the
// dK/dV sweeps are split into parts of at least kDkdvPartMin iterations, run by
// workgroups of their own, and summed by a reduction pass.
constexpr int kDkdvSplitGroups = 1024;
constexpr int kDkdvPartMin = 512;
constexpr float kSparseLog2Tau = -3.33f;     // log2 of 0.1: tolerances that may skip many tiles

// Iterations of the dK/dV sweep of the key block starting at key kb0 of a sequence
// (Nq query rows, the last aligned with the last of Nk keys): every (query tile, head
// of the GQA group) from the last query tile down to the block's diagonal.
constexpr int dkdv_iterations(int Nq, int Nk, int kb0, int grp) {
  const long first_q = (long)kb0 - ((long)Nk - Nq);
  const int qi_start = first_q <= 0 ? 0 : (int)(first_q / kBq);
  return grp * ((Nq + kBq - 1) / kBq - qi_start);
}

// Parts of the dK/dV sweeps (fixed-length batches): one per sweep when the key
// blocks alone give kDkdvSplitGroups workgroups; otherwise parts of the smallest
// power of two >= kDkdvPartMin iterations that gives at most ~kDkdvSplitGroups
// parts over all sweeps, so that a long sweep (the first key blocks', or one that
// retains every tile) no longer sets the kernel's time alone.
inline void dkdv_split(int B, int Hq, int Hkv, int Nq, int Nk, int* psize, int* nparts) {
  const int grp = Hq / Hkv, nkblk = (Nk + kBwdKeys - 1) / kBwdKeys;
  *psize = 1 << 30;
  *nparts = 1;
  if ((long)nkblk * B * Hkv >= kDkdvSplitGroups) return;
  long total = 0;
  for (int j = 0; j < nkblk; ++j) total += dkdv_iterations(Nq, Nk, j * kBwdKeys, grp);
  total *= (long)B * Hkv;
  const int longest = dkdv_iterations(Nq, Nk, 0, grp);
  long ps = kDkdvPartMin;
  while (ps * 2 * kDkdvSplitGroups <= total) ps *= 2;
  if (ps >= longest) return;
  *psize = (int)ps;
  *nparts = (int)((longest + ps - 1) / ps);
}
// Packed batches, whose lengths only the device knows: the same rule on what the host
// knows, blocks of the total and sweeps up to the longest sequence's, half of it long on
// average.  A sequence of at most psize iterations stays in one part.
inline void dkdv_split_packed(int num_seqs, int max_q, int total_k, int Hq, int Hkv, int* psize,
                              int* nparts) {
  const long blocks = (long)Hkv * (total_k / kBwdKeys + num_seqs);
  const long longest = (long)(Hq / Hkv) * ((max_q + kBq - 1) / kBq);
  *psize = 1 << 30;
  *nparts = 1;
  if (blocks >= kDkdvSplitGroups) return;
  long ps = kDkdvPartMin;
  while (ps * 4 * kDkdvSplitGroups <= blocks * longest) ps *= 2;
  if (ps >= longest) return;
  *psize = (int)ps;
  *nparts = (int)((longest + ps - 1) / ps);
}

// Time (us) of a dK/dV pass over n sweeps of `total` iterations in all, the longest of
// `longest`: the pairs kernel takes ~0.5 us per iteration and tile of 32 keys, four items per
// 128 keys, the blocks kernel ~1.14 us, each some iterations more per item, and a CU holds
// one item at a time.  It is the longest sweep's chain where CUs are idle, else the chip's
// share of all of them, in whole rounds where the sweeps are few and alike.
inline double dkdv_time(bool pairs, double n, double total, double longest) {
  const double items = pairs ? 4 * n : n, us = pairs ? 0.5 : 1.14, more = pairs ? 6 : 8;
  const double chain = (longest + more) * us;
  double t = std::max(chain, items / kNumCus * (total / n + more) * us);
  if (total >= 0.7 * n * longest && items < 3 * kNumCus)
    t = std::max(t, std::ceil(items / kNumCus) * chain);
  return t;
}

// The dK/dV kernels of a call: pairs (all sweeps), blocks (all sweeps), or each sequence by
// the tiles that the dQ pass retained.
enum class DkdvRule { kPairs, kBlocks, kBySequence };
struct DkdvPlan {
  DkdvRule rule;
  bool parts;          // the sweeps run in the call's parts (else whole),
  bool block_parts;    // those of the blocks kernel too, where both kernels run
};
constexpr long kPairsGridMax = 16384;        // 128-key sweeps, four workgroups each
constexpr long kPairsSweeps = 272;           // ~4 items of pairs per CU

// Packed batches: only the device knows the lengths.  Taken as the worst of two batches
// that the host cannot tell from others, sequences all as long as the longest, and the
// longest alone with the rest of no length: workgroups go round the XCDs, and round their
// shader engines, in turn, so that a sequence's have only a share of the chip (`reach`) where
// the sequences' number has factors of two (one of 8192 tokens among 23 of 64, 2 heads, D =
// 64: 48 slices, 1 / 8 of the chip; backward by blocks / pairs 857 / 1219 us).  Parts help
// where neither batch fills the chip without them (8192 + 4096 + 2048 + 1024 + 512 tokens, 8/2
// heads, D = 128: whole 1389 us, parts 1020) and cost the partial sums where one does (2 x 8192,
// 16/4 heads: 2083 / 2194).  Where the sequences go by their decisions, the pairs' sweeps,
// most of all an attention sink's, are uneven, and run in parts in any case (a sequence of
// 16384 among eight shorter ones, 8/2 heads, language-model-like: 1591 / 1221).
template <class P>
inline DkdvPlan dkdv_plan_packed(const P& p, int D) {
  const int grp = p.Hq / p.Hkv, slices = p.B * p.Hkv;
  const double grid = (double)p.nkblk * slices, longest = (double)grp * ((p.max_len + kBq - 1) / kBq);
  if (grid > kPairsGridMax) return {DkdvRule::kBlocks, false, false};   // mostly empty workgroups
  const double n = std::min(grid, (double)p.Hkv * (p.Nk / kBwdKeys + p.B));
  const double reach = std::min(1.0, (double)p.Hkv / std::gcd(slices, 32));
  const double sweeps = std::max(n, p.Hkv * p.nkblk / reach), total = sweeps * longest / 2;
  const double empty = (grid - n) / kNumCus * 1.2;                      // us, per workgroup and sweep
  const bool may_skip = p.log2tau >= kSparseLog2Tau;
  const double half = may_skip && D == 128 && longest < 512 ? 0.5 : 1.0;   // as for fixed lengths
  double best = dkdv_time(false, sweeps, total, longest) + empty;
  double pairs = dkdv_time(true, sweeps, half * total, half * longest) + 4 * empty;
  bool pair_parts = false, block_parts = false;
  const bool can_split = p.nparts > 1 && grid * p.nparts <= kPairsGridMax;
  if (can_split) {
    const double parts = total / p.psize + sweeps / 2, more = (p.nparts - 1) * grid / kNumCus * 1.2;
    const double pp = 1.05 * dkdv_time(true, parts, total, p.psize) + 4 * (empty + more);
    const double bp = 1.05 * dkdv_time(false, parts, total, p.psize) + empty + more + 20;
    pair_parts = may_skip || pp < pairs;
    pairs = std::min(pairs, pp);
    block_parts = bp < 0.9 * best;
    if (block_parts) best = bp;
  }
  if (pairs < 0.9 * best) return {DkdvRule::kPairs, pair_parts, false};
  if (may_skip && longest >= 512) return {DkdvRule::kBySequence, can_split, block_parts};
  return {DkdvRule::kBlocks, block_parts, block_parts};
}

// The kernel of the sweeps where every tile is retained is the one that dkdv_time finds ahead
// (us per backward, blocks / pairs, tau = 1e-3, D = 128 unless stated; n sweeps: 8 heads GQA
// 4:1, n = 16 (1024 tokens) 211 / 117, n = 64 (4096 tokens) 729 / 395, n = 256 (4 x 4096) 779 /
// 715; 16 x 2048, 16 heads, n = 256, 156 / 152; 32 heads x 1024, n = 256, 103 / 105; against
// more keys than queries, whose sweeps are alike: 512 rows x 4096 keys, 32/8 heads, n = 256,
// 181 / 227; 2 x 2048 x 8192, 8/2 heads, n = 256, 571 / 750; 256 x 2048, 32/8 heads, n = 128,
// 76 / 70; 8192 tokens, 8/1 heads, 160 parts, 903 / 985).  With n = 512 blocks are always
// ahead (463 / 564).
//
// Sequences that skip are the pairs' in any case (tau = 1, language-model-like, D = 128: 32
// heads x 1024 87 / 75, 512 x 4096 rows 188 / 144), but a tolerance below 0.1 does not promise
// that they do.  mala_bwd_choose_kernel marks them, both kernels are launched and each skips
// the other's sequences, for 5-20 us in all where none is sparse (a backward of 8 x 4096
// tokens, GQA 8/2: D = 128 838 / 848, D = 64 843 / 848; 16384 tokens, D = 64: 2062 / 2054).
// Language-model-like tokens at tau = 1, D = 128: 8 x 4096 850 / 530, 32768 4478 / 3168, 2 x
// 2048 x 8192 516 / 351.
template <class P>
inline DkdvPlan dkdv_plan(const P& p, int D) {
  if (p.cu) return dkdv_plan_packed(p, D);
  const bool parts = p.nparts > 1;
  if ((long)p.nkblk * p.B * p.Hkv * p.nparts > kPairsGridMax) return {DkdvRule::kBlocks, parts, parts};
  const int grp = p.Hq / p.Hkv;
  const long longest = std::min<long>(p.psize, (long)grp * ((p.max_len + kBq - 1) / kBq));
  const bool may_skip = p.log2tau >= kSparseLog2Tau;
  const long least = D == 128 ? 256 : 512;   // iterations that pay for the ~20 us of the choice
  long n = 0, total = 0;
  for (int j = 0; j < p.nkblk; ++j) {
    const int its = dkdv_iterations(p.Nq, p.Nk, j * kBwdKeys, grp);
    total += its;
    n += (its + (long)p.psize - 1) / p.psize;
  }
  n *= (long)p.B * p.Hkv;
  total *= (long)p.B * p.Hkv;
  // sweeps too short for the choice by sequence: at D = 128 half of the tiles (94% of the
  // blocks' iterations) is as many as any of the workloads' inputs retains
  const double half = may_skip && D == 128 && longest < least ? 0.5 : 1.0, some = half < 1.0 ? 0.94 : 1.0;
  if (n <= kPairsSweeps && dkdv_time(true, n, half * total, half * longest) <=
                               dkdv_time(false, n, some * total, some * longest))
    return {DkdvRule::kPairs, parts, false};
  return {may_skip && longest >= (n <= kPairsSweeps ? least : 512) ? DkdvRule::kBySequence
                                                                   : DkdvRule::kBlocks, parts, parts};
}

// Longest time (in the lengths' unit) that one of `cus` CUs is busy with n workgroups whose
// lengths fall evenly from longest to shortest, the longest first, one on a CU at a time: the
// mean share, or r rounds of which the last begins with the length of workgroup (r - 1) cus.
inline double launch_span(double n, double shortest, double longest, double cus) {
  const double mean = n * (shortest + longest) / 2 / cus;
  double t = longest;
  for (int r = 2; (r - 1) * cus < n; ++r) {
    const double x = r * (longest - (longest - shortest) * (r - 1) * cus / n);
    if (x <= t) break;   // rises, then falls with r
    t = x;
  }
  return std::max(mean, t);
}

// Whether the kernels of one workgroup per 32 query rows (the forward's and the dQ pass's,
// steps of four key tiles, ~3 more to fill and drain the pipeline) are ahead of those of 256
// rows, whose chain goes tile by tile: by the span of either's workgroups over the CUs.
// The times are fits (us: a step, a tile, what the latter kernel takes longer to start) over
// 1600 calls of 1 to 128 heads x sequences, 96 to 4096 rows, up to 17000 keys; a tile takes
// longer on inputs with many low terms (D = 128: 0.8-1.5 us), and the rates are near the
// lower end, so that the choice rarely costs time.
//
// Packed batches, whose lengths only the device knows: ahead in both of the batches that the
// host cannot tell from others, sequences all as long as the longest, and the longest alone
// with the rest of no length, which has only the CUs that its (sequence, head) slices reach
// (as for dkdv_plan_packed).  Workgroups without rows cost ~1 us of a CU each.
constexpr int kRowsTiles = 4;   // key tiles per step of those kernels
struct RowsRates {
  double first, step, tile;
};
template <class P>
inline bool rows_ahead(const P& p, const RowsRates& c) {
  const long stage = kRowsTiles * kBk, older = p.max_len_k - p.max_len;   // keys every row sees
  const double longest = (double)((p.max_len_k + stage - 1) / stage), shortest = (double)(older / stage + 1);
  const double tiles = (double)((p.max_len_k + kBk - 1) / kBk);
  const double first_block = (double)((older + std::min(255, p.max_len - 1)) / kBk + 1);
  const long r32 = (p.max_len + kBq - 1) / kBq, r256 = (p.max_len + 255) / 256;   // of a sequence
  const long slices = (long)p.B * p.Hq, grid = r32 * slices;
  if (grid > 16 * kNumCus) return false;
  const auto ahead = [&](long n32, long n256, double cus) {
    return c.step * launch_span(n32, shortest + 3, longest + 3, cus) + (double)(grid - n32) / kNumCus <=
           c.first + c.tile * launch_span(n256, first_block, tiles, cus);
  };
  if (!p.cu) return ahead(grid, r256 * slices, kNumCus);
  const double reach = std::min(1.0, (double)p.Hq / std::gcd(slices, 32l));
  return ahead(std::min(grid, (long)p.Hq * (p.Nq / kBq + p.B)),
               std::min(r256 * slices, (long)p.Hq * (p.Nq / 256 + p.B)), kNumCus) &&
         ahead(r32 * p.Hq, r256 * p.Hq, kNumCus * reach);
}

// Measured (us, kernel of 256 rows / of 32; tau = 1e-3, D = 128 unless stated): 32 heads x 256
// 17.8 / 10.7, x 512 28.1 / 20.5, x 1024 47.8 / 49.3, x 2048 85 / 129; 8 heads x 2048 76.8 /
// 37.4, x 4096 136 / 106, 512 x 8192 245 / 81; D = 64, 12 x 2 heads x 1172 42.7 / 45.9, 4 x 16
// heads x 134 7.9 / 11.2, packed 4298 + 389 + 139 + 38 tokens, 4 heads 126 / 205.  One step
// (up to 128 keys) stays with the other kernel (64 x 64: 6.4 / 8.6).  The counters of V tiles
// are defined by groups of 256 rows, so calls with counters stay there too.
template <class P>
inline bool fwd_takes_rows(const P& p, int D) {
  return !p.counters && p.max_len_k > kRowsTiles * kBk &&
         rows_ahead(p, D == 128 ? RowsRates{2.4, 1.32, 0.91} : RowsRates{2.4, 1.24, 0.79});
}

// Measured (us per backward, kernel of 256 rows / of 32, D = 128 GQA 8/2 unless stated): 128
// tokens 28.7 / 25.8, 1024 119 / 84, 4096 396 / 349, 8192 833 / 875; MHA 8 heads 2048 138 / 87,
// 32 heads 2048 238 / 298; D = 64, packed 4298 + 389 + 139 + 38 tokens, 4/2 heads 426 / 469.
// From tau = 0.1 on the other kernel may skip for less (language-model-like at tau = 1: 2048
// tokens 177 / 157, 4096 331 / 339).
template <class P>
inline bool dq_takes_rows(const P& p, int D) {
  const bool may_skip = p.log2tau >= kSparseLog2Tau;
  if (D == 128) return rows_ahead(p, may_skip ? RowsRates{6.0, 1.41, 0.70} : RowsRates{4.0, 1.41, 1.13});
  return rows_ahead(p, may_skip ? RowsRates{3.0, 1.02, 0.85} : RowsRates{3.0, 1.06, 0.95});
}

}  // namespace mala
