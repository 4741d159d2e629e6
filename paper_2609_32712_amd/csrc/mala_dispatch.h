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

// Whether a call's time is the chain of one row block's key tiles and not the chip's
// throughput, so that the kernels of one workgroup per 32 query rows (the forward's and
// the dQ pass's) are ahead of those of 256 rows.  In units of one step of the former (four
// key tiles, ~1.1 us) its row blocks take the mean of (stages + 3) each over the CUs; the
// chain of the latter takes `chain` such units per stage of the longest block.  Packed
// batches hold at most total / 32 + sequences row blocks, taken as long as the longest.
constexpr int kRowsTiles = 4;   // key tiles per stage of those kernels
template <class P>
inline bool few_row_blocks(const P& p, int chain) {
  const long stage = kRowsTiles * kBk;
  const long longest = (p.max_len_k + stage - 1) / stage;
  const long grid = (long)((p.max_len + kBq - 1) / kBq) * p.B * p.Hq;
  long blocks = grid;
  if (p.cu && (long)p.Hq * (p.Nq / kBq + p.B) < grid) blocks = (long)p.Hq * (p.Nq / kBq + p.B);
  if (grid > 16 * kNumCus) return false;
  if (blocks <= kNumCus) return true;
  const long shortest = (p.max_len_k - p.max_len) / stage + 1;
  const long mean2 = p.cu ? 2 * longest : shortest + longest;   // twice the mean
  return blocks * (mean2 + 6) <= 2l * chain * kNumCus * longest;
}

}  // namespace mala
