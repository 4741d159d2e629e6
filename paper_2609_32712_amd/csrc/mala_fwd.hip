// MALA forward (Algorithm 1) for gfx950.
//
// One workgroup = 8 wavefronts = 256 consecutive query rows of one (batch, query
// head); each wavefront owns 32 rows, which is the decision tile's B_q.  K and V
// are staged through double-buffered LDS 64 keys at a time, from the workgroup's
// highest legal key down to key 0 (the diagonal-first traversal of the Online
// Sparse Softmax paragraph); the next stage moves straight into LDS (buffer loads
// with the LDS flag) while the current one is processed.  Inside a stage each
// wavefront visits its two 32-key decision tiles high half first, so every
// wavefront sees its tiles in strictly descending order.
//
// Per decision tile (32 keys x the wavefront's 32 rows):
//   S^T = K_j Q_i^T       8 (D = 128) bf16 MFMAs 32x32x16, fp32 accumulate; each
//                         lane holds one query row and 16 of the 32 keys, so the
//                         row max is 15 in-lane max + one permlane32 swap;
//   online test           skip iff every row with a legal key has
//                         rowmax - m - log2(l) < log2(tau) - log2(L_q) (base-2 units,
//                         equivalent to the natural-log test), rows with l == 0
//                         always retain; one ballot makes the branch wave-uniform;
//   retained path         lazy rescale of O and l (only when some row's max grew by
//                         more than 2^8), P = exp2(S - m) as a bf16 hi term, plus a
//                         lo term when the tile holds more than kFwdLoShare of some
//                         row's normalizer, O^T += V^T P^T (8 MFMAs per term, V^T
//                         operand through ds_read_b64_tr_b16).
// A skipped tile costs its QK MFMAs, one max reduction and one compare.
#include "mala_device.h"
#include "mala_kernels.h"

namespace mala {

// The two forward kernels below give the same bits: they share the order of every sum,
// and neither leaves the rounding of a row quantity to the compiler: contraction is off
// and fused operations are written out, in the functions here and in both kernels.

// -log2(tau / L_q) of query row q (L_q = q + 1 + off).
__device__ __forceinline__ float row_threshold(float log2tau, int q, long off) {
#pragma clang fp contract(off)
  return log2f((float)(q + 1 + off)) - log2tau;
}
// The online test of a row whose largest raw score in the tile is raw: the tile's
// largest scaled score against log2 of the retained normalizer l (reference m), both sides
// negated: so -m need not be kept in a register, and the 256-row kernel is the instruction
// stream that the compiler made of mt - m - log2(l) >= thr by contraction.
__device__ __forceinline__ bool online_demand(float raw, float scale2, float m, float l, float nthr) {
#pragma clang fp contract(off)
  return (l == 0.f) | (__builtin_fmaf(raw, -scale2, m) + fast_log2(l) <= nthr);
}
// Scores of a tile's key rows ka against the wavefront's query rows, k-steps in order.
template <int KS>
__device__ __forceinline__ f32x16 fwd_scores(const bf16x8 (&ka)[KS], const bf16x8 (&qreg)[KS]) {
  f32x16 s;
#pragma unroll
  for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) s = mfma32(ka[kk], qreg[kk], s);
  return s;
}
// Raw scores of a lane (masked keys -inf) and their maximum over the lane's 16 keys;
// keys 8 (r / 4) + r % 4 > lim are masked (lane offset 4 h taken off lim by the caller).
__device__ __forceinline__ float masked_max(const f32x16& s, bool need_mask, int lim, float (&sv)[16]) {
  float mt = kNegInf;
  if (need_mask) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float x = (8 * (r >> 2) + (r & 3) <= lim) ? s[r] : kNegInf;
      sv[r] = x;
      mt = fmaxf(mt, x);
    }
  } else {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      sv[r] = s[r];
      mt = fmaxf(mt, sv[r]);
    }
  }
  return mt;
}
// P = exp2(s scale2 - m) in place with one rounding of the argument, and the row's sum
// as a tree (over both halves of the column).  A row with no legal key so far keeps
// m = -inf: shift by 0 so that exp2(-inf) = 0.
__device__ __forceinline__ float fwd_probabilities(float (&sv)[16], float scale2, float m) {
#pragma clang fp contract(off)
  const float shift = (m == kNegInf) ? 0.f : m;
#pragma unroll
  for (int r = 0; r < 16; ++r) sv[r] = fast_exp2(__builtin_fmaf(sv[r], scale2, -shift));
  float ps4[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) ps4[g] = (sv[4 * g] + sv[4 * g + 1]) + (sv[4 * g + 2] + sv[4 * g + 3]);
  return halves_sum((ps4[0] + ps4[1]) + (ps4[2] + ps4[3]));
}
// Lazy rescaling: the factor that takes a row from reference m to m_new.
__device__ __forceinline__ float rescale(float m, float m_new) {
  return (m_new == kNegInf) ? 1.f : fast_exp2(m - m_new);
}

template <int D>
__global__ __launch_bounds__(kFwdWaves * 64) void mala_fwd_kernel(FwdParams p) {
#pragma clang fp contract(off)
  constexpr int NT = kFwdWaves * 64;     // threads per workgroup
  constexpr int KS = D / 16;             // k-steps of the QK product
  constexpr int DB = D / 32;             // 32-wide output column blocks
  constexpr int STAGE = tile_elems<D>(kFwdStage);
  // double-buffered K and V stages: the next stage is fetched while the current one
  // is processed
  __shared__ __attribute__((aligned(16))) bf16 Ks[2 * STAGE];
  __shared__ __attribute__((aligned(16))) bf16 Vs[2 * STAGE];
  // statistics: per stage buffer and decision tile, t + 1 once some wavefront
  // retained the tile of stage t (stage-tagged: no clearing between stages); the
  // workgroup's counter sums
  __shared__ int vneed[2][kFwdStage / kBk];
  __shared__ unsigned long long bcnt[kNumCounters];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, c = lane & 31, G = lane >> 4, t16 = lane & 15;
  // lane bases of the LDS tile reads: operand rows (row c) and transposed rows
  const int rdo = rd_base<D>(c, h), tro = tr_base<D>(4 * h + (t16 >> 2), G & 1, t16);
  const int BH = p.B * p.Hq;
  const int bh = blockIdx.x % BH;
  const int qblk = p.nqblk - 1 - (int)(blockIdx.x / BH);   // longest rows first
  const int b = bh / p.Hq, hq = bh % p.Hq, hkv = hq / (p.Hq / p.Hkv);
  const Seg sg = seq_slice(p, b);
  const int Nq = sg.Nq, Nk = sg.Nk;
  if (qblk * kFwdRows >= Nq) return;   // past the end of a packed sequence
  const long off = (long)Nk - Nq;
  const int offi = Nk - Nq;   // off as an int (|off| < 2^31)
  const int q0w = qblk * kFwdRows + wave * kBq;
  const int qrow = q0w + c;
  const bool row_valid = qrow < Nq;

  const long qbase = sg.qb + (long)hq * p.Nq;    // row 0 of this (sequence, head)
  const long kbase = sg.kb + (long)hkv * p.Nk;
  const bf16* Qp = p.q + qbase * D;
  const bf16* Kp = p.k + kbase * D;
  const bf16* Vp = p.v + kbase * D;

  // Q^T as the B operand: lane (h, c) holds Q[qrow][16kk + 8h .. +7]
  bf16x8 qreg[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
    qreg[kk] = row_valid ? load8(Qp + (long)qrow * D + 16 * kk + 8 * h) : zero8();

  float m = kNegInf, l = 0.f;
  f32x16 acc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
  int cnt = 0;          // retained diagonal tiles in which this row has a legal key
  unsigned n_ret_m = 0;  // retained diagonal tiles
  const float nthr = row_threshold(p.log2tau, qrow, off);   // -log2(tau / L_q)

  const int qlast_w = min(q0w + kBq - 1, Nq - 1);
  const int jdiag = (q0w < Nq) ? (int)((qlast_w + off) / kBk) : -1;
  const int nvalid = max(0, min(kBq, Nq - q0w));
  const int qlast_g = min(qblk * kFwdRows + kFwdRows - 1, Nq - 1);
  const int ttop = (int)((qlast_g + off) / kFwdStage);
  unsigned n_legal = 0, n_ret = 0, n_vneed = 0;
  unsigned long long hsum = 0;   // fingerprints of the retained tiles
  const bool stats = p.counters != nullptr;
  if (stats) {
    if (tid < 2 * (kFwdStage / kBk)) vneed[tid / (kFwdStage / kBk)][tid % (kFwdStage / kBk)] = 0;
    blk_init(bcnt);
  }

  // K / V stages move with buffer loads straight into LDS (keys past the end read
  // as zeros): wavefront w issues the 64-position loads w, w + 8, ... of each slot.
  // The loads of stage t - 1 overlap the compute of stage t and are waited for just
  // before the stage's closing barrier.
  constexpr int NIS = STAGE / 512;           // 64-position loads per stage slot
  static_assert(NIS * 512 == STAGE, "whole loads per slot");
  constexpr int NJS = (NIS + kFwdWaves - 1) / kFwdWaves;
  uint32_t dma_off[NJS];
#pragma unroll
  for (int u = 0; u < NJS; ++u) dma_off[u] = dma_lane_offset<D>(64 * (wave + kFwdWaves * u) + lane);
  auto fetch = [&](int t, int buf) {
    const long k0 = (long)t * kFwdStage;
    const uint32_t nb = (uint32_t)(Nk - k0) * (uint32_t)D * 2u;
    const i32x4 rk = rsrc_words(Kp + k0 * D, nb), rvv = rsrc_words(Vp + k0 * D, nb);
#pragma unroll
    for (int u = 0; u < NJS; ++u) {
      const int j = wave + kFwdWaves * u;
      if (j < NIS) {
        buf_load_lds16(rk, dma_off[u], Ks + buf * STAGE + 512 * j);
        buf_load_lds16(rvv, dma_off[u], Vs + buf * STAGE + 512 * j);
      }
    }
  };

  fetch(ttop, 0);
  wait_vm();   // (also the Q loads above, so that no wait for them lands in the loop)
  __syncthreads();

  for (int t = ttop; t >= 0; --t) {
    const int buf = (ttop - t) & 1;
    if (t > 0) fetch(t - 1, buf ^ 1);
    const bf16* kr = lds_pin(Ks + buf * STAGE + rdo);
    const bf16* vtb = lds_pin(Vs + buf * STAGE + tro);

    // statistics: the tag each retained tile of this stage found in vneed (t + 1:
    // another wavefront marked it first); compared after the stage, so that the
    // exchange's result is not waited for in the middle of the tile's work
    int vtag[2] = {t + 1, t + 1};
    if (2 * t <= jdiag) {
      // the two tiles in descending key order: the high half first
#pragma unroll
      for (int sub = 1; sub >= 0; --sub) {
        const int j = 2 * t + sub;
        if (j > jdiag) continue;            // above this wavefront's diagonal
        const int kb = j * kBk;
        ++n_legal;
        // score discovery (all K operands are read from LDS first)
        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        {
          bf16x8 ka[KS];
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) ka[kk] = load8(kr + sub * kBk * (D + 8) + rd_step<D>(kk));
#pragma unroll
          for (int kk = 0; kk < KS; ++kk) s = mfma32(ka[kk], qreg[kk], s);
        }

        const bool need_mask = (kb + kBk - 1 > q0w + offi) || (q0w + kBq > Nq);
        float sv[16];
        float mt = kNegInf;
        if (need_mask) {
          // keys of this lane: kb + 8 (r / 4) + 4 h + r % 4; legal iff key <= qrow + off
          const int lim = row_valid ? qrow + offi - kb - 4 * h : -1000000;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float x = (8 * (r >> 2) + (r & 3) <= lim) ? s[r] : kNegInf;
            sv[r] = x;
            mt = fmaxf(mt, x);
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            sv[r] = s[r];
            mt = fmaxf(mt, sv[r]);
          }
        }
        // the row max of the raw scores, then scaled (scale2 > 0 and rounding is
        // monotonic, so this is the max of the scaled scores)
        const float raw = halves_max(mt);
        mt = raw * p.scale2;

        // the online test (rows with no legal key in the tile do not vote); m + log2(l)
        // is log2 of the retained normalizer whichever reference m the row uses
        const bool voter = row_valid & (kb <= qrow + offi);
        const bool demand = voter & online_demand(raw, p.scale2, m, l, nthr);
        if (!wave_any(demand)) continue;    // skipped: m, l and O unchanged
        ++n_ret;
        // off the diagonal every valid row votes: those tiles are counted per wavefront
        if (need_mask) {
          ++n_ret_m;
          cnt += voter ? 1 : 0;
        }
        // O^T[d][q] += V^T[d][key] P^T[key][q]; V^T rows through transposed LDS reads,
        // issued before the softmax work so that their latency hides under it
        bf16x8 va[DB][2];
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            const bf16* vt = vtb + (sub * kBk + 16 * ks) * (D + 8) + tr_step<D>(db);
            va[db][ks] = cat(lds_read_tr(vt), lds_read_tr(vt + 8 * (D + 8)));
          }
        if (stats) {
          hsum += tile_hash(b, hq, q0w / kBq, j);
          // the first wavefront to retain this tile of the stage counts its V tile
          if (lane == 0) vtag[sub] = atomicExch(&vneed[buf][sub], t + 1);
        }

        // Lazy rescaling: a row's reference m moves only when some row of the
        // wavefront would otherwise see P = exp2(s - m) above 2^8; O and l are then
        // rescaled.  The result is the same softmax; P stays in [0, 2^8].
        if (wave_any(mt > m + 8.f)) {
          const float m_new = fmaxf(m, mt);
          const float alpha = (m_new == kNegInf) ? 1.f : fast_exp2(m - m_new);
          l *= alpha;
          m = m_new;
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
        }
        // a row with no legal key so far keeps m = -inf: shift by 0 so exp2(-inf) = 0
        const float shift = (m == kNegInf) ? 0.f : m;
        // P = exp2(s scale2 - shift) with one rounding; the row sum as a tree
#pragma unroll
        for (int r = 0; r < 16; ++r) sv[r] = fast_exp2(__builtin_fmaf(sv[r], p.scale2, -shift));
        float ps4[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) ps4[g] = (sv[4 * g] + sv[4 * g + 1]) + (sv[4 * g + 2] + sv[4 * g + 3]);
        const float ps = halves_sum((ps4[0] + ps4[1]) + (ps4[2] + ps4[3]));
        l += ps;
        // P as two bf16 terms where it matters: the backward's D = rowsum(O * dO)
        // cancels against dP for dominant keys, so their probabilities must be
        // accurate well beyond one bf16 rounding.  A tile whose mass is a small
        // share of every row's retained normalizer (this tile included) runs the
        // high term only.
        const bool need_lo = wave_any(ps > kFwdLoShare * l);
        const bf16x8 ph[2] = {hi_bf16x8(sv), hi_bf16x8(sv + 8)};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int db = 0; db < DB; ++db) acc[db] = mfma32(va[db][ks], ph[ks], acc[db]);
        if (need_lo) {
          const bf16x8 pl[2] = {lo_bf16x8(sv, ph[0]), lo_bf16x8(sv + 8, ph[1])};
#pragma unroll
          for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] = mfma32(va[db][ks], pl[ks], acc[db]);
        }
      }
    }
    wait_vm();
    __syncthreads();
    n_vneed += (vtag[0] != t + 1) + (vtag[1] != t + 1);
  }

  // epilogue: O <- O / l, LSE = (m + log2 l) * ln 2
  if (row_valid) {
    const float inv = 1.f / l;
    const long orow = (qbase + qrow) * D;
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 v4 = {acc[db][4 * g] * inv, acc[db][4 * g + 1] * inv, acc[db][4 * g + 2] * inv,
                    acc[db][4 * g + 3] * inv};
        store_out4(p.o, orow + 32 * db + 8 * g + 4 * h, v4, p.o_bf16);
      }
    if (h == 0) {
      p.lse[qbase + qrow] = (m + fast_log2(l)) * kLn2;
      if (p.row_tiles) p.row_tiles[qbase + qrow] = cnt + (int)(n_ret - n_ret_m);
    }
  }
  if (stats) {
    if (lane == 0) {
      blk_add(bcnt, kCntLegal, n_legal);
      blk_add(bcnt, kCntRetained, n_ret);
      blk_add(bcnt, kCntSlots, (unsigned long long)n_ret * kBk * nvalid);
      blk_add(bcnt, kCntSetHash, hsum);
      blk_add(bcnt, kCntVNeeded, n_vneed);
    }
    if (tid == 0) blk_add(bcnt, kCntVTiles, (unsigned long long)(ttop + 1) * (kFwdStage / kBk));
    blk_flush(bcnt, p.counters);
  }
}

// Forward of small grids: one workgroup of eight wavefronts per 32 query rows, so that a
// call with few rows (a short sequence, a prefill chunk, few heads) still gives the chip
// workgroups to run, and the key tiles of a row block are worked on several at once.
//
// What bounds such calls is the latency of a row block's chain of key tiles (scores,
// test, exponentials, P V, the next tile): ~2100 cycles per tile for a wavefront of the
// kernel above, whether or not another one shares its SIMD.  Only two links of the chain
// are really serial, the test (l grows by the tile's sum) and the accumulation of O;
// both keep their order here, so the results are the same bits.  The tiles go through a
// pipeline of three steps, four tiles (a stage of 128 keys) at a time, one barrier per
// step:
//   * producers (wavefronts 0-3, one tile each), step n: scores of stage n, row maxima to
//     LDS;
//   * producers, step n + 1: from the row maxima, the rows' references m through the
//     stage as if all its tiles were retained; P of the own tile for its reference, as
//     bf16 terms, and its row sums to LDS.  The producers also move K (each its own
//     tile, a stage ahead) and V into LDS;
//   * consumers (wavefronts 4-7), step n + 2: the tests in order, then columns 32 w ..
//     32 w + 31 of O over the retained tiles, in order.  A retained tile whose P has
//     another reference than the row's (a skipped tile was to move it) is formed again
//     by the consumers, who then tell the producers the reference.
// A step takes ~2500 cycles per stage (~630 per tile), bound by the producers: ~1000 for
// scores and P, ~800 to issue the stage's 68 KB of loads, the rest waits.  512 rows x
// 8 heads against 16384 keys: 465 -> 145 us; one head over 1024 rows (D = 128): 43 -> 16
// us.  K straight into operand registers instead of LDS took 1600 cycles of issue per
// step (32-byte pieces of a row per load), a fetch of V by the consumers 1300.
template <int D>
__global__ __launch_bounds__(2 * kRowsTiles * 64) void mala_fwd_rows_kernel(FwdParams p) {
#pragma clang fp contract(off)
  constexpr int W = kRowsTiles, KS = D / 16, DB = D / 32;
  constexpr int STAGE = tile_elems<D>(W * kBk);
  static_assert(DB <= W, "one column block per consumer");
  constexpr int NKL = (tile_elems<D>(kBk) + 511) / 512;   // 64-position loads per K tile
  __shared__ __attribute__((aligned(16))) bf16 Vs[2 * STAGE];
  __shared__ __attribute__((aligned(16))) bf16 Ks[W * NKL * 512];
  __shared__ __attribute__((aligned(16))) bf16x8 Ps[2][W][4][64];  // hi0, hi1, lo0, lo1 of a tile
  __shared__ float redm[3][W][32];                // per tile and row: raw maximum
  __shared__ f32x2 redp[2][W][32];                // per tile and row: sum and reference of P
  // from the consumers, per stage parity and row: l, m and whether the references differed
  __shared__ f32x2 rowlm[2][32];
  __shared__ int resync[2];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, c = lane & 31, G = lane >> 4, t16 = lane & 15;
  const int BH = p.B * p.Hq;
  const int bh = blockIdx.x % BH;
  const int qt = (int)(gridDim.x / BH) - 1 - (int)(blockIdx.x / BH);   // longest rows first
  const int b = bh / p.Hq, hq = bh % p.Hq, hkv = hq / (p.Hq / p.Hkv);
  const Seg sg = seq_slice(p, b);
  const int Nq = sg.Nq, Nk = sg.Nk;
  const int q0w = qt * kBq;
  if (q0w >= Nq) return;   // past the end of a packed sequence
  const int offi = Nk - Nq;
  const int qrow = q0w + c;
  const bool row_valid = qrow < Nq;
  const long qbase = sg.qb + (long)hq * p.Nq;    // row 0 of this (sequence, head)
  const long kbase = sg.kb + (long)hkv * p.Nk;
  const bf16* Kp = p.k + kbase * D;
  const int jdiag = (min(q0w + kBq, Nq) - 1 + offi) / kBk;
  const int ttop = jdiag / W, T = ttop + 1;      // stage n holds tiles 4 (ttop - n) ..

  // slot u of stage n is key tile W (ttop - n) + W - 1 - u
  const uint32_t koff = (uint32_t)(c * D + 8 * h) * 2u;
  auto load_k = [&](int j, bf16x8 (&ka)[KS]) {
    const long k0 = (long)j * kBk;
    // tiles above the diagonal (and past the last stage) read nothing
    const auto rk = make_rsrc(Kp + max(k0, 0l) * D,
                              j >= 0 && j <= jdiag ? (uint32_t)(Nk - k0) * (uint32_t)D * 2u : 0u);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
      ka[kk] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, koff + 32u * kk, 0, 0));
  };
  // masked raw scores of tile j and their row maxima
  auto row_max = [&](int j, const f32x16& s, float (&sv)[16]) {
    const int kb = j * kBk;
    const bool need_mask = (kb + kBk - 1 > q0w + offi) || (q0w + kBq > Nq);
    return halves_max(masked_max(s, need_mask, row_valid ? qrow + offi - kb - 4 * h : -1000000, sv));
  };
  if (tid < 2) resync[tid] = 0;
  if (tid < 64) rowlm[tid >> 5][tid & 31] = f32x2{0.f, kNegInf};
  __syncthreads();
  bf16x8 qreg[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
    qreg[kk] = row_valid ? load8(p.q + (qbase + qrow) * D + 16 * kk + 8 * h) : zero8();

  if (wave < W) {
    const bf16* Vp = p.v + kbase * D;
    constexpr int NIS = STAGE / 512;           // 64-position loads per V stage
    static_assert(NIS * 512 == STAGE, "whole loads per stage");
    constexpr int NJS = (NIS + W - 1) / W;
    uint32_t dma_off[NJS];
#pragma unroll
    for (int u = 0; u < NJS; ++u) dma_off[u] = dma_lane_offset<D>(64 * (wave + W * u) + lane);
    auto fetch_v = [&](int n) {
      const long k0 = (long)(ttop - n) * (W * kBk);
      const i32x4 rv = rsrc_words(Vp + k0 * D, (uint32_t)(Nk - k0) * (uint32_t)D * 2u);
#pragma unroll
      for (int u = 0; u < NJS; ++u) {
        const int j = wave + W * u;
        if (j < NIS) buf_load_lds16(rv, dma_off[u], Vs + (n & 1) * STAGE + 512 * j);
      }
    };
    float m = kNegInf;     // predicted reference
    float sv[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sv[r] = kNegInf;
    // this wavefront's K tile of a stage, to its own LDS slot
    bf16* Kw = Ks + wave * NKL * 512;
    uint32_t k_off[NKL];
#pragma unroll
    for (int u = 0; u < NKL; ++u) k_off[u] = dma_lane_offset<D>(64 * u + lane);
    auto fetch_k = [&](int j) {
      const long k0 = (long)max(j, 0) * kBk;
      // tiles above the diagonal and past the last stage read as zeros
      const i32x4 rk = rsrc_words(Kp + k0 * D, j >= 0 && j <= jdiag
                                                   ? (uint32_t)(Nk - k0) * (uint32_t)D * 2u : 0u);
#pragma unroll
      for (int u = 0; u < NKL; ++u) buf_load_lds16(rk, k_off[u], Kw + 512 * u);
    };
    fetch_k(W * ttop + W - 1 - wave);
    const bf16* kr = lds_pin(Kw + rd_base<D>(c, h));
    for (int n = 0; n <= T; ++n) {
      const int j = W * (ttop - n) + W - 1 - wave;
      wait_vm();                                // K of stage n
      if (n > 0) fetch_v(n - 1);                // read by the consumers at step n + 1
      const int pb = (n - 1) & 1;
      bf16x8 ka[KS];
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) ka[kk] = load8(kr + rd_step<D>(kk));
      // the slot is free once its reads have arrived: the next stage's tile takes it
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(ka[kk])::"memory");
      fetch_k(j - W);
      float mt[W];
#pragma unroll
      for (int u = 0; u < W; ++u) mt[u] = redm[(n + 2) % 3][u][c];
      const f32x2 lm = rowlm[pb][c];            // l and m after stage n - 3
      if (__builtin_amdgcn_readfirstlane(resync[pb])) {
        m = lm[1];          // stage n - 3 ended with another reference: through n - 2 from there
#pragma unroll
        for (int u = 0; u < W; ++u) {
          const float x = redm[(n + 1) % 3][u][c] * p.scale2;
          if (wave_any(x > m + 8.f)) m = fmaxf(m, x);
        }
      }
      // step n of stage n, the scores, under step n of stage n - 1, references and P (no
      // branch between them, so that one's MFMAs run under the other's vector work)
      const f32x16 sc = fwd_scores<KS>(ka, qreg);
      float mw = m;
#pragma unroll
      for (int u = 0; u < W; ++u) {
        const float x = mt[u] * p.scale2;
        const bool mv = (n > 0) & wave_any(x > m + 8.f);
        m = mv ? fmaxf(m, x) : m;
        mw = wave == u ? m : mw;
      }
      const float ps = fwd_probabilities(sv, p.scale2, mw);
      const bf16x8 p0 = hi_bf16x8(sv), p1 = hi_bf16x8(sv + 8);
      Ps[pb][wave][0][lane] = p0;
      Ps[pb][wave][1][lane] = p1;
      if (h == 0) redp[pb][wave][c] = f32x2{ps, mw};
      // The lo terms wherever the test of the tile's share can ask for them.  A tile used
      // with this P has reference mw, and what l held after stage n - 3 is by then
      // 2^(lm[1] - mw) of it (the margin is beyond any rounding of the rescalings) and has
      // only grown since.  (Tiles of another reference are formed again.)
      if (wave_any(ps > kFwdLoShare * 0.999f * (lm[0] * rescale(lm[1], mw)))) {
        Ps[pb][wave][2][lane] = lo_bf16x8(sv, p0);
        Ps[pb][wave][3][lane] = lo_bf16x8(sv + 8, p1);
      }
      const float raw = row_max(j, sc, sv);
      if (h == 0) redm[n % 3][wave][c] = raw;
      wait_vm_keep<NKL>();                      // this wavefront's V loads have landed
      __syncthreads();
    }
    __syncthreads();
    return;
  }

  // consumers
  const int cw = wave - W;
  const int tro = tr_base<D>(4 * h + (t16 >> 2), G & 1, t16);
  const float nthr = row_threshold(p.log2tau, qrow, offi);
  float m = kNegInf, l = 0.f;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
  int cnt = 0;   // retained tiles in which this row has a legal key

  for (int s = 0; s < T + 2; ++s) {
    if (s >= 2) {
      const int n = s - 2, pb = n & 1, rm = n % 3;
      const int jtop = W * (ttop - n) + W - 1;           // slot 0's tile
      // the row's last legal key relative to slot u is lim + kBk u
      const int lim = row_valid ? qrow + offi - jtop * kBk : -1000000;
      const bf16* vtb = lds_pin(Vs + pb * STAGE + tro + 8 * min(cw, DB - 1));
      auto v_operand = [&](int u, int ks) {
        const bf16* vt = vtb + ((W - 1 - u) * kBk + 16 * ks) * (D + 8);
        return cat(lds_read_tr(vt), lds_read_tr(vt + 8 * (D + 8)));
      };
      bool bad = false;
      float mt[W];
      f32x2 sr[W];
#pragma unroll
      for (int u = 0; u < W; ++u) {
        mt[u] = redm[rm][u][c];
        sr[u] = redp[pb][u][c];
      }
      // all the slots at once, as if each were retained: the normalizer m + log2(l) only
      // grows, so a slot that passes the test against its last value (with a margin
      // beyond any rounding) passes its own
      float al[W], lu = l, mm = m;
      int lo = 0, moves = 0;
      unsigned long long differ = 0;
#pragma unroll
      for (int u = 0; u < W; ++u) {
        mt[u] *= p.scale2;
        if (wave_any(mt[u] > mm + 8.f)) {
          const float m_new = fmaxf(mm, mt[u]);
          al[u] = rescale(mm, m_new);
          lu *= al[u];
          mm = m_new;
          moves |= 1 << u;
        }
        differ |= __builtin_amdgcn_ballot_w64(sr[u][1] != mm);
        lu += sr[u][0];
        lo |= (wave_any(sr[u][0] > kFwdLoShare * lu) ? 1 : 0) << u;
      }
      const float need = 0.01f - nthr + (mm + fast_log2(lu));
      bool all = (jtop <= jdiag) & (differ == 0);
#pragma unroll
      for (int u = 0; u < W; ++u)
        all &= (__builtin_amdgcn_ballot_w64(lim + kBk * u >= 0) &
                __builtin_amdgcn_ballot_w64(mt[u] >= need)) != 0;
      if (all) {
        l = lu;
        m = mm;
#pragma unroll
        for (int u = 0; u < W; ++u) cnt += lim + kBk * u >= 0 ? 1 : 0;
        bf16x8 va[W][2], pp[W][2], pl[W][2];
#pragma unroll
        for (int u = 0; u < W; ++u)
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) {
            va[u][ks] = v_operand(u, ks);
            pp[u][ks] = Ps[pb][u][ks][lane];
          }
        if (lo) {
#pragma unroll
          for (int u = 0; u < W; ++u)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) pl[u][ks] = Ps[pb][u][2 + ks][lane];
        }
#pragma unroll
        for (int u = 0; u < W; ++u) {
          if ((moves >> u) & 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] *= al[u];
          }
          acc = mfma32(va[u][0], pp[u][0], acc);
          acc = mfma32(va[u][1], pp[u][1], acc);
          if ((lo >> u) & 1) {
            acc = mfma32(va[u][0], pl[u][0], acc);
            acc = mfma32(va[u][1], pl[u][1], acc);
          }
        }
      } else {
#pragma unroll 1
        for (int u = max(0, jtop - jdiag); u < W; ++u) {
          const bool voter = lim + kBk * u >= 0;
          const float rw = redm[rm][u][c];
          const f32x2 pr = redp[pb][u][c];
          if (!wave_any(voter & online_demand(rw, p.scale2, m, l, nthr))) continue;
          const float x = rw * p.scale2;
          if (wave_any(x > m + 8.f)) {
            const float m_new = fmaxf(m, x);
            const float alpha = rescale(m, m_new);
            l *= alpha;
            m = m_new;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] *= alpha;
          }
          cnt += voter ? 1 : 0;
          const bf16x8 v0 = v_operand(u, 0), v1 = v_operand(u, 1);
          bf16x8 p0, p1, p2, p3;
          float ps = pr[0];
          if (wave_any(pr[1] != m)) {
            // P again, from the keys: its reference was not the row's
            bad = true;
            float sv[16];
            bf16x8 ka[KS];
            load_k(jtop - u, ka);
            row_max(jtop - u, fwd_scores<KS>(ka, qreg), sv);
            ps = fwd_probabilities(sv, p.scale2, m);
            p0 = hi_bf16x8(sv);
            p1 = hi_bf16x8(sv + 8);
            p2 = lo_bf16x8(sv, p0);
            p3 = lo_bf16x8(sv + 8, p1);
          } else {
            p0 = Ps[pb][u][0][lane];
            p1 = Ps[pb][u][1][lane];
            p2 = Ps[pb][u][2][lane];   // meaningful where the share below asks for them
            p3 = Ps[pb][u][3][lane];
          }
          l += ps;
          acc = mfma32(v0, p0, acc);
          acc = mfma32(v1, p1, acc);
          if (wave_any(ps > kFwdLoShare * l)) {
            acc = mfma32(v0, p2, acc);
            acc = mfma32(v1, p3, acc);
          }
        }
      }
      if (cw == 0) {
        if (h == 0) rowlm[s & 1][c] = f32x2{l, m};
        if (lane == 0) resync[s & 1] = bad ? 1 : 0;
      }
    }
    __syncthreads();
  }

  if (row_valid) {
    const float inv = 1.f / l;
    if (cw < DB) {
      const long orow = (qbase + qrow) * D;
#pragma unroll
      for (int g = 0; g < 4; ++g)
        store_out4(p.o, orow + 32 * cw + 8 * g + 4 * h,
                   f32x4{acc[4 * g] * inv, acc[4 * g + 1] * inv, acc[4 * g + 2] * inv,
                         acc[4 * g + 3] * inv}, p.o_bf16);
    }
    if (cw == 0 && h == 0) {
      p.lse[qbase + qrow] = (m + fast_log2(l)) * kLn2;
      if (p.row_tiles) p.row_tiles[qbase + qrow] = cnt;
    }
  }
}

hipError_t launch_fwd(const FwdParams& p, int D, hipStream_t st) {
  if (fwd_takes_rows(p, D)) {
    dim3 grid((unsigned)((p.max_len + kBq - 1) / kBq) * p.B * p.Hq), block(2 * kRowsTiles * 64);
    if (D == 128)
      hipLaunchKernelGGL(mala_fwd_rows_kernel<128>, grid, block, 0, st, p);
    else
      hipLaunchKernelGGL(mala_fwd_rows_kernel<64>, grid, block, 0, st, p);
    return hipGetLastError();
  }
  dim3 grid((unsigned)p.nqblk * p.B * p.Hq), block(kFwdWaves * 64);
  if (D == 128)
    hipLaunchKernelGGL(mala_fwd_kernel<128>, grid, block, 0, st, p);
  else
    hipLaunchKernelGGL(mala_fwd_kernel<64>, grid, block, 0, st, p);
  return hipGetLastError();
}

}  // namespace mala
