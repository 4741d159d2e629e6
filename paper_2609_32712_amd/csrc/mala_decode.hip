// MALA split-KV decode for gfx950 (Fused Execution section and its appendix:
// each split tests its tiles against its own partial normalizer, with L = Nk).
//
// One wavefront (= one workgroup) owns one split of one (batch, KV head) and
// serves up to 16 query heads of the GQA group at once (larger groups take
// ceil(group / 16) wavefronts), so the K and V bytes of a tile are read once per
// 16 heads.  Decode is HBM-bound: K is always read (score
// discovery), V only when at least one head of the group retains the tile.
//
// With per-sequence cache lengths n_b, sequence b sees keys [0, n_b) (L = n_b) and
// its ceil(n_b / 32) tiles are cut into the splits as for a cache of n_b tokens.
//
// Per 32-key tile, in descending order inside the split:
//   S^T = K_t Q^T     2 x 4 (D = 128) MFMAs 16x16x32; K arrives in registers in
//                     whole contiguous rows (1 KB per load instruction), passes
//                     through LDS and is read back as the A operands; lane
//                     (g, col) holds query head col and 8 of the 32 keys; K is
//                     prefetched two tiles ahead
//   test              per head against that head's running (m, l) of the split
//   retained (any)    V tile (fetched one tile ahead when a look-ahead test says
//                     it may be needed) -> LDS; per head P = exp2(S - m_new) (0 for
//                     heads that skip); O^T += V^T P^T with V^T through
//                     ds_read_b64_tr_b16.
// Every K and V load is a streaming buffer load (each byte is read once per call)
// that is always issued: rows past the cache length, tiles outside the split and V
// tiles the look-ahead test rules out have a resource of 0 bytes, read as zeros and
// move no data.  With no load under a
// branch, the compiler's waits count exactly the loads a step needs, so the next
// K tile and the next V tile stay in flight while a tile is processed.
// Partials (O / l, lse, count) go to the workspace; a second kernel merges the
// splits with the normalizer-aware (log-sum-exp weighted) reduction.  With one split the
// outputs are written at once.  Calls of few splits run a team of wavefronts per split
// (mala_decode_team_kernel).
#include "mala_device.h"
#include "mala_kernels.h"

namespace mala {

// The result of split s for head bh (of lane group g's columns): O / l, lse (natural log)
// and the retained-tile count, as a partial, or as the outputs when there is one split.  A
// split without tiles has l = 0 (o = 0, lse = -inf: the merge skips it); a NaN or Inf input
// leaves l NaN, which must reach the merge as NaN, not as an empty split.
template <int D>
__device__ __forceinline__ void write_split(const DecParams& p, long bh, int s, int g,
                                            const f32x4 (&acc)[D / 16], float m, float l, int cnt) {
  const float inv = l != 0.f ? 1.f / l : 0.f;
  const float lse = l != 0.f ? (m + fast_log2(l)) * kLn2 : kNegInf;
  if (p.S == 1) {
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
      store_out4(p.o, bh * D + 16 * db + 4 * g, acc[db] * inv, p.o_bf16);
    if (g == 0) {
      p.lse[bh] = lse;
      if (p.head_tiles) p.head_tiles[bh] = cnt;
    }
    return;
  }
  float* pp = p.part + (bh * p.S + s) * (D + kDecStride);
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
    *reinterpret_cast<f32x4*>(pp + 16 * db + 4 * g) = acc[db] * inv;
  if (g == 0) {
    pp[D] = lse;
    pp[D + 1] = __int_as_float(cnt);
  }
}

template <int D>
__global__ __launch_bounds__(64) void mala_decode_split_kernel(DecParams p) {
  constexpr int KS = D / 32;   // k-steps of 32 over head_dim
  constexpr int NDB = D / 16;  // 16-row blocks of O^T
  constexpr int LD = D + 8;
  constexpr int VCH = kDecBk * D / 8 / 64;   // 16-byte V chunks per lane per tile
  __shared__ __attribute__((aligned(16))) bf16 Ks[kDecBk * LD];
  __shared__ __attribute__((aligned(16))) bf16 Vs[kDecBk * LD];

  const int lane = threadIdx.x, g = lane >> 4, col = lane & 15;
  const int s = blockIdx.x % p.S;
  const int chunk = (blockIdx.x / p.S) % p.nchunk;     // heads 16 chunk .. 16 chunk + 15
  const int bhk = blockIdx.x / p.S / p.nchunk;
  const int b = bhk / p.Hkv, hkv = bhk % p.Hkv, grp = p.Hq / p.Hkv;
  const int nh = min(16, grp - 16 * chunk);             // query heads of this wavefront
  // this sequence's cache length n (clamped into [0, Nk]), its tiles and split range
  int n = p.Nk, T = p.T, tps = p.tps;
  float thr2 = p.thr2;
  if (p.lens) {
    n = min(max(p.lens[b], 0), p.Nk);
    T = (n + kDecBk - 1) / kDecBk;
    tps = (T + p.S - 1) / p.S;
    thr2 = p.log2tau - log2f((float)n);   // L = n (n = 0 leaves no tile to test)
  }
  const int t_lo = s * tps, t_hi = min(T, t_lo + tps);
  const bool head_valid = col < nh;
  const int hq = hkv * grp + 16 * chunk + col;

  bf16x8 qreg[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
    qreg[kk] = head_valid ? load8(p.q + ((long)b * p.Hq + hq) * D + 32 * kk + 8 * g) : zero8();
  wait_vm();   // no wait for these loads is left for the tile loop

  const bf16* Kp = p.k + (long)bhk * p.Nk * D;
  const bf16* Vp = p.v + (long)bhk * p.Nk * D;

  float m = kNegInf, l = 0.f;
  f32x4 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  int cnt = 0;
  unsigned vloads = 0, vfetch = 0;   // V tiles consumed / fetched (statistics)
  unsigned long long hsum = 0;       // fingerprints of this head's retained tiles

  // A K or V tile in registers as whole rows: lane chunk e holds the 16 bytes at
  // byte 16 (lane + 64 e) of the tile, row (lane + 64 e) / (D / 8).  The resource
  // covers the tile's rows below n when the tile is wanted and nothing otherwise.
  auto tile_rsrc = [&](const bf16* base, int t, bool want) {
    const long k0 = (long)max(t, 0) * kDecBk;
    const long rows = want && t >= 0 ? min((long)kDecBk, (long)n - k0) : 0;
    return make_rsrc(base + k0 * D, (uint32_t)(rows > 0 ? rows * D * 2 : 0));
  };
  bf16x8 kr[VCH], vr[VCH];
  auto load_k = [&](int t) {
    const auto r = tile_rsrc(Kp, t, t >= t_lo);
#pragma unroll
    for (int e = 0; e < VCH; ++e) kr[e] = buf_load8_stream(r, 16u * (lane + 64 * e));
  };
  auto load_v = [&](int t, bool want) {
    const auto r = tile_rsrc(Vp, t, want && t >= t_lo);
#pragma unroll
    for (int e = 0; e < VCH; ++e) vr[e] = buf_load8_stream(r, 16u * (lane + 64 * e));
  };
  // tile rows to LDS (row stride LD keeps the operand reads below conflict-free)
  auto to_lds = [&](bf16* dst, const bf16x8 (&x)[VCH]) {
#pragma unroll
    for (int e = 0; e < VCH; ++e) {
      const int ch = lane + 64 * e;
      store8(dst + (ch / (D / 8)) * LD + (ch % (D / 8)) * 8, x[e]);
    }
  };
  // Base-2 scores of the tile whose K is in kr, for this lane's head (8 keys), and
  // their max over the tile; the next K tile (t - 1) starts loading as soon as kr
  // is in LDS.  One wavefront per workgroup: its LDS accesses complete in issue
  // order, so the reads below see the stores and the next stores follow the reads.
  auto scores = [&](int t, float (&sv)[8]) {
    to_lds(Ks, kr);
    load_k(t - 1);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s0 = mfma16(load8(Ks + col * LD + 32 * kk + 8 * g), qreg[kk], s0);
      s1 = mfma16(load8(Ks + (16 + col) * LD + 32 * kk + 8 * g), qreg[kk], s1);
    }
    const long kb = (long)t * kDecBk;
    float mt = kNegInf;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x0 = s0[r] * p.scale2, x1 = s1[r] * p.scale2;
      if (kb + 4 * g + r >= n) x0 = kNegInf;
      if (kb + 16 + 4 * g + r >= n) x1 = kNegInf;
      sv[r] = x0;
      sv[4 + r] = x1;
      mt = fmaxf(mt, fmaxf(x0, x1));
    }
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    return fmaxf(mt, __shfl_xor(mt, 32));
  };

  // Pipeline: while tile t is decided and processed, K of tile t - 1 is already in
  // registers (its scores are computed first) and K of t - 2 is loading.  Whether
  // tile t - 1 can still be retained is checked against the state BEFORE tile t's
  // update; since the retained normalizer only grows, a tile that fails this check
  // fails the real test too, so V of t - 1 is fetched early exactly when it may be
  // needed (with a small margin against fp32 rounding of the normalizer).
  constexpr float kHintMargin = 1e-2f;
  float sv[8], sn[8];
  float mt = kNegInf, mtn = kNegInf;
  if (t_hi > t_lo) {
    load_k(t_hi - 1);
    mt = scores(t_hi - 1, sv);   // also starts K of t_hi - 2
    load_v(t_hi - 1, true);      // the first tile of a split is always retained (l = 0)
    ++vfetch;
  }
  for (int t = t_hi - 1; t >= t_lo; --t) {
    const bool has_next = t - 1 >= t_lo;
    mtn = scores(t - 1, sn);     // zeros past the split's first tile, not used then
    const float lse_run = m + fast_log2(l);
    const bool demand = head_valid && (l == 0.f || (mt - lse_run >= thr2));
    const bool hint =
        has_next && wave_any(head_valid && (l == 0.f || (mtn - lse_run >= thr2 - kHintMargin)));
    // V of tile t goes to LDS, and V of t - 1 (if the look-ahead test wants it) starts
    // loading into the freed registers before tile t's update runs
    const bool any_demand = wave_any(demand);
    if (any_demand) to_lds(Vs, vr);
    load_v(t - 1, hint);
    vfetch += hint ? 1u : 0u;
    if (any_demand) {
      ++vloads;
      float alpha = 1.f, m_new = m;
      if (demand) {
        m_new = fmaxf(m, mt);
        alpha = fast_exp2(m - m_new);
      }
      float ps = 0.f;
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        const float e = demand ? fast_exp2(sv[r] - m_new) : 0.f;
        sv[r] = e;
        ps += e;
      }
      ps += __shfl_xor(ps, 16);
      ps += __shfl_xor(ps, 32);
      if (demand) {
        l = alpha * l + ps;
        m = m_new;
        ++cnt;
        if (p.counters) hsum += tile_hash(b, hq, 0, t);
      }
      bf16x8 ph, pl;
      split_bf16x8(sv, ph, pl);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const bf16* vrow = Vs + (4 * g + (col >> 2)) * LD + 16 * db + 4 * (col & 3);
        const bf16x8 a = cat(lds_read_tr(vrow), lds_read_tr(vrow + 16 * LD));
        acc[db] = mfma16(a, ph, acc[db] * alpha);
        acc[db] = mfma16(a, pl, acc[db]);
      }
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) sv[r] = sn[r];
    mt = mtn;
  }

  if (head_valid) write_split<D>(p, (long)b * p.Hq + hq, s, g, acc, m, l, cnt);
  if (p.counters) {
    if (head_valid && g == 0 && cnt) {
      atomicAdd(&p.counters[kCntRetained], (unsigned long long)cnt);
      atomicAdd(&p.counters[kCntSlots], (unsigned long long)cnt * kDecBk);
      atomicAdd(&p.counters[kCntSetHash], hsum);
    }
    if (lane == 0) {
      atomicAdd(&p.counters[kCntLegal], (unsigned long long)(t_hi > t_lo ? t_hi - t_lo : 0) * nh);
      if (vfetch) atomicAdd(&p.counters[kCntVTiles], (unsigned long long)vfetch);
      if (vloads) atomicAdd(&p.counters[kCntVNeeded], (unsigned long long)vloads);
    }
  }
}

// Decode of few splits: W wavefronts per split, a key tile each, so that calls whose splits
// do not fill the chip (one sequence, few heads, short caches) read and score W tiles of a
// split at once.  What bounds such a call is the latency of a split's chain of tiles (~1.2
// us each for the kernel above); only the test is serial.  Per round of W tiles, from the
// last one down: every wavefront scores its tile and publishes the tile's maximum and sum
// per head (reference: that maximum); barrier; every wavefront takes the W tests in order,
// carrying (m, l) of the split; a wavefront whose tile some head retains accumulates its
// P V against a reference of its own (the largest maximum of its retained tiles).  The W
// accumulators are brought to the split's reference and added at the end.  K and V of the
// next round load while a round is worked on; V is fetched for every tile.
template <int D, int W>
__global__ __launch_bounds__(W * 64) void mala_decode_team_kernel(DecParams p) {
  constexpr int KS = D / 32;   // k-steps of 32 over head_dim
  constexpr int NDB = D / 16;  // 16-row blocks of O^T
  constexpr int LD = D + 8;
  constexpr int VCH = kDecBk * D / 8 / 64;   // 16-byte chunks per lane per tile
  __shared__ __attribute__((aligned(16))) bf16 Ks[W][kDecBk * LD];
  __shared__ __attribute__((aligned(16))) bf16 Vs[W][kDecBk * LD];
  __shared__ f32x2 red[2][W][16];            // per tile and head: maximum, sum
  __shared__ float refs[W][16];              // the wavefronts' references at the end

  const int lane = threadIdx.x & 63, g = lane >> 4, col = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s = blockIdx.x % p.S;
  const int chunk = (blockIdx.x / p.S) % p.nchunk;     // heads 16 chunk .. 16 chunk + 15
  const int bhk = blockIdx.x / p.S / p.nchunk;
  const int b = bhk / p.Hkv, hkv = bhk % p.Hkv, grp = p.Hq / p.Hkv;
  const int nh = min(16, grp - 16 * chunk);             // query heads of this workgroup
  int n = p.Nk, T = p.T, tps = p.tps;
  float thr2 = p.thr2;
  if (p.lens) {
    n = min(max(p.lens[b], 0), p.Nk);
    T = (n + kDecBk - 1) / kDecBk;
    tps = (T + p.S - 1) / p.S;
    thr2 = p.log2tau - log2f((float)n);   // L = n (n = 0 leaves no tile to test)
  }
  const int t_lo = s * tps, t_hi = min(T, t_lo + tps);
  const bool head_valid = col < nh;
  const int hq = hkv * grp + 16 * chunk + col;
  const bf16* Kp = p.k + (long)bhk * p.Nk * D;
  const bf16* Vp = p.v + (long)bhk * p.Nk * D;

  // tile rows at or past n, and tiles outside the split, read as zeros
  bf16x8 kr[VCH], vr[VCH];
  auto load = [&](const bf16* base, int t, bf16x8 (&x)[VCH]) {
    const long k0 = (long)max(t, 0) * kDecBk;
    const long rows = t >= t_lo ? min((long)kDecBk, (long)n - k0) : 0;
    const auto r = make_rsrc(base + k0 * D, (uint32_t)(rows > 0 ? rows * D * 2 : 0));
#pragma unroll
    for (int e = 0; e < VCH; ++e) x[e] = buf_load8_stream(r, 16u * (lane + 64 * e));
  };
  auto to_lds = [&](bf16* dst, const bf16x8 (&x)[VCH]) {
#pragma unroll
    for (int e = 0; e < VCH; ++e) {
      const int ch = lane + 64 * e;
      store8(dst + (ch / (D / 8)) * LD + (ch % (D / 8)) * 8, x[e]);
    }
  };
  load(Kp, t_hi - 1 - w, kr);
  load(Vp, t_hi - 1 - w, vr);
  bf16x8 qreg[KS];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk)
    qreg[kk] = head_valid ? load8(p.q + ((long)b * p.Hq + hq) * D + 32 * kk + 8 * g) : zero8();

  float m = kNegInf, l = 0.f;        // of the split
  float ref = kNegInf;               // of this wavefront's accumulator
  f32x4 acc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
  int cnt = 0;
  unsigned vloads = 0;               // V tiles consumed (statistics)
  unsigned long long hsum = 0;       // fingerprints of this head's retained tiles

  for (int t0 = t_hi - 1, round = 0; t0 >= t_lo; t0 -= W, ++round) {
    const int t = t0 - w;
    // the wavefront's LDS accesses complete in issue order: its reads below see the
    // stores, the next round's stores follow the reads
    to_lds(Ks[w], kr);
    load(Kp, t - W, kr);
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      s0 = mfma16(load8(Ks[w] + col * LD + 32 * kk + 8 * g), qreg[kk], s0);
      s1 = mfma16(load8(Ks[w] + (16 + col) * LD + 32 * kk + 8 * g), qreg[kk], s1);
    }
    const long kb = (long)t * kDecBk;
    float sv[8], mt = kNegInf;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x0 = s0[r] * p.scale2, x1 = s1[r] * p.scale2;
      if (kb + 4 * g + r >= n) x0 = kNegInf;
      if (kb + 16 + 4 * g + r >= n) x1 = kNegInf;
      sv[r] = x0;
      sv[4 + r] = x1;
      mt = fmaxf(mt, fmaxf(x0, x1));
    }
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    // a tile of -inf scores only (masked keys) is retained at tau = 0 and sums to 0, not NaN
    const float shift = mt == kNegInf ? 0.f : mt;
    float ps = 0.f;
#pragma unroll
    for (int r = 0; r < 8; ++r) ps += fast_exp2(sv[r] - shift);
    ps += __shfl_xor(ps, 16);
    ps += __shfl_xor(ps, 32);
    if (g == 0) red[round & 1][w][col] = f32x2{mt, ps};
    to_lds(Vs[w], vr);
    load(Vp, t - W, vr);
    __syncthreads();
    // the tests of the round's tiles in order
    f32x2 rd[W];
#pragma unroll
    for (int u = 0; u < W; ++u) rd[u] = red[round & 1][u][col];
    bool mine = false;
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const bool demand = (t0 - u >= t_lo) & head_valid &
                          ((l == 0.f) | (rd[u][0] - (m + fast_log2(l)) >= thr2));
      if (u == w) mine = demand;
      if (demand) {
        const float m_new = fmaxf(m, rd[u][0]);
        l = l * fast_exp2(m - m_new) + rd[u][1] * fast_exp2(rd[u][0] - m_new);
        m = m_new;
        ++cnt;
        if (p.counters) hsum += tile_hash(b, hq, 0, t0 - u);
      }
      if (p.counters) vloads += wave_any(demand) ? 1u : 0u;
    }
    if (wave_any(mine)) {
      float alpha = 1.f;
      if (mine) {   // the accumulator is 0 until a tile with a finite maximum sets ref
        const float r_new = fmaxf(ref, mt);
        alpha = r_new == kNegInf ? 1.f : fast_exp2(ref - r_new);
        ref = r_new;
      }
      const float rs = ref == kNegInf ? 0.f : ref;
#pragma unroll
      for (int r = 0; r < 8; ++r) sv[r] = mine ? fast_exp2(sv[r] - rs) : 0.f;
      bf16x8 ph, pl;
      split_bf16x8(sv, ph, pl);
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const bf16* vrow = Vs[w] + (4 * g + (col >> 2)) * LD + 16 * db + 4 * (col & 3);
        const bf16x8 a = cat(lds_read_tr(vrow), lds_read_tr(vrow + 16 * LD));
        acc[db] = mfma16(a, ph, acc[db] * alpha);
        acc[db] = mfma16(a, pl, acc[db]);
      }
    }
  }

  // add the accumulators: through LDS (the V tiles' slots, 16 heads x D floats each), the
  // first wavefront sums
  if (w) {
    float* out = reinterpret_cast<float*>(Vs[w]);
    static_assert(sizeof(Vs[0]) >= 16 * D * sizeof(float), "an accumulator fits a V tile");
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      *reinterpret_cast<f32x4*>(out + (db * 64 + lane) * 4) = acc[db];
    if (g == 0) refs[w][col] = ref;
  }
  __syncthreads();
  if (w == 0) {
    // (a wavefront without retained tiles holds zeros and ref = -inf)
    const float f0 = ref == kNegInf ? 1.f : fast_exp2(ref - m);
#pragma unroll
    for (int db = 0; db < NDB; ++db) acc[db] *= f0;
#pragma unroll
    for (int u = 1; u < W; ++u) {
      const float r = refs[u][col], f = r == kNegInf ? 1.f : fast_exp2(r - m);
      const float* in = reinterpret_cast<const float*>(Vs[u]);
#pragma unroll
      for (int db = 0; db < NDB; ++db)
        acc[db] += *reinterpret_cast<const f32x4*>(in + (db * 64 + lane) * 4) * f;
    }
    if (head_valid) write_split<D>(p, (long)b * p.Hq + hq, s, g, acc, m, l, cnt);
    if (p.counters) {
      const unsigned long long tiles = t_hi > t_lo ? t_hi - t_lo : 0;
      if (head_valid && g == 0 && cnt) {
        atomicAdd(&p.counters[kCntRetained], (unsigned long long)cnt);
        atomicAdd(&p.counters[kCntSlots], (unsigned long long)cnt * kDecBk);
        atomicAdd(&p.counters[kCntSetHash], hsum);
      }
      if (lane == 0 && tiles) {
        atomicAdd(&p.counters[kCntLegal], tiles * nh);
        atomicAdd(&p.counters[kCntVTiles], tiles);
        atomicAdd(&p.counters[kCntVNeeded], (unsigned long long)vloads);
      }
    }
  }
}

// Normalizer-aware merge of the split partials: lse = logsumexp_s lse_s,
// o = sum_s exp(lse_s - lse) o_s.  One workgroup per (batch, query head).
//
// What bounds it is latency: a few KB per head, read once.  Every wavefront takes the
// splits' lse over its lanes (one load and a wave reduction per 64 splits instead of
// three serial passes), the weights go through LDS 256 splits at a time, and the
// workgroup's 256 threads read the partial rows as 16-byte chunks, NG splits at once,
// the first two rows of each group before the weights are known.  With one wavefront
// that walked the splits three times this kernel took 24 us for 512 heads x 16 splits
// (D = 128); a decode call over 16 ragged 8192-token caches went from 74.2 to 54.7 us,
// one over a single 4096-token cache (32 heads x 8 splits) from 33.5 to 25.2 us.
constexpr int kCombineThreads = 256;
template <int D>
__global__ __launch_bounds__(kCombineThreads) void mala_decode_combine_kernel(
    const float* part, void* o, bool o_bf16, float* lse, int32_t* head_tiles, int S) {
  constexpr int LPR = D / 4;                     // lanes per partial row (16 bytes each)
  constexpr int NG = kCombineThreads / LPR;      // splits read at once
  constexpr int LD = D + kDecStride;
  __shared__ float wts[kCombineThreads];
  __shared__ __attribute__((aligned(16))) f32x4 sums[kCombineThreads];
  const long bh = blockIdx.x;
  const float* pp = part + bh * S * LD;
  const int tid = threadIdx.x, lane = tid & 63;
  const int grp = tid / LPR, cl = tid % LPR;
  const auto row = [&](int s) { return *reinterpret_cast<const f32x4*>(pp + (long)s * LD + 4 * cl); };
  f32x4 x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
  if (grp < S) x0 = row(grp);
  if (grp + NG < S) x1 = row(grp + NG);

  float mx = kNegInf;
  int cnt = 0;
  float l0 = kNegInf;                            // this lane's split of the first 64
  for (int s = lane; s < S; s += 64) {
    const f32x2 lc = *reinterpret_cast<const f32x2*>(pp + (long)s * LD + D);
    if (s == lane) l0 = lc[0];
    mx = fmaxf(mx, lc[0]);
    cnt += __float_as_int(lc[1]);
  }
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) {
    mx = fmaxf(mx, __shfl_xor(mx, w));
    cnt += __shfl_xor(cnt, w);
  }
  float z = 0.f;
  for (int s = lane; s < S; s += 64) {
    const float ls = s == lane ? l0 : pp[(long)s * LD + D];
    if (ls != kNegInf) z += expf(ls - mx);
  }
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) z += __shfl_xor(z, w);
  const float L = mx + logf(z);

  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < S; s0 += kCombineThreads) {
    if (s0) __syncthreads();                     // the last chunk's weights have been read
    float w = 0.f;                               // an empty split (o = 0, lse = -inf) adds nothing
    if (s0 + tid < S) {
      const float ls = pp[(long)(s0 + tid) * LD + D];
      w = ls != kNegInf ? expf(ls - L) : 0.f;
    }
    wts[tid] = w;
    __syncthreads();
    const int n = min(S - s0, kCombineThreads);
    int s = grp;
    if (s0 == 0) {
      if (s < n) acc += wts[s] * x0;
      s += NG;
      if (s < n) acc += wts[s] * x1;
      s += NG;
    }
#pragma unroll 4
    for (; s < n; s += NG) acc += wts[s] * row(s0 + s);
  }
  sums[tid] = acc;
  __syncthreads();
  if (tid < LPR) {
#pragma unroll
    for (int g = 1; g < NG; ++g) acc += sums[g * LPR + tid];
    store_out4(o, bh * D + 4 * tid, acc, o_bf16);
  }
  if (tid == 0) {
    lse[bh] = L;
    if (head_tiles) head_tiles[bh] = cnt;
  }
}

// Up to one split per CU the chain of a split's tiles sets the time and a team takes it
// (us per decode call with its merge, one wavefront / team of 4 / of 8 per split; D = 128):
// 64 splits of 16 tiles 26.5 / 16.2 / 15.8, 256 of 16 27.9 / 19.6 / 20.9, 256 of 256 313 / 163
// / 167, 64 of 782 881 / 378 / 327; D = 64, 128 of 64 65 / 31.8 / 26.7.  With 512 splits one
// wavefront each does as well (28.9 / 28.8 / 36.5) and fetches only the V tiles it needs.
template <int D>
static void launch_decode_t(const DecParams& p, hipStream_t st) {
  const unsigned n = (unsigned)p.B * p.Hkv * p.nchunk * p.S;
  const int w = n > (unsigned)kNumCus || p.tps < 2 ? 1 : n <= 128 && p.tps >= 32 ? 8 : 4;
  if (w == 8)
    hipLaunchKernelGGL((mala_decode_team_kernel<D, 8>), dim3(n), dim3(512), 0, st, p);
  else if (w == 4)
    hipLaunchKernelGGL((mala_decode_team_kernel<D, 4>), dim3(n), dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL(mala_decode_split_kernel<D>, dim3(n), dim3(64), 0, st, p);
  if (p.S > 1)
    hipLaunchKernelGGL(mala_decode_combine_kernel<D>, dim3((unsigned)p.B * p.Hq),
                       dim3(kCombineThreads), 0, st, p.part, p.o, (bool)p.o_bf16, p.lse,
                       p.head_tiles, p.S);
}

hipError_t launch_decode(const DecParams& p, int D, hipStream_t st) {
  if (D == 128)
    launch_decode_t<128>(p, st);
  else
    launch_decode_t<64>(p, st);
  return hipGetLastError();
}

}  // namespace mala
