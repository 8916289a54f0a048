// The C = 128 screen for per-column weights (device code), a kernel of its own
// and the whitened screen's way for the column blocks that it does not take.
#pragma once

#include <math.h>

#include "awsrc_internal.h"
#include "mfma_bf16.h"
#include "rescore64.h"

namespace awsrc {

// The u fragments of NB x 16 tiles (rows row0 + 16 nb + n) over the C = 32
// NKS coordinates of column block blk, per-column weights: lane (n, g) holds
// coordinates 32 ks + 8 g .. + 7 of each of its NB rows, split exactly in
// three bf16 parts; en[nb] gets the tile's weighted energy sum_j d_j r_j^2
// (over the four lanes n, n + 16, n + 32, n + 48 that share a row).  Every
// load is issued before any is used: the residual as 2 NB NKS chunks of four
// weights, the column weights as 2 NKS chunks (the same for every row).
template <int C, int NB>
__device__ __forceinline__ void load_u_col(const EncodeArgs& a, int64_t row0, int blk, int n, int g,
                                           u32x4 (&uh)[NB][C / 32], u32x4 (&um)[NB][C / 32],
                                           u32x4 (&ul)[NB][C / 32], float (&en)[NB]) {
  constexpr int NKS = C / 32;
  constexpr int NCH = 2 * NB * NKS;
  int64_t o[NCH];
  bool valid[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int64_t row = row0 + 16 * nb + n;
    valid[nb] = row < a.rows;
    const int64_t rr = valid[nb] ? row : a.rows - 1;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int64_t base = rr * a.cols + (int64_t)blk * C + 32 * ks + 8 * g;
      o[2 * (nb * NKS + ks)] = base;
      o[2 * (nb * NKS + ks) + 1] = base + 4;
    }
  }
  gf32x4 dv[2 * NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    dv[2 * ks] = gload4f(a.d + (int64_t)blk * C + 32 * ks + 8 * g);
    dv[2 * ks + 1] = gload4f(a.d + (int64_t)blk * C + 32 * ks + 8 * g + 4);
  }
  float rv[NCH][4];
  load_residual4<NCH>(a.W, a.w_dtype, a.W0, o, rv);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float e = 0.0f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      float u[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float r = rv[2 * (nb * NKS + ks) + (k >> 2)][k & 3];
        const float dj = dv[2 * ks + (k >> 2)][k & 3];
        u[k] = valid[nb] ? dj * r : 0.0f;
        e = fmaf(dj * r, r, e);
      }
      split3(u, uh[nb][ks], um[nb][ks], ul[nb][ks]);
    }
    e += __shfl_xor(e, 16, 64);
    en[nb] = e + __shfl_xor(e, 32, 64);
  }
}

// ----------------------------------------------------------------------------
// C = 128, per-column weights.  The u fragments of a 128-coordinate tile take
// twice the registers, so a wavefront holds 32 consecutive rows of one column
// block (2 groups of 16 tiles x 4 K steps x 3 bf16 parts) and gives the two
// seeds of a pair to its two lane halves: lane = (seed of the pair, tile).
// The seed is then uniform per half only, so each lane reads its seed's
// per-column factors with vector loads (two addresses per wavefront).  The
// bound works on raw b (without the 1/sqrt(128) of the basis), so it comes
// out C times larger and the threshold is scaled by C instead; a scoring
// round scales b by 1/sqrt(128) and solves again (not a power of two, so
// raw units would round the fp16 scale differently).
//
// Every candidate gets the forward solve with its seed's factor and the bound
// b^T (G + eps I)^-1 b on every rounding of its fit (screen_fwd); those whose
// bound reaches the re-score window below the tile's current best (over both
// halves) wait in one queue per wavefront, appended in step order, and a
// scoring round takes the 64 oldest, one per lane (each reading its entry's
// factor again), after which each owner lane inserts its results in queue
// order (seed order), as in the per-element screen.  Each half keeps its own
// top two, merged at the end.
constexpr int kHalvesTS = 12;      // LDS stride (floats) of one lane's coefficients
constexpr int kHalvesQC = 128;     // queue slots
constexpr int kHalvesRing = 4;     // factor ring slots (pairs)
constexpr int kHalvesBound = 36;   // floats of a factor entry that the bound reads: L and 1/e
// floats of LDS of a wavefront: coefficients, queue, factor ring (16-byte aligned pieces)
constexpr int kHalvesLds = 64 * kHalvesTS + 9 * kHalvesQC + kHalvesRing * 2 * kHalvesBound;

// One wavefront: 32 rows from row0 of column block blk over seed range `split`.
template <int C, bool POW2>
__device__ __forceinline__ void screen_halves(const EncodeArgs& a, const u32x4* __restrict__ frag, int stride, int blk,
                                              int64_t row0, int split, float* lds) {
  constexpr int PB = 8;
  constexpr int NKS = C / 32;
  constexpr int TS = kHalvesTS;
  constexpr int LS = PB * (PB - 1) / 2;
  constexpr int NF = LS + 2 * PB;   // the whole factor entry (the full score also reads e)
  constexpr int NBD = LS + PB;      // L and 1/e: what the bound reads
  constexpr int QC = kHalvesQC;
  constexpr int QW = PB + 1;        // words per entry: raw b, then seed | owner lane << 24
  static_assert(NBD % 4 == 0 && NF % 4 == 0, "factor pieces are 16 bytes");
  constexpr int NR = kHalvesRing;
  constexpr int NPC = 2 * NBD / 4;   // 16-byte pieces of a pair's two bound entries
  static_assert(NBD == kHalvesBound && QW == 9, "LDS pieces");
  float* const tb = lds;
  float* const qb = tb + 64 * TS;
  float* const fr = qb + QW * QC;  // [slot][seed of the pair][L, 1/e]
  const int lane = threadIdx.x & 63;
  const int nbk_cols = (int)(a.cols / C);
  const int nsplit = a.nsplit;
  const int n_pairs_all = (a.S + 1) / 2;
  const int pp = (n_pairs_all + nsplit - 1) / nsplit;
  const int pair0 = split * pp;
  const int pair1 = pair0 + pp < n_pairs_all ? pair0 + pp : n_pairs_all;
  const int n = lane & 15, g = lane >> 4;

  // u fragments, and each tile's weighted energy sum_j d_j r_j^2 (over the
  // four lanes n, n + 16, n + 32, n + 48 that share a row)
  u32x4 uh[2][NKS], um[2][NKS], ul[2][NKS];
  float en[2];
  load_u_col<C, 2>(a, row0, blk, n, g, uh, um, ul, en);
  const int half = lane >> 5;
  const int64_t my_row = row0 + (lane & 31);
  const bool my_valid = my_row < a.rows;
  const float energy = en[(lane >> 4) & 1];  // this lane's tile, 16 nb + n
  const float qmax = (float)((1 << (a.b - 1)) - 1);
  const float inv_qmax = 1.0f / qmax;
  constexpr float isq = C == 64 ? 0.125f : 0.08838834764831845f;  // 1/sqrt(C)
  float tg0 = -INFINITY, tg1 = -INFINITY;
  uint32_t ts0 = 0, ts1 = 0;  // seed words: seed | kEdge flag
  float thr = -INFINITY;
  // the pruning threshold of this lane's tile: the re-score window below the
  // best over both halves (lane ^ 32), one percent wider, the wide one when
  // that best is a knife edge; in units of the raw bound (C times the bound
  // of the scaled b)
  auto update_thr = [&]() {
    const auto r0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(tg0), __float_as_uint(tg0), false, false);
    const auto r1 = __builtin_amdgcn_permlane32_swap(ts0, ts0, false, false);
    const float og = __uint_as_float(half ? r0[0] : r0[1]);
    const uint32_t ow = half ? r1[0] : r1[1];
    const float best = fmaxf(tg0, og);
    const bool edge = ((tg0 >= og ? ts0 : ow) & kEdge) != 0;
    thr = slack_thr(best - 1.01f * rescore_window(best, energy, edge)) * (float)C;
  };
  int qhead = 0, qtail = 0;  // wavefront-uniform queue counters
  int nscored = 0;
  const uint64_t lt = lane ? (~0ull >> (64 - lane)) : 0ull;
  auto load_factor = [&](int s_, float (&f)[NF], int pieces) {
    const f32x4* fv = reinterpret_cast<const f32x4*>(a.colfac + ((size_t)blk * a.S + s_) * stride);
#pragma unroll
    for (int i = 0; i < NF / 4; ++i) {
      if (i < pieces) {
        const f32x4 v = fv[i];
        f[4 * i] = v[0]; f[4 * i + 1] = v[1]; f[4 * i + 2] = v[2]; f[4 * i + 3] = v[3];
      }
    }
  };
  // The bound's factor entries reach the wavefront through an LDS ring: at
  // the step of pair k every lane loads one 16-byte piece of pair k + 2's two
  // entries (lanes with the same piece load the same one) and stores the
  // piece it loaded at the step before (pair k + 1's); the bound of pair k
  // reads its seed's entry from slot k.  The wavefront barriers of every step
  // order the stores before the reads.
  const int pc = lane % NPC;
  // the piece's seed within its pair and its byte offset in the seed's entry;
  // the block's rows of the table from a wavefront-uniform base
  const int psel = pc / (NBD / 4);
  const uint32_t pofs = 16u * (uint32_t)(pc % (NBD / 4)), strideB = 4u * (uint32_t)stride;
  const char* fac_blk = reinterpret_cast<const char*>(a.colfac + (size_t)blk * a.S * stride);
  auto fac_piece = [&](int pr) -> f32x4 {
    const int s_ = min(2 * pr + psel, a.S - 1);
    return *reinterpret_cast<const f32x4*>(fac_blk + __umul24((uint32_t)s_, strideB) + pofs);
  };
  auto fac_store = [&](int pr, const f32x4& v) {
    *reinterpret_cast<f32x4*>(&fr[(pr & (NR - 1)) * (2 * NBD) + 4 * pc]) = v;
  };
  auto score_round = [&](int cnt) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const bool mine = lane < cnt;
    const int slot = (qhead + lane) & (QC - 1);
    int ol = 0;
    if (mine) {
      float bs[PB];
#pragma unroll
      for (int i = 0; i < PB; ++i) bs[i] = qb[i * QC + slot] * isq;
      const uint32_t word = __float_as_uint(qb[PB * QC + slot]);
      const int es = (int)(word & 0xFFFFu);
      ol = (int)(word >> 24);
      float f[NF];
      load_factor(es, f, NF / 4);
      bool edge;
      const float gsc = screen_score_ldl<PB, POW2, 0>(bs, f, qmax, inv_qmax, &edge);
      qb[slot] = gsc;
      qb[QC + slot] = __uint_as_float((uint32_t)es | (edge ? kEdge : 0u));
    }
    uint64_t mm = __ballot(mine);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
      const uint64_t bal = __ballot((ol >> b) & 1);
      mm &= ((lane >> b) & 1) ? bal : ~bal;
    }
    nscored += __popcll(mm);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    while (__ballot(mm != 0) != 0) {
      if (mm != 0) {
        const int r = (qhead + __builtin_ctzll(mm)) & (QC - 1);
        const float gsc = qb[r];
        const uint32_t sw = __float_as_uint(qb[QC + r]);
        const bool c0 = gsc > tg0, c1 = gsc > tg1;
        tg1 = c0 ? tg0 : (c1 ? gsc : tg1);
        ts1 = c0 ? ts0 : (c1 ? sw : ts1);
        tg0 = c0 ? gsc : tg0;
        ts0 = c0 ? sw : ts0;
        mm &= mm - 1;
      }
    }
    qhead += cnt;
    update_thr();
  };

  const u32x4* fp = frag + (size_t)pair0 * (NKS * 64) + lane;
  auto project = [&](const u32x4 (&F)[NKS], f32x4 (&acc)[2]) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const bf16x8 A = as_bf16x8(F[ks]);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, as_bf16x8(uh[nb][ks]), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, as_bf16x8(um[nb][ks]), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, as_bf16x8(ul[nb][ks]), c, 0, 0, 0);
      }
      acc[nb] = c;
    }
  };
  // rows 4g..4g+3 of the product = (seed g/2 of the pair, columns 4(g&1)..+3)
  // of tiles 16nb + n; lane (seed half, tile) reads them back
  auto stash = [&](const f32x4 (&acc)[2]) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      *reinterpret_cast<f32x4*>(&tb[((g >> 1) * 32 + 16 * nb + n) * TS + 4 * (g & 1)]) = acc[nb];
  };
  u32x4 F[NKS];
  {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) F[ks] = fp[ks * 64];
    f32x4 acc[2];
    project(F, acc);
    stash(acc);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) F[ks] = fp[NKS * 64 + ks * 64];
  }
  fac_store(pair0, fac_piece(pair0));
  f32x4 fnext = fac_piece(pair0 + 1);
  for (int pair = pair0; pair < pair1; ++pair) {
    const int s = 2 * pair + half;
    // pair + 1's pieces (loaded a step ago) into the ring, pair + 2's in flight
    fac_store(pair + 1, fnext);
    fnext = fac_piece(pair + 2);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    float f[NF];
    {
      const float* fe = &fr[(pair & (NR - 1)) * (2 * NBD) + half * NBD];
#pragma unroll
      for (int i = 0; i < NBD / 4; ++i) {
        const f32x4 v = *reinterpret_cast<const f32x4*>(&fe[4 * i]);
        f[4 * i] = v[0]; f[4 * i + 1] = v[1]; f[4 * i + 2] = v[2]; f[4 * i + 3] = v[3];
      }
    }
    float bv[PB];
    {
      const f32x4 b0 = *reinterpret_cast<const f32x4*>(&tb[lane * TS]);
      const f32x4 b1 = *reinterpret_cast<const f32x4*>(&tb[lane * TS + 4]);
      bv[0] = b0[0]; bv[1] = b0[1]; bv[2] = b0[2]; bv[3] = b0[3];
      bv[4] = b1[0]; bv[5] = b1[1]; bv[6] = b1[2]; bv[7] = b1[3];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    f32x4 accN[2];
    project(F, accN);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) F[ks] = fp[(size_t)(pair - pair0 + 2) * (NKS * 64) + ks * 64];
    float wv[PB];
    const float bnd = screen_fwd<PB>(bv, f, wv);
    const bool keep = (int)(bnd > thr) & (int)my_valid & (int)(s < a.S);
    // every lane stores its candidate (raw b), the kept ones first from the
    // tail on, the dropped ones after them (at most 63 wait before a step, so
    // the 64 slots written are free); the tail takes in the kept ones only
    const uint64_t kb = __ballot(keep);
    const int nk = __popcll(kb);
    const int pos = keep ? __popcll(kb & lt) : nk + __popcll(~kb & lt);
    const int qslot = (qtail + pos) & (QC - 1);
#pragma unroll
    for (int i = 0; i < PB; ++i) qb[i * QC + qslot] = bv[i];
    qb[PB * QC + qslot] = __uint_as_float((uint32_t)s | ((uint32_t)lane << 24));
    qtail += nk;
#pragma unroll
    for (int i = 0; i < 24; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
    }
    if (qtail - qhead >= 64) score_round(64);
    stash(accN);
  }
  if (qtail > qhead) score_round(qtail - qhead);
#pragma unroll
  for (int k = 32; k >= 1; k >>= 1) nscored += __shfl_xor(nscored, k, 64);
  if (lane == 0) atomicAdd(a.scored, (unsigned long long)nscored);
  // merge the two halves' lists of each tile: (gain desc, seed asc)
  const float og0 = __shfl(tg0, lane + 32, 64), og1 = __shfl(tg1, lane + 32, 64);
  const uint32_t os0 = (uint32_t)__shfl((int)ts0, lane + 32, 64), os1 = (uint32_t)__shfl((int)ts1, lane + 32, 64);
  if (half == 0 && my_valid) {
    auto better = [](float ga, uint32_t sa, float gb, uint32_t sb) {
      return ga > gb || (ga == gb && list_seed(sa) < list_seed(sb));
    };
    float r0, r1;
    uint32_t q0, q1;
    if (better(tg0, ts0, og0, os0)) {
      r0 = tg0; q0 = ts0;
      const bool m = better(tg1, ts1, og0, os0);
      r1 = m ? tg1 : og0; q1 = m ? ts1 : os0;
    } else {
      r0 = og0; q0 = os0;
      const bool m = better(tg0, ts0, og1, os1);
      r1 = m ? tg0 : og1; q1 = m ? ts0 : os1;
    }
    const int64_t at = ((my_row * nbk_cols + blk) * nsplit + split) * kTop;
    a.top_gain[at + 0] = r0;
    a.top_gain[at + 1] = r1;
    a.top_seed[at + 0] = q0;
    a.top_seed[at + 1] = q1;
  }
}

}  // namespace awsrc
