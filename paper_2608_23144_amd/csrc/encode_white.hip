// Encoder seed search with per-column weights through a whitened basis
// (C = 128, P <= 8, generator version 1).
//
// With G + eps I = L diag(e) L^T of a (column block, seed), the bound that
// decides whether a candidate has to be scored is
//
//   b^T (G + eps I)^-1 b = |M v|^2,   M = diag(e)^-1/2 L^-1 B_s^T D^1/2,   v = D^1/2 r,
//
// and M, whose rows have norm at most one, belongs to the block and the seed
// and not to the tile.  k_whiten writes M as fp16 matrix-core fragments, and
// the screen forms |M v|^2 of a seed pair for 64 tiles with sixteen
// v_mfma_f32_16x16x32_f16, without a triangular solve per candidate.
//
// M and v are rounded to fp16 for this bound only, never for a result: the
// rounding changes |M v| by at most kWhiteSlack |v| (below), the threshold is
// lowered by that much, and every candidate that reaches it is scored from
// fp32 u = d .* r with the fp32 factor, as in the other screens.  So the kept
// lists are those of scoring every candidate, in the best and in the second
// wherever the second lies inside the re-score's window.  (How many candidates
// are scored depends a little on the two wavefronts' timing, what is kept does
// not.)  Column blocks in which a few channels carry most of the weight, and
// those whose weights are not positive numbers, run the other C = 128 screen
// in this kernel (white_takes).
//
// One workgroup = two wavefronts = 64 consecutive rows of one column block.
// Both wavefronts hold v of all 64 tiles (64 VGPRs) and take alternate seed
// pairs, so a fragment read serves 64 tiles: a pair's fragments are 4 KB per
// wavefront and step, and with 32 tiles per read the L1 (64 bytes a cycle)
// would take twice as long as the matrix cores.  u stays in LDS (32 KB, four
// workgroups per CU) for the scoring rounds: the survivors wait in one queue
// per wavefront, and a round takes 64 of them, one per lane, each lane forming
// the P projections of its own (tile, seed) by folding the tile's sign-flipped
// u coordinate bit by coordinate bit (the Sylvester signs of column c are the
// product over the bits of c).
//
// Measured, one decoder layer of a 32B model (seven modules, 3.8 M tiles, S =
// 1024): screen 22.4 -> 11.8 ms, the whole encode 24.6 -> 14.1 ms.  Of the
// 11.8 ms about 7 are the bound (some 500 cycles a step of 128 candidates, of
// which the sixteen matrix instructions take 256 and 65 vector instructions 260:
// with the fragments in L1 it is 0.9 ms less, and neither interleaving the two
// kinds nor reading further ahead gained) and 4.2 the rounds (2% of the
// candidates, some 1,700 vector instructions for 64 of them).  In all it counts
// 144 vector instructions a step.
#include <math.h>

#include "awsrc_internal.h"
#include "mfma_bf16.h"
#include "rescore64.h"
#include "screen_halves.h"

namespace awsrc {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f16x8 as_f16x8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

constexpr int kC = 128;
constexpr int kPB = 8;
constexpr int kWhiteTiles = 64;  // tiles per workgroup
constexpr float kRootC = 0.08838834764831845f;  // 1/sqrt(C)

// Bound on the error of |M~ v~| (M and v rounded to fp16) relative to |v|, for
// the M of the factor as stored in fp32, the one that the scores use:
// |M - M~|_F <= 2^-11 sqrt(8), |M|_2 <= 1 and |v - v~| <= 2^-11 |v| give
// 2^-11 (sqrt(8) + 1) = 1.87e-3; the rest covers the fp32 sums of a product
// (2e-5), the entries of M below fp16's normal range (1e-6) and the forward
// substitution.  Each of that one's at most seven steps a row rounds vectors no
// longer than sqrt(G_pp), and a pivot e_p brings them to the scale of M: in fp32
// 7 sqrt(8) 2^-24 sqrt(G_pp / e_p), 4e-5 at a ratio of kWhiteIll (measured: 4e-6
// there, 1.6e-4 at 2^20, always 1.5e-7 times the root).  Above it, where a few
// channels carry most of a block's weight, the substitution runs in fp64.
constexpr float kWhiteSlack = 2.0e-3f;
constexpr float kWhiteIll = 1024.0f;

// The power of two that brings a vector of squared norm e to [2^9.5, 2^10.5).
__device__ __forceinline__ float vscale(float e) {
  const int x = (int)((__float_as_uint(e) >> 23) & 0xFFu);
  return __uint_as_float((uint32_t)(127 + ((147 - x) >> 1)) << 23);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

// Rows of M at eight coordinates with weights d8: fragments o[p], by forward
// substitution in T.  neg[p]: their signs in column p; f: L packed by rows, then
// diag(e)^-1/2.
template <typename T>
__device__ __forceinline__ void whiten8(const float (&d8)[8], const uint32_t (&neg)[kPB], int P,
                                        const float (&f)[kPB * (kPB - 1) / 2 + kPB], u32x4 (&o)[kPB]) {
  constexpr int PB = kPB, LS = PB * (PB - 1) / 2;
#pragma unroll
  for (int e2 = 0; e2 < 4; ++e2) {
    uint32_t hb[2][PB];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int e = 2 * e2 + h;
      const T sd = __builtin_amdgcn_sqrtf(d8[e]) * kRootC;
      T w[PB];
#pragma unroll
      for (int p = 0; p < PB; ++p) {
        T t = p < P ? (((neg[p] >> e) & 1u) ? -sd : sd) : (T)0;
#pragma unroll
        for (int k = 0; k < p; ++k) t = __builtin_elementwise_fma(-(T)f[ltri(p, k)], w[k], t);
        w[p] = t;
        hb[h][p] = (uint32_t)__half_as_ushort(__float2half_rn((float)(t * (T)f[LS + p])));
      }
    }
#pragma unroll
    for (int p = 0; p < PB; ++p) o[p][e2] = hb[0][p] | (hb[1][p] << 16);
  }
}

// M of column blocks blk0 .. as fragments white[block][pair][ks][lane]: eight
// fp16 of row m = lane % 16 (seed 2 pair + m / 8, column m % 8) at coordinates
// 32 ks + 8 (lane / 16) + e; rows of absent seeds and columns are zero.  One
// thread per (seed, ks, lane / 16).
__global__ __launch_bounds__(256) void k_whiten(EncodeArgs a, int stride, int blk0, u32x4* __restrict__ white) {
  constexpr int C = kC, PB = kPB, NKS = C / 32, LS = PB * (PB - 1) / 2;
  constexpr int TPS = NKS * 4;  // threads per seed
  const int n_pairs = (a.S + 1) / 2;
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int s = i / TPS, ks = (i % TPS) / 4, g = i % 4;
  if (s >= 2 * n_pairs) return;
  const int blk = blk0 + blockIdx.y;
  u32x4* out = white + (((size_t)blockIdx.y * n_pairs + (s >> 1)) * NKS + ks) * 64 + 16 * g + 8 * (s & 1);
  if (s >= a.S) {
#pragma unroll
    for (int p = 0; p < PB; ++p) out[p] = u32x4{0u, 0u, 0u, 0u};
    return;
  }
  const float* fs = a.colfac + ((size_t)blk * a.S + s) * stride;
  float f[LS + PB];
#pragma unroll
  for (int k = 0; k < (LS + PB) / 4; ++k) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(fs + 4 * k);
    f[4 * k] = v[0]; f[4 * k + 1] = v[1]; f[4 * k + 2] = v[2]; f[4 * k + 3] = v[3];
  }
  float most = f[LS];  // the largest 1 / e
#pragma unroll
  for (int p = 1; p < PB; ++p) most = p < a.P ? fmaxf(most, f[LS + p]) : most;
  const bool ill = most > kWhiteIll * f[LS];
#pragma unroll
  for (int p = 0; p < PB; ++p) f[LS + p] = __builtin_amdgcn_sqrtf(f[LS + p]);
  const int j0 = 32 * ks + 8 * g;
  uint32_t neg[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p)
    neg[p] = p < a.P ? (uint32_t)(a.basis.mask[((size_t)s * a.P + p) * 2 + (j0 >> 6)] >> (j0 & 63)) & 0xFFu : 0u;
  const float* dp = a.d + (int64_t)blk * C + j0;
  float d8[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) d8[e] = dp[e];
  u32x4 o[PB];
  if (ill) whiten8<double>(d8, neg, a.P, f, o);
  else whiten8<float>(d8, neg, a.P, f, o);
#pragma unroll
  for (int p = 0; p < PB; ++p) out[p] = o[p];
}

// two wavefronts per SIMD: at most 256 VGPRs, and the LDS allows four workgroups per CU
// (one 64-bit value waits in scratch memory from before the loop over the seeds
// until after it)
template <bool POW2>
__global__ __launch_bounds__(128, 2) void k_screen_white(EncodeArgs a, const u32x4* __restrict__ white, int stride,
                                                         int blk0) {
  constexpr int C = kC, PB = kPB, NKS = C / 32, NT = kWhiteTiles;
  constexpr int LS = PB * (PB - 1) / 2, NF = LS + 2 * PB;
  constexpr int QC = 256;  // queue slots of a wavefront: at most 63 entries wait before a step of 128 candidates
  __shared__ __attribute__((aligned(16))) float lu[C * NT];  // u, [coordinate][tile]
  static_assert(2 * kHalvesLds <= C * NT && kHalvesLds % 4 == 0, "room for both wavefronts of the other screen");
  __shared__ uint32_t queue[2][QC];                          // seed | tile << 16
  __shared__ float res_g[2][64];
  __shared__ uint32_t res_s[2][64];
  __shared__ float s_thr[2][NT];
  __shared__ uint64_t s_best[2][NT];  // each wavefront's best score of a tile, edge flag above it
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int nbk_cols = (int)(a.cols / C);
  const int nsplit = a.nsplit;
  // workgroups go to the 8 XCDs round-robin; each XCD takes a contiguous run
  // of work items in column-block-major order, so that the row groups of a
  // block read its M (2 KB a seed) from one L2
  const int64_t nwg = gridDim.x;
  const int64_t xcd = blockIdx.x % 8, q8 = nwg / 8, rem = nwg % 8;
  const int64_t item = xcd * q8 + (xcd < rem ? xcd : rem) + blockIdx.x / 8;
  const int nrg = (int)((a.rows + NT - 1) / NT);
  const int split = (int)(item % nsplit);
  const int64_t rest = item / nsplit;
  const int lblk = (int)(rest / nrg);
  const int blk = blk0 + lblk;
  const int64_t row0 = (rest % nrg) * NT;
  const int n_pairs = (a.S + 1) / 2;
  const int pp = (n_pairs + nsplit - 1) / nsplit;
  const int pair0 = split * pp;
  const int pair1 = pair0 + pp < n_pairs ? pair0 + pp : n_pairs;
  const int n = lane & 15, g = lane >> 4;
  if (!white_takes(a.d + (int64_t)blk * C)) {  // both wavefronts alike
    if (row0 + 32 * wv < a.rows)
      screen_halves<C, POW2>(a, static_cast<const u32x4*>(a.frag), stride, blk, row0 + 32 * wv, split,
                             lu + wv * kHalvesLds);
    return;
  }

  // v fragments (coordinates 32 ks + 8 g .. + 7 of tiles 16 nb + n), scaled
  // per tile by a power of two so that |v| lies in [2^9.5, 2^10.5), and u to LDS
  // (each wavefront stores half of the tiles)
  u32x4 vf[4][NKS];
  float en[4];
  uint32_t finite = 0;  // bit nb: tile 16 nb + n has no infinite or NaN u
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int64_t row = row0 + 16 * nb + n;
    const bool valid = row < a.rows;
    int64_t o[2 * NKS];
    gf32x4 dv[2 * NKS];
#pragma unroll
    for (int q = 0; q < 2 * NKS; ++q) {
      const int64_t at = (int64_t)blk * C + 32 * (q >> 1) + 8 * g + 4 * (q & 1);
      o[q] = (valid ? row : a.rows - 1) * a.cols + at;
      dv[q] = gload4f(a.d + at);
    }
    float rv[2 * NKS][4];
    load_residual4<2 * NKS>(a.W, a.w_dtype, a.W0, o, rv);
    float e = 0.0f, z = 0.0f;
#pragma unroll
    for (int q = 0; q < 2 * NKS; ++q)
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float r = valid ? rv[q][k] : 0.0f;
        const float u = valid ? dv[q][k] * r : 0.0f;
        rv[q][k] = r;
        e = fmaf(u, r, e);
        z = fmaf(u, 0.0f, z);
        if (wv == (nb >> 1)) lu[(32 * (q >> 1) + 8 * g + 4 * (q & 1) + k) * NT + 16 * nb + n] = u;
      }
    e += __shfl_xor(e, 16, 64);
    e += __shfl_xor(e, 32, 64);
    z += __shfl_xor(z, 16, 64);
    z += __shfl_xor(z, 32, 64);
    finite |= (uint32_t)(z == 0.0f) << nb;
    en[nb] = e;
    const float sc = vscale(e);
#pragma unroll
    for (int q = 0; q < 2 * NKS; ++q)
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        uint32_t hb[2];
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const int k = 2 * k2 + x;
          hb[x] = (uint32_t)__half_as_ushort(__float2half_rn(__builtin_amdgcn_sqrtf(dv[q][k]) * (rv[q][k] * sc)));
        }
        vf[nb][q >> 1][2 * (q & 1) + k2] = hb[0] | (hb[1] << 16);
      }
    // the packed form here and now: left to itself the compiler carries the
    // fp32 values of all four groups to the first use, and spills
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(vf[nb][ks]));
    __builtin_amdgcn_sched_barrier(0);
  }
  // lane = tile where the lists are kept
  const float energy = g == 0 ? en[0] : g == 1 ? en[1] : g == 2 ? en[2] : en[3];
  const float vsc = vscale(energy);
  const float slack_v = kWhiteSlack * sqrtf(energy);
  const bool my_valid = row0 + lane < a.rows;
  // no score of a tile with an infinite or NaN u is a number: it keeps the empty list
  const bool my_screened = my_valid && ((finite >> g) & 1u);
  const float qmax = (float)((1 << (a.b - 1)) - 1);
  const float inv_qmax = 1.0f / qmax;
  float tg0 = -INFINITY, tg1 = -INFINITY;
  uint32_t ts0 = 0, ts1 = 0;  // seed words: seed | kEdge flag
  s_best[wv][lane] = (uint64_t)__float_as_uint(-INFINITY);
  __syncthreads();

  // where candidates are screened: lane (n, g) holds seed g / 2 of the pair
  // for tiles 16 nb0 + n and 16 (nb0 + 1) + n
  const int sh = g >> 1, nb0 = 2 * (g & 1);
  const uint32_t tile0 = 16 * nb0 + n;
  // rows past the end are never kept
  float thr2[2] = {row0 + tile0 < a.rows && ((finite >> nb0) & 1u) ? -1.0f : INFINITY,
                   row0 + tile0 + 16 < a.rows && ((finite >> nb0) & 2u) ? -1.0f : INFINITY};
  int qhead = 0, qtail = 0;  // wavefront-uniform queue counters
  unsigned long long nscored = 0;
  const int P = a.P;
  const uint32_t s_end = (uint32_t)(2 * pair1 < a.S ? 2 * pair1 : a.S);

  auto score_round = [&](int cnt) {
    wave_sync();
    const bool mine = lane < cnt;
    uint32_t et = 0;
    int es = 0;
    float bs[PB], gsc = 0.0f;
    bool edge = false;
    auto score = [&]() {
      const f32x4* fv = reinterpret_cast<const f32x4*>(a.colfac + ((size_t)blk * a.S + es) * stride);
      float f[NF];
#pragma unroll
      for (int i = 0; i < NF / 4; ++i) {
        const f32x4 v = fv[i];
        f[4 * i] = v[0]; f[4 * i + 1] = v[1]; f[4 * i + 2] = v[2]; f[4 * i + 3] = v[3];
      }
      gsc = screen_score_ldl<PB, POW2, 0>(bs, f, qmax, inv_qmax, &edge);
    };
    if (mine) {
      const uint32_t word = queue[wv][(qhead + lane) & (QC - 1)];
      es = (int)(word & 0xFFFFu);
      et = word >> 16;
      const uint32_t* sgw = reinterpret_cast<const uint32_t*>(a.basis.sign + (size_t)es * 2);
      uint32_t sg[NKS];
#pragma unroll
      for (int c = 0; c < NKS; ++c) sg[c] = sgw[c];
      const uint64_t cw = *reinterpret_cast<const uint64_t*>(a.basis.col + (size_t)es * kMaxP);
      // b_p = sum_j (-1)^popc(j & c_p) sigma_j u_j, 16 coordinates at a time:
      // a level per bit of the coordinate halves the values, with the sign
      // that the bit of c_p gives
      float b[PB];
      auto sign_of = [&](int p, int k) {  // +-1 by bit k of c_p
        const uint32_t h = (uint32_t)(cw >> (32 * (p >> 2)));
        return __uint_as_float((h << (31 - 8 * (p & 3) - k) & 0x80000000u) | 0x3F800000u);
      };
      float sf[PB][4];
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int k = 0; k < 4; ++k) sf[p][k] = sign_of(p, k);
      // the blocks in Gray-code order, last first: neighbours differ in one
      // bit of the block number, so each joins with one fused multiply-add
#pragma unroll
      for (int i8 = C / 16 - 1; i8 >= 0; --i8) {
        const int c = i8 ^ (i8 >> 1);
        float x[16];
#pragma unroll
        for (int i = 0; i < 16; ++i)
          x[i] = __uint_as_float(__float_as_uint(lu[(16 * c + i) * NT + et]) ^
                                 (sg[c >> 1] << (31 - (16 * (c & 1) + i)) & 0x80000000u));
#pragma unroll
        for (int p = 0; p < PB; ++p) {
          float y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) y[i] = fmaf(sf[p][3], x[i + 8], x[i]);
#pragma unroll
          for (int k = 2; k >= 0; --k)
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (i < (1 << k)) y[i] = fmaf(sf[p][k], y[i + (1 << k)], y[i]);
          if (i8 == C / 16 - 1) {
            b[p] = y[0];
          } else {
            // the Gray codes of i8 and i8 + 1 differ in the lowest set bit of i8 + 1
            b[p] = fmaf(sign_of(p, 4 + __builtin_ctz(i8 + 1)), b[p], y[0]);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int p = 0; p < PB; ++p) bs[p] = p < P ? b[p] * kRootC : 0.0f;
      score();
    }
    // A candidate on a knife edge (a few in a thousand) is scored again from
    // the projection that k_screen_mfma_halves forms, bit by bit, so that the
    // two screens take the same side: a differing rounding costs up to a
    // percent of the score and can drop a seed out of the list.  Every column
    // of the product is the same tile.
    if (const uint64_t edges = __ballot(edge)) {
      for (uint64_t em = edges; em; em &= em - 1) {
        const int l = __builtin_ctzll(em);
        const int t1 = __builtin_amdgcn_readlane((int)et, l), s1 = __builtin_amdgcn_readlane(es, l);
        const int p1 = lane & 7;
        f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
          float uk[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) uk[k] = lu[(32 * ks + 8 * g + k) * NT + t1];
          u32x4 h, m, lo, A;
          split3(uk, h, m, lo);
          const uint64_t* mk = a.basis.mask + ((size_t)s1 * P + (p1 < P ? p1 : 0)) * 2;
          const uint32_t bits = (uint32_t)(mk[ks >> 1] >> (32 * (ks & 1) + 8 * g));
#pragma unroll
          for (int q = 0; q < 4; ++q)
            A[q] = p1 < P ? 0x3F803F80u | ((bits >> (2 * q)) & 1u) << 15 | ((bits >> (2 * q + 1)) & 1u) << 31 : 0u;
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A), as_bf16x8(h), c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A), as_bf16x8(m), c, 0, 0, 0);
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A), as_bf16x8(lo), c, 0, 0, 0);
        }
#pragma unroll
        for (int p = 0; p < PB; ++p) {
          const float v = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(c[p & 3]), 16 * (p >> 2)));
          bs[p] = lane == l ? v * kRootC : bs[p];
        }
      }
      if ((edges >> lane) & 1) score();
    }
    if (mine) {
      res_g[wv][lane] = gsc;
      res_s[wv][lane] = (uint32_t)es | (edge ? kEdge : 0u);
    }
    // the round's lanes whose entry is of this lane's tile
    uint64_t mm = __ballot(mine);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const uint64_t bal = __ballot((et >> k) & 1);
      mm &= ((lane >> k) & 1) ? bal : ~bal;
    }
    nscored += cnt;
    wave_sync();
    while (__ballot(mm != 0) != 0) {
      if (mm != 0) {
        const int r = __builtin_ctzll(mm);
        const float gsc = res_g[wv][r];
        const uint32_t sw = res_s[wv][r];
        const bool c0 = gsc > tg0, c1 = gsc > tg1;
        tg1 = c0 ? tg0 : (c1 ? gsc : tg1);
        ts1 = c0 ? ts0 : (c1 ? sw : ts1);
        tg0 = c0 ? gsc : tg0;
        ts0 = c0 ? sw : ts0;
        mm &= mm - 1;
      }
    }
    qhead += cnt;
    // The threshold of this lane's tile: the re-score window below the best
    // of both wavefronts' lists so far (the other's only rises, and one 64-bit
    // access carries its score and its edge flag), one percent wider, the wide
    // one when that best is a knife edge; lowered by the fp16 slack.
    __hip_atomic_store(&s_best[wv][lane], (uint64_t)__float_as_uint(tg0) | (uint64_t)(ts0 & kEdge) << 32,
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const uint64_t ob = __hip_atomic_load(&s_best[wv ^ 1][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const float og = __uint_as_float((uint32_t)ob);
    const float best = fmaxf(tg0, og);
    const bool bedge = (tg0 >= og ? (ts0 & kEdge) : (uint32_t)(ob >> 32)) != 0;
    const float thr = slack_thr(best - 1.01f * rescore_window(best, energy, bedge));
    const float x = thr >= 0.0f ? sqrtf(thr) - slack_v : -1.0f;
    s_thr[wv][lane] = !my_screened ? INFINITY : x >= 0.0f ? (x * vsc) * (x * vsc) : -1.0f;
    wave_sync();
    thr2[0] = s_thr[wv][tile0];
    thr2[1] = s_thr[wv][tile0 + 16];
  };

  const u32x4* fp = white + (size_t)lblk * n_pairs * (NKS * 64) + lane;
  auto load_frag = [&](int pair, u32x4 (&F)[NKS]) {
    const u32x4* f0 = fp + (size_t)(pair < n_pairs ? pair : n_pairs - 1) * (NKS * 64);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) F[ks] = f0[ks * 64];
  };
  auto project = [&](const u32x4 (&F)[NKS], f32x4 (&acc)[4]) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) acc[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int nb = 0; nb < 4; ++nb)
        acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(F[ks]), as_f16x8(vf[nb][ks]), acc[nb], 0, 0, 0);
  };
  // rows 4g..4g+3 of the product = (seed g / 2 of the pair, columns 4 (g & 1)
  // .. + 3) of tiles 16 nb + n: half of a candidate's |M v|^2 in lane rows g
  // and g ^ 1, which trade halves
  auto halves = [&](const f32x4 (&acc)[4], float (&sq)[4]) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
      sq[nb] = fmaf(acc[nb][0], acc[nb][0], acc[nb][1] * acc[nb][1]) +
               fmaf(acc[nb][2], acc[nb][2], acc[nb][3] * acc[nb][3]);
  };
  // Fragments are read two steps ahead, into two register sets that take
  // turns.  A round runs as soon as 64 candidates wait, so the first step's
  // scores are there before the second step is bounded.
  auto step = [&](int pair, u32x4 (&F)[NKS]) {
    f32x4 acc[4];
    project(F, acc);
    load_frag(pair + 4, F);
    float sq[4];
    halves(acc, sq);
    bool keep[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(sq[t]), __float_as_uint(sq[t + 2]), false, false);
      keep[t] = !(__uint_as_float(r[0]) + __uint_as_float(r[1]) <= thr2[t]);  // NaN is kept
    }
    const uint32_t s = 2 * pair + sh;
    if (__ballot(keep[0] | keep[1]) != 0) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const bool k = (int)keep[t] & (int)(s < s_end) & (int)(thr2[t] < INFINITY);
        const uint64_t kb = __ballot(k);
        const int pos = __builtin_amdgcn_mbcnt_hi((uint32_t)(kb >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)kb, 0u));
        if (k) queue[wv][(qtail + pos) & (QC - 1)] = s | (tile0 + 16 * t) << 16;
        qtail += __popcll(kb);
      }
    }
  };
  u32x4 FA[NKS], FB[NKS];
  load_frag(pair0 + wv, FA);
  load_frag(pair0 + wv + 2, FB);
  for (int pair = pair0 + wv; pair < pair1; pair += 4) {
    step(pair, FA);
    while (qtail - qhead >= 64) score_round(64);
    step(pair + 2, FB);
    const int least = pair + 4 < pair1 ? 64 : 1;  // the last step empties the queue
    while (qtail - qhead >= least) score_round(qtail - qhead < 64 ? qtail - qhead : 64);
  }
  if (lane == 0) atomicAdd(a.scored, nscored);

  // the second wavefront's lists to the first, which merges: (gain desc, seed asc)
  __syncthreads();
  if (wv == 1) {
    lu[lane] = tg0;
    lu[NT + lane] = tg1;
    lu[2 * NT + lane] = __uint_as_float(ts0);
    lu[3 * NT + lane] = __uint_as_float(ts1);
  }
  __syncthreads();
  if (wv == 0 && my_valid) {
    const float og0 = lu[lane], og1 = lu[NT + lane];
    const uint32_t os0 = __float_as_uint(lu[2 * NT + lane]), os1 = __float_as_uint(lu[3 * NT + lane]);
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
    const int64_t at = (((row0 + lane) * nbk_cols + blk) * nsplit + split) * kTop;
    a.top_gain[at + 0] = r0;
    a.top_gain[at + 1] = r1;
    a.top_seed[at + 0] = q0;
    a.top_seed[at + 1] = q1;
  }
}

// M of every block and seed takes 2 C P' bytes (P' = 8); more column blocks
// than fit kWhiteBytes are screened in several launches.
constexpr size_t kWhiteBytes = (size_t)128 << 20;

// Where the whitened screen is the faster one.  Its table costs S C P / 2
// fused multiply-adds and 2 KB a seed per column block, whatever the rows; its
// scoring rounds cost more than k_screen_mfma_halves' (which has the fp32
// projections at hand), and every tile's first four seeds are scored.  Whole
// encode calls, that screen against this one, us: 5120 x 5120 S = 1024 1360 ->
// 807, S = 512 768 -> 580, S = 256 478 -> 459, S = 128 332 -> 389; 2048 x 5120
// S = 512 378 -> 320, S = 256 245 -> 252; 1024 x 5120 S = 1024 363 -> 323,
// S = 512 229 -> 250; 512 x 11008 S = 1024 373 -> 407; 512 x 27648 S = 1024
// 809 -> 993.  So: 256 seeds, 1024 rows and 2^25 candidates.
bool white_supported(int C, int P, int S, int d_mode, int gen_version, int64_t rows, int64_t cols) {
  return C == kC && P <= kPB && d_mode == AWSRC_D_PER_COL && gen_version == 1 && S >= 256 && rows >= 1024 &&
         rows * (cols / C) * S >= ((int64_t)1 << 25);
}

static size_t white_block_bytes(int S) { return (size_t)((S + 1) / 2) * (kC / 32) * 64 * 16; }

static int64_t white_blocks(int S, int64_t nb) {
  int64_t n = (int64_t)(kWhiteBytes / white_block_bytes(S));
  if (n < 1) n = 1;
  return n < nb ? n : nb;
}

size_t white_bytes(int S, int64_t cols) { return (size_t)white_blocks(S, cols / kC) * white_block_bytes(S); }

template <bool POW2>
static hipError_t run_white(const EncodeArgs& a, void* ws, hipStream_t st) {
  const int64_t nb = a.cols / kC, step = white_blocks(a.S, nb);
  u32x4* white = static_cast<u32x4*>(ws);
  const int64_t nrg = (a.rows + kWhiteTiles - 1) / kWhiteTiles;
  const int threads = 2 * ((a.S + 1) / 2) * (kC / 32) * 4;
  for (int64_t b0 = 0; b0 < nb; b0 += step) {
    const int64_t n = nb - b0 < step ? nb - b0 : step;
    hipLaunchKernelGGL(k_whiten, dim3((unsigned)((threads + 255) / 256), (unsigned)n), dim3(256), 0, st, a,
                       colfac_stride(kPB), (int)b0, white);
    hipLaunchKernelGGL((k_screen_white<POW2>), dim3((unsigned)(n * nrg * a.nsplit)), dim3(128), 0, st, a, white,
                       colfac_stride(kPB), (int)b0);
  }
  return hipGetLastError();
}

hipError_t launch_white_screen(const EncodeArgs& a, void* ws, hipStream_t st) {
  const hipError_t e = launch_mfma_frags(a.basis, kC, a.P, a.S, a.frag, st);  // for the blocks that white_takes leaves
  if (e != hipSuccess) return e;
  return a.scale_fmt == AWSRC_SCALE_POW2 ? run_white<true>(a, ws, st) : run_white<false>(a, ws, st);
}

}  // namespace awsrc
