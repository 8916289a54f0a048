// Encoder screen for per-element weights with the seeded coordinate
// permutation (generator version 2), C = 64, P <= 8, every module in one
// launch.
//
// With the permutation a tile's Gram entries are no longer gathers from one
// transform of its weights: G_pq = sum_j d_j B[j,p] B[j,q] has other signs for
// every seed.  They are a matrix product like the projections, d (the same
// for every seed) against the +-1 products of two sign columns, so both run
// on the matrix cores here, from exact three-way bf16 splits of u = d .* r
// and of d.
//
//   * The 16 rows of a product are 4 seeds x 4 entries, so that lane (tile n,
//     g) receives the four entries of seed 4 R + g: two products for b, seven
//     for the 28 Gram entries (each 2 K steps x 3 parts).  Lane (n, g) then
//     owns one candidate, tile n and seed 4 R + g, without any exchange.
//   * The +-1 rows of four seeds (18 KB) are expanded in LDS by the workgroup,
//     one group ahead, from 64 bytes of sign patterns per seed: the byte of
//     eight coordinates (or the XOR of two columns' bytes) looks up its eight
//     bf16 signs.  Four wavefronts (64 rows of one column block) share them;
//     stored in memory they would take 4.6 KB per seed.
//   * Every candidate gets the LDL^T factor and its exact bound, as in the
//     version-1 screen; when some lane's bound reaches the re-score window of
//     its tile's best, the wavefront scores its candidates, the factors being
//     in registers (a queue entry would have to carry all 44 of them).
//
// What bounds it: the vector ALUs, 327 instructions per 64 candidates (the factor
// and bound about 200 of them, the expansion and the scoring), beside 54 matrix
// instructions; the two take turns more than they overlap (0.31 and 0.21 of
// 0.52 ms).  Attention projections of a 3B layer (9.4 M weights, S = 256), whole
// encode: 12.19 ms on the general vector screen (a transform of the permuted
// weights per candidate), 0.57 ms here.
#include <math.h>

#include "awsrc_internal.h"
#include "mfma_bf16.h"
#include "rescore64.h"

namespace awsrc {

namespace {

constexpr int kC = 64;
constexpr int kPB = 8;
constexpr int kWaves = kPermRows / 16;
constexpr int kTabs = 9;  // row tables per four seeds: two of b, seven of Gram entries

// The other lane's value, lanes 16 and 32 apart.
__device__ __forceinline__ uint32_t xor16(uint32_t x, int g) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return (g & 1) ? r[0] : r[1];
}
__device__ __forceinline__ uint32_t xor32(uint32_t x, int g) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  return (g & 2) ? r[0] : r[1];
}
__device__ __forceinline__ float xorf(float x, int g, bool far) {
  return __uint_as_float(far ? xor32(__float_as_uint(x), g) : xor16(__float_as_uint(x), g));
}

}  // namespace

template <bool POW2, bool FULLP>
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(3)))
void k_screen_perm64(EncodeArgs a, ModEntry one, const ModEntry* __restrict__ mods, int n_mods) {
  constexpr int PB = kPB, NL = PB * (PB - 1) / 2, NF = NL + 2 * PB;
  __shared__ u32x4 af[2][kTabs * 2][64];  // row tables of a group of four seeds: [table, K step][lane]
  __shared__ u32x4 lut[256];              // bit i of the index set: element i is -1, else +1
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int n = lane & 15, g = lane >> 4;
  const int64_t item = blockIdx.x;
  ModEntry md = one;
  if (n_mods > 1) md = mods[find_module<&ModEntry::item2_off>(mods, n_mods, item)];
  const int nbk = (int)(md.cols / kC);
  const int64_t local = item - md.item2_off;
  const int blk = (int)(local % nbk);
  const int64_t row = (local / nbk) * kPermRows + 16 * wv + n;
  const bool valid = row < md.rows;
  {
    u32x4 w;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      w[d] = 0x3F803F80u | (((uint32_t)tid >> (2 * d)) & 1u) << 15 | (((uint32_t)tid >> (2 * d + 1)) & 1u) << 31;
    lut[tid] = w;
  }
  // u and d operands: coordinates 32 ks + 8 g .. + 7 of tile n, in three parts
  // each; u / sqrt(C) and d / C (exact), rows past the end repeat the last one
  u32x4 up[2][3], dp[2][3];
  float energy = 0.0f, d0 = 0.0f;
  {
    int64_t o[4];
    const int64_t base = (valid ? row : md.rows - 1) * md.cols + (int64_t)blk * kC + 8 * g;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      o[2 * ks] = base + 32 * ks;
      o[2 * ks + 1] = base + 32 * ks + 4;
    }
    gf32x4 dv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) dv[c] = gload4f(md.d + o[c]);
    float rv[4][4];
    load_residual4<4>(md.W, a.w_dtype, md.W0, o, rv);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      float u[8], dd[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = dv[2 * ks + (e >> 2)][e & 3], r = rv[2 * ks + (e >> 2)][e & 3];
        u[e] = 0.125f * (d * r);
        dd[e] = d * (1.0f / kC);
        energy = fmaf(d * r, r, energy);
        d0 += dd[e];
      }
      split3(u, up[ks][0], up[ks][1], up[ks][2]);
      split3(dd, dp[ks][0], dp[ks][1], dp[ks][2]);
    }
    energy += xorf(energy, g, false);
    energy += xorf(energy, g, true);
    d0 += xorf(d0, g, false);
    d0 += xorf(d0, g, true);
  }
  const int P = a.P, nR = (a.S + 3) / 4;
  const float qmax = (float)((1 << (a.b - 1)) - 1);
  const float inv_qmax = 1.0f / qmax;
  const float diag = fmaf((float)a.lambda, d0, d0);  // G_pp + eps

  // This thread's part of the expansion: rows lane % 16 of the tables
  // (tid >> 7) + 2 k, K step (tid >> 6) & 1: coordinate byte 4 ks + g of seed
  // (lane % 16) / 4, columns pa and pb (pb none for the tables of b).
  constexpr int NE = (kTabs + 1) / 2;
  const int eks = wv & 1, eq = n >> 2, ek = n & 3;
  uint32_t psh[NE];  // shifts 8 pa | 8 pb << 8 | second column present << 16 | row live << 17
#pragma unroll
  for (int k = 0; k < NE; ++k) {
    const int tb = (wv >> 1) + 2 * k;
    int pa, pb = 0;
    if (tb < 2) {
      pa = 4 * tb + ek;
    } else {
      const int e = 4 * (tb - 2) + ek;
      pa = 1;
      while (ltri(pa + 1, 0) <= e) ++pa;
      pb = e - ltri(pa, 0);
    }
    psh[k] = (uint32_t)(8 * (pa & 7)) | (uint32_t)(8 * pb) << 8 | (tb < 2 ? 0u : 1u << 16) |
             (tb < kTabs && (FULLP || pa < P) ? 1u << 17 : 0u);
  }
  auto seed_bytes = [&](int R) -> uint64_t {
    const int s = min(4 * R + eq, a.S - 1);
    return a.basis.sbytes(s)[4 * eks + g];
  };
  auto expand = [&](uint64_t m8, u32x4 (&dst)[kTabs * 2][64]) {
#pragma unroll
    for (int k = 0; k < NE; ++k) {
      const int tb = (wv >> 1) + 2 * k;
      if (tb >= kTabs) break;
      const uint32_t xa = (uint32_t)(m8 >> (psh[k] & 0xFFu)) & 0xFFu;
      const uint32_t xb = (uint32_t)(m8 >> ((psh[k] >> 8) & 0xFFu)) & 0xFFu;
      u32x4 w = lut[xa ^ ((psh[k] & (1u << 16)) ? xb : 0u)];
      if (!FULLP && !(psh[k] & (1u << 17))) w = u32x4{0, 0, 0, 0};
      dst[2 * tb + eks][lane] = w;
    }
  };

  // this lane's top two (its seeds increase, so strict comparisons keep the
  // earlier seed first among equal scores) and its tile's pruning threshold:
  // the re-score window below the best over the tile's four lanes, one percent
  // wider, as in the version-1 screen
  float tg0 = -INFINITY, tg1 = -INFINITY, thr = -INFINITY;
  uint32_t ts0 = 0, ts1 = 0;
  int nscored = 0;
  __syncthreads();  // lut
  expand(seed_bytes(0), af[0]);
  uint64_t m8 = seed_bytes(1);
  for (int R = 0; R < nR; ++R) {
    __syncthreads();  // af[R & 1] is written, and every wavefront is done with the other one
    const u32x4(&A)[kTabs * 2][64] = af[R & 1];
    f32x4 acc[kTabs];
#pragma unroll
    for (int tb = 0; tb < kTabs; ++tb) {
      f32x4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const bf16x8 w = as_bf16x8(A[2 * tb + ks][lane]);
#pragma unroll
        for (int k = 0; k < 3; ++k)
          c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, as_bf16x8(tb < 2 ? up[ks][k] : dp[ks][k]), c, 0, 0, 0);
      }
      acc[tb] = c;
    }
    if (R + 1 < nR) expand(m8, af[(R + 1) & 1]);
    m8 = seed_bytes(R + 2);
    float gq[NL], b[PB], f[NF], w[PB];
#pragma unroll
    for (int e = 0; e < NL; ++e) gq[e] = acc[2 + e / 4][e % 4];
#pragma unroll
    for (int p = 0; p < PB; ++p) b[p] = acc[p / 4][p % 4];
    screen_factor<PB, FULLP>(gq, diag, P, f);
    const float bnd = screen_fwd<PB>(b, f, w);
    const int s = 4 * R + g;
    const bool keep = (int)(bnd > thr) & (int)valid & (int)(s < a.S);
    if (__ballot(keep) != 0) {
      bool edge;
      const float gain = screen_gain_w<PB, POW2, 0>(w, f, qmax, inv_qmax, &edge);
      const uint32_t sw = (uint32_t)s | (edge ? kEdge : 0u);
      const bool c0 = keep && gain > tg0, c1 = keep && gain > tg1;
      tg1 = c0 ? tg0 : (c1 ? gain : tg1);
      ts1 = c0 ? ts0 : (c1 ? sw : ts1);
      tg0 = c0 ? gain : tg0;
      ts0 = c0 ? sw : ts0;
      nscored += keep;
      float best = tg0;
      uint32_t bw = ts0;
#pragma unroll
      for (int far = 0; far < 2; ++far) {
        const float og = xorf(best, g, far);
        const uint32_t ow = far ? xor32(bw, g) : xor16(bw, g);
        bw = best >= og ? bw : ow;
        best = fmaxf(best, og);
      }
      thr = slack_thr(best - 1.01f * rescore_window(best, energy, (bw & kEdge) != 0));
    }
  }
#pragma unroll
  for (int k = 32; k >= 1; k >>= 1) nscored += __shfl_xor(nscored, k, 64);
  if (lane == 0) atomicAdd(a.scored, (unsigned long long)nscored);
  // merge the tile's four lists: (gain desc, seed asc)
  auto better = [](float ga, uint32_t sa, float gb, uint32_t sb) {
    return ga > gb || (ga == gb && list_seed(sa) < list_seed(sb));
  };
#pragma unroll
  for (int far = 0; far < 2; ++far) {
    const float og0 = xorf(tg0, g, far), og1 = xorf(tg1, g, far);
    const uint32_t os0 = far ? xor32(ts0, g) : xor16(ts0, g), os1 = far ? xor32(ts1, g) : xor16(ts1, g);
    const bool mine = better(tg0, ts0, og0, os0);
    const bool second = mine ? better(tg1, ts1, og0, os0) : better(tg0, ts0, og1, os1);
    const float n1 = mine ? (second ? tg1 : og0) : (second ? tg0 : og1);
    const uint32_t m1 = mine ? (second ? ts1 : os0) : (second ? ts0 : os1);
    tg0 = mine ? tg0 : og0;
    ts0 = mine ? ts0 : os0;
    tg1 = n1;
    ts1 = m1;
  }
  if (g == 0 && valid) {
    const int64_t at = (md.tile_off + row * nbk + blk) * kTop;
    *reinterpret_cast<float2*>(a.top_gain + at) = make_float2(tg0, tg1);
    *reinterpret_cast<uint2*>(a.top_seed + at) = make_uint2(ts0, ts1);
  }
}

bool perm_batched_supported(int C, int P, int d_mode, int gen_version) {
  return C == kC && P <= kPB && d_mode == AWSRC_D_PER_ELEM && gen_version == 2;
}

hipError_t launch_perm_screen(const EncodeArgs& a, const ModEntry& one, const ModEntry* mods, int n_mods,
                              int64_t items2, hipStream_t st) {
  const dim3 grid((unsigned)items2), blk(64 * kWaves);
  if (a.scale_fmt == AWSRC_SCALE_POW2) {
    if (a.P == kPB) hipLaunchKernelGGL((k_screen_perm64<true, true>), grid, blk, 0, st, a, one, mods, n_mods);
    else hipLaunchKernelGGL((k_screen_perm64<true, false>), grid, blk, 0, st, a, one, mods, n_mods);
  } else {
    if (a.P == kPB) hipLaunchKernelGGL((k_screen_perm64<false, true>), grid, blk, 0, st, a, one, mods, n_mods);
    else hipLaunchKernelGGL((k_screen_perm64<false, false>), grid, blk, 0, st, a, one, mods, n_mods);
  }
  return hipGetLastError();
}

}  // namespace awsrc
