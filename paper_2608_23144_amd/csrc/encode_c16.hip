// Encoder seed search for C = 16, P <= 4 (the paper's operating point is
// (C, P, b, S) = (16, 4, 4, 16)): screen and fp64 re-score of every tile of
// every module in one launch, for both weight modes and both generator
// versions.
//
// What bounds it: vector issue.  With per-element weights it counts 302 vector
// instructions per 64 candidates, of them some 130 the scoring chain of Eq. (3)
// and Sec. 3.2, the rest loads, knife edges and the re-score; at four cycles each
// that is the launch's time.  The projections and the Gram entries are left to
// the matrix cores (6 instructions per 64 candidates).
//
//   * Tiles are 16 consecutive weights, so a module is one linear array of
//     them; a wavefront takes 64 consecutive tiles and reads them with
//     16-byte loads, two lanes per tile.
//   * u = d .* r and d are split exactly into three bf16 parts.  K = 32 of a
//     v_mfma_f32_16x16x32_bf16 holds the 16 coordinates of two parts (hi and
//     mid, brought side by side by one v_permlane32_swap per register for two
//     groups of 16 tiles), a second one the lo part and zeros; the +-1 rows
//     are the same in both halves of K, so a row table of 32 lanes serves.
//   * The 16 rows of a product are 4 seeds x 4 entries, ordered so that lane
//     (tile n, g) receives the four entries of seed 4 R + g: one product for
//     b_0..b_3, and with per-element weights two for the six Gram entries and
//     the mean of d (from products of two sign columns, which serve either
//     generator version).  A lane then owns a whole candidate without any
//     exchange.
//   * With per-column weights the Gram side belongs to the column block and the
//     seed: k_c16_factors builds its factor from fp64 sums, as the other
//     per-column screens have it, 64 bytes a (block, seed) that the lanes read
//     from the caches.  (Factored per candidate in fp32, one channel 1e5 / 1e6
//     times the others cost 1331 / 4958 of 15,360 tiles their best seed; from
//     the table 1092 / 4095, in the general screen 1025 / 4080.)
//   * Every candidate is scored in full (with 16 seeds, four per lane, there
//     is little to prune).  One whose rounding is on a knife edge (about 1e-3
//     of them) is scored again in the general screen's arithmetic: with
//     power-of-two scales a flipped rounding moves the score by percents.  So
//     is one whose Gram matrix is close to singular (kIll).  Each lane keeps
//     its two best, the four lanes of a tile merge, and the re-score runs in
//     the same wavefront with one lane per tile, from the residual and weights
//     kept in LDS.
//
// On the gate, up and down projections of a 3B layer (67.6 M weights, bf16,
// per-element weights, S = 16): 3884 us with the general vector screen and
// re-score, 503 us here, 90 of them in the knife-edge scores (a copy of the
// tensors takes 160).  11008 x 2048 with per-column weights: 985 -> 200 us.
#include <math.h>

#include "awsrc_internal.h"
#include "basis_gen.h"
#include "mfma_bf16.h"
#include "rescore64.h"
#include "screen_valu.h"

namespace awsrc {

namespace {

constexpr int kC = 16;
constexpr int kPB = 4;
constexpr int kNT = 64;       // tiles per wavefront
constexpr int kRow = 20;      // floats per LDS row of a tile (16-byte aligned rows)
// A candidate with a pivot e_p below kIll e_0 (e_0 is the mean of d) is scored
// in the general screen's arithmetic: where a few channels carry nearly all of
// d the Gram matrix is close to singular, the pivots are what is left of sums
// that cancel, and the score is decided by the order of those sums.  One
// channel of each tile 1e5 / 1e6 times the others, per element, tiles (of
// 15,360) whose best seed in 64 bits is lost: general screen 1142 / 4586,
// the products here 1342 / 5081, with this rule 1144 / 4586.  At 100 times 1e-4
// of the candidates are below it, at 1000 times 1%, without outliers none.  The
// test costs 1.5% (the MLP projections below: 495 -> 503 us); an 11008 x 2048 module
// with one channel in 1000 at 1e5 takes 277 us instead of 208.
constexpr float kIll = 0x1p-10f;
constexpr int kBlocks = 3;    // row tables per four seeds: b, and two of Gram entries

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The lower half of the wavefront keeps x and gives its y for the upper half's x:
// x = [x.lower | y.lower], y = [x.upper | y.upper].
__device__ __forceinline__ void swap32(uint32_t& x, uint32_t& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = r[0];
  y = r[1];
}

__device__ __forceinline__ f32x4 mfma(const u32x4& A, const u32x4& B, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A), as_bf16x8(B), c, 0, 0, 0);
}

__device__ __forceinline__ double flip(double x, uint32_t mask, int j) {
  const uint64_t s = (uint64_t)((mask << (31 - j)) & 0x80000000u) << 32;
  return __longlong_as_double((long long)((uint64_t)__double_as_longlong(x) ^ s));
}

// A tile's kept list: two entries, best first (gain descending, seed ascending).
struct Top2 {
  float g0 = -INFINITY, g1 = -INFINITY;
  uint32_t s0 = 0, s1 = 0;
  __device__ __forceinline__ void add(float g, uint32_t s) {  // seeds in increasing order
    const bool c0 = g > g0, c1 = g > g1;
    g1 = c0 ? g0 : (c1 ? g : g1);
    s1 = c0 ? s0 : (c1 ? s : s1);
    g0 = c0 ? g : g0;
    s0 = c0 ? s : s0;
  }
  __device__ __forceinline__ void merge(float og0, float og1, uint32_t os0, uint32_t os1) {
    auto better = [](float ga, uint32_t sa, float gb, uint32_t sb) {
      return ga > gb || (ga == gb && list_seed(sa) < list_seed(sb));
    };
    const bool mine = better(g0, s0, og0, os0);
    const bool second = mine ? better(g1, s1, og0, os0) : better(g0, s0, og1, os1);
    const float n1 = mine ? (second ? g1 : og0) : (second ? g0 : og1);
    const uint32_t m1 = mine ? (second ? s1 : os0) : (second ? s0 : os1);
    g0 = mine ? g0 : og0;
    s0 = mine ? s0 : os0;
    g1 = n1;
    s1 = m1;
  }
};

// What is known of a seed besides its row tables.
struct SeedInfo {
  uint32_t mask[2];  // sign columns, 16 bits each (bit j set: B_s[j, p] < 0; 0 for p >= P)
  uint32_t col;      // selected Hadamard columns, a byte each (0 for p >= P)
  uint32_t pad_;
  uint64_t inv;      // pi^-1: nibble i is the coordinate whose Hadamard row is i
  uint64_t pad2_;
};
static_assert(sizeof(SeedInfo) == 32, "table entry");

// A factor table entry (per-column weights): L, 1/e and e of col_factor64, padded to whole 64 bytes.
constexpr int kFac = 16;
constexpr int kFacLen = kPB * (kPB - 1) / 2 + 2 * kPB;
static_assert(kFacLen <= kFac, "factor entry");

// Entry k of the length-16 transform of x, in the operation order of the
// in-place butterflies (so the same value bit for bit).
__device__ __forceinline__ float wht16_entry(const float (&x)[kC], uint32_t k) {
  float v[kC];
#pragma unroll
  for (int i = 0; i < kC; ++i) v[i] = x[i];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const uint32_t s = (k << (31 - b)) & 0x80000000u;
#pragma unroll
    for (int i = 0; i < (kC >> (b + 1)); ++i) v[i] = v[2 * i] + __uint_as_float(__float_as_uint(v[2 * i + 1]) ^ s);
  }
  return v[0];
}

// The score of one candidate in the general vector screen's arithmetic
// (projections summed in coordinate order; per element, Gram entries from the
// transform of the tile's weights; per column, the factor table f): for
// candidates on a knife edge, see screen_valu.h.  r, d: the tile's LDS rows.
template <bool POW2, bool PE>
__device__ __forceinline__ float general_score(const EncodeArgs& a, const SeedInfo& si, const float* r, const float* d,
                                               const float (&f)[kFacLen], float qmax, float inv_qmax, bool* edge) {
  constexpr int PB = kPB;
  const int P = a.P;
  const uint32_t m[PB] = {si.mask[0] & 0xFFFFu, si.mask[0] >> 16, si.mask[1] & 0xFFFFu, si.mask[1] >> 16};
  float bv[PB] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int j = 0; j < kC; ++j) {
    const float u = d[j] * r[j];
#pragma unroll
    for (int p = 0; p < PB; ++p) bv[p] += ((m[p] >> j) & 1u) ? -u : u;
  }
#pragma unroll
  for (int p = 0; p < PB; ++p) bv[p] = p < P ? bv[p] * 0.25f : 0.0f;
  if constexpr (!PE) {
    return screen_score_ldl<PB, POW2, 0>(bv, f, qmax, inv_qmax, edge);
  } else {
    uint32_t c[PB];
#pragma unroll
    for (int p = 0; p < PB; ++p) c[p] = (si.col >> (8 * p)) & 15u;
    float x[kC], G[PB][PB];
#pragma unroll
    for (int i = 0; i < kC; ++i) x[i] = d[(uint32_t)(si.inv >> (4 * i)) & 15u];
    const float sum = wht16_entry(x, 0);
    const float eps = (float)a.lambda * sum * 0.0625f;
#pragma unroll
    for (int p = 0; p < PB; ++p) {
#pragma unroll
      for (int q = 0; q < p; ++q) G[p][q] = p < P ? wht16_entry(x, c[p] ^ c[q]) * 0.0625f : 0.0f;
      G[p][p] = p < P ? sum * 0.0625f + eps : 1.0f;
    }
    return chol_score32<PB>(bv, G, eps, qmax, inv_qmax, POW2, edge);
  }
}

}  // namespace

// Tables of four seeds per block: each seed's SeedInfo, and the +-1 row
// tables of the matrix products, row 4 q + k belonging to seed 4 R + q:
//   table 0  column k;   table 1  column products (1,0) (2,0) (2,1) (3,0);
//   table 2  column products (3,1) (3,2), all ones, zeros.
// Rows of seeds >= S and of columns >= P are zero.  Lane l < 32 holds
// coordinates 8 (l / 16) .. + 7 of row l % 16.
__global__ __launch_bounds__(64) void k_c16_tables(uint64_t key, int P, int S, int gen_version,
                                                   u32x4* __restrict__ frag, SeedInfo* __restrict__ info,
                                                   unsigned long long* scored, unsigned long long n_scored) {
  __shared__ uint64_t s_key[4][kC];
  __shared__ uint8_t s_at[4][kC];    // Hadamard row of coordinate j
  __shared__ uint32_t s_col[4][kPB];
  __shared__ uint32_t s_mask[4][kPB];
  if (blockIdx.x == 0 && threadIdx.x == 0) *scored = n_scored;
  const int R = blockIdx.x, q = threadIdx.x >> 4, j = threadIdx.x & 15;
  const int s = 4 * R + q;
  const uint64_t base = (uint64_t)s << 32;
  const uint32_t sign = (uint32_t)splitmix64(key, base) & 0xFFFFu;
  if (j == 0) {
    uint64_t used[2] = {0ull, 0ull};
    for (int p = 0; p < kPB; ++p) s_col[q][p] = p < P ? (uint32_t)draw_column(key, base, 1, kC, p, used) : 0u;
  }
  if (gen_version == 2) s_key[q][j] = splitmix64(key, base + (uint64_t)(1 + P + j));
  __syncthreads();
  int at = j;
  if (gen_version == 2) {
    at = 0;
    const uint64_t kj = s_key[q][j];
    for (int i = 0; i < kC; ++i) {
      const uint64_t ki = s_key[q][i];
      at += (ki < kj) || (ki == kj && i < j);
    }
  }
  s_at[q][j] = (uint8_t)at;
  __syncthreads();
  if (j < kPB) {
    uint32_t m = 0;
    if (j < P)
      for (int i = 0; i < kC; ++i)
        m |= (((sign >> i) & 1u) ^ (uint32_t)(__popc((unsigned)s_at[q][i] & s_col[q][j]) & 1)) << i;
    s_mask[q][j] = m;
  }
  __syncthreads();
  if (j == 0 && s < S) {
    SeedInfo si{};
    si.mask[0] = s_mask[q][0] | (s_mask[q][1] << 16);
    si.mask[1] = s_mask[q][2] | (s_mask[q][3] << 16);
    for (int p = 0; p < kPB; ++p) si.col |= s_col[q][p] << (8 * p);
    for (int i = 0; i < kC; ++i) si.inv |= (uint64_t)i << (4 * s_at[q][i]);
    info[s] = si;
  }
  for (int i = threadIdx.x; i < kBlocks * 32; i += 64) {
    const int tb = i >> 5, l = i & 31, m = l & 15;
    const int mq = m >> 2, k = m & 3;
    const uint32_t* mk = s_mask[mq];
    uint32_t x;
    bool live = 4 * R + mq < S;
    if (tb == 0) {
      x = mk[k];
      live = live && k < P;
    } else {
      const int e = 4 * (tb - 1) + k;  // entry of the packed strict lower triangle, 6: ones, 7: none
      const int a = e == 0 ? 1 : (e < 3 ? 2 : 3), b = e == 0 ? 0 : (e < 3 ? e - 1 : e - 3);
      x = e < 6 ? mk[a] ^ mk[b] : 0u;
      live = live && (e < 6 ? a < P : e == 6);
    }
    x >>= 8 * (l >> 4);
    u32x4 w;
#pragma unroll
    for (int d = 0; d < 4; ++d)
      w[d] = live ? 0x3F803F80u | (((x >> (2 * d)) & 1u) << 15) | (((x >> (2 * d + 1)) & 1u) << 31) : 0u;
    frag[((size_t)R * kBlocks + tb) * 32 + l] = w;
  }
}

// Per-column weights: the factor of G + eps I of every (column block, seed),
// from fp64 sums (col_factor64), one thread each; blocks of the modules
// follow each other (ModEntry::item2_off).
__global__ __launch_bounds__(256) void k_c16_factors(EncodeArgs a, ModEntry one, const ModEntry* __restrict__ mods,
                                                     int n_mods, const SeedInfo* __restrict__ info, int64_t blocks) {
  constexpr int PB = kPB;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= blocks * a.S) return;
  const int64_t blk = i / a.S;
  const int s = (int)(i % a.S);
  ModEntry md = one;
  if (n_mods > 1) md = mods[find_module<&ModEntry::item2_off>(mods, n_mods, blk)];
  const float* dp = md.d + (blk - md.item2_off) * kC;
  const SeedInfo si = info[s];
  const uint32_t m[PB] = {si.mask[0] & 0xFFFFu, si.mask[0] >> 16, si.mask[1] & 0xFFFFu, si.mask[1] >> 16};
  double sum = 0.0, G[PB][PB];
#pragma unroll
  for (int p = 0; p < PB; ++p)
#pragma unroll
    for (int q = 0; q < p; ++q) G[p][q] = 0.0;
#pragma unroll
  for (int j = 0; j < kC; j += 4) {
    const gf32x4 v = gload4f(dp + j);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double x = (double)v[k];
      sum += x;
#pragma unroll
      for (int p = 0; p < PB; ++p)
#pragma unroll
        for (int q = 0; q < p; ++q) G[p][q] += flip(x, m[p] ^ m[q], j + k);
    }
  }
  const double eps = a.lambda * (sum / kC);
#pragma unroll
  for (int p = 0; p < PB; ++p) {
#pragma unroll
    for (int q = 0; q < p; ++q) G[p][q] = p < a.P ? G[p][q] / kC : 0.0;
    G[p][p] = p < a.P ? sum / kC + eps : 1.0;
  }
  float f[kFac] = {};
  col_factor64<PB>(G, f);
#pragma unroll
  for (int k = 0; k < kFac; k += 4)
    *reinterpret_cast<f32x4*>(a.colfac + i * kFac + k) = f32x4{f[k], f[k + 1], f[k + 2], f[k + 3]};
}

// PE: per-element weights; else the Gram side comes from the factor table.
template <bool POW2, bool FULLP, bool PE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_encode_c16(EncodeArgs a, ModEntry one, const ModEntry* __restrict__ mods,
                                                   int n_mods, const u32x4* __restrict__ frag,
                                                   const SeedInfo* __restrict__ info) {
  constexpr int LS = kPB * (kPB - 1) / 2;
  __shared__ __attribute__((aligned(16))) float rsh[kNT * kRow], dsh[kNT * kRow];
  __shared__ float tgs[2][kNT];
  __shared__ uint32_t tss[2][kNT];
  const int lane = threadIdx.x, n = lane & 15, g = lane >> 4;
  const int64_t item = blockIdx.x;
  ModEntry md = one;
  if (n_mods > 1) md = mods[find_module(mods, n_mods, item)];
  const uint32_t nb = (uint32_t)(md.cols / kC);
  const int64_t T = md.rows * (int64_t)nb;
  const int64_t t0 = (item - md.item_off) * kNT;

  // lane (n, g): eight coordinates (from 8 (g & 1)) of tiles 16 (g >> 1) + n
  // and 32 + 16 (g >> 1) + n; tiles past the end repeat the last one
  int64_t o[4], od[4];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int64_t tt = t0 + 32 * i + 16 * (g >> 1) + n;
    const int64_t t = tt < T ? tt : T - 1;
    o[2 * i] = t * kC + 8 * (g & 1);
    o[2 * i + 1] = o[2 * i] + 4;
    od[2 * i] = PE ? o[2 * i] : (int64_t)((uint32_t)t % nb) * kC + 8 * (g & 1);
    od[2 * i + 1] = od[2 * i] + 4;
  }
  gf32x4 dv[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) dv[c] = gload4f(md.d + od[c]);
  float rv[4][4];
  load_residual4<4>(md.W, a.w_dtype, md.W0, o, rv);

  const int P = a.P, nR = (a.S + 3) / 4;
  const float qmax = (float)((1 << (a.b - 1)) - 1);
  const float inv_qmax = 1.0f / qmax;
  const float lam = (float)a.lambda;
  const u32x4* fl = frag + (lane & 31);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    float u[8], dd[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float d = dv[2 * i + (e >> 2)][e & 3];
      u[e] = 0.25f * (d * rv[2 * i + (e >> 2)][e & 3]);  // 1/sqrt(C), exact
      dd[e] = 0.0625f * d;                               // 1/C, exact
    }
    {
      const int row = (32 * i + 16 * (g >> 1) + n) * kRow + 8 * (g & 1);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        *reinterpret_cast<f32x4*>(rsh + row + 4 * h) = f32x4{rv[2 * i + h][0], rv[2 * i + h][1], rv[2 * i + h][2], rv[2 * i + h][3]};
        *reinterpret_cast<f32x4*>(dsh + row + 4 * h) = f32x4{dv[2 * i + h][0], dv[2 * i + h][1], dv[2 * i + h][2], dv[2 * i + h][3]};
      }
    }
    wave_sync();
    // operands of the two groups of 16 tiles: [hi | mid] and [lo | 0]
    u32x4 U0[2], U1[2], D0[2], D1[2];
    auto operands = [](const float (&x8)[8], u32x4 (&X0)[2], u32x4 (&X1)[2]) {
      split3(x8, X0[0], X0[1], X1[0]);
      X1[1] = u32x4{0, 0, 0, 0};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        uint32_t x = X0[0][e], y = X0[1][e];
        swap32(x, y);
        X0[0][e] = x; X0[1][e] = y;
        x = X1[0][e]; y = X1[1][e];
        swap32(x, y);
        X1[0][e] = x; X1[1][e] = y;
      }
    };
    operands(u, U0, U1);
    if constexpr (PE) operands(dd, D0, D1);
    // per-column weights: this lane's tiles' rows of the factor table
    const float* fr[2];
    if constexpr (!PE) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int64_t tt = t0 + 32 * i + 16 * k + n;
        const uint32_t t = (uint32_t)(tt < T ? tt : T - 1);
        fr[k] = a.colfac + (md.item2_off + (int64_t)(t % nb)) * a.S * kFac;
      }
    }
    Top2 top[2];
    u32x4 A0 = fl[0], A1, A2;
    if constexpr (PE) { A1 = fl[32]; A2 = fl[64]; }
    for (int R = 0; R < nR; ++R) {
      const int s = 4 * R + g;
      f32x4 bq[2], ga[2], gb[2], fv[2][kFac / 4];
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      if constexpr (!PE) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int c = 0; c < kFac / 4; ++c)
            fv[k][c] = *reinterpret_cast<const f32x4*>(fr[k] + (s < a.S ? s : a.S - 1) * kFac + 4 * c);
      }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if constexpr (PE) {
          ga[k] = mfma(A1, D1[k], mfma(A1, D0[k], z));
          gb[k] = mfma(A2, D1[k], mfma(A2, D0[k], z));
        }
        bq[k] = mfma(A0, U1[k], mfma(A0, U0[k], z));
      }
      const u32x4* fn = fl + (size_t)(R + 1 < nR ? R + 1 : R) * (kBlocks * 32);
      A0 = fn[0];
      if constexpr (PE) { A1 = fn[32]; A2 = fn[64]; }
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        // G + eps I = L diag(e) L^T (the layout of the per-column table)
        float f[kFacLen];
        if constexpr (PE) {
          const float gq[LS] = {ga[k][0], ga[k][1], ga[k][2], ga[k][3], gb[k][0], gb[k][1]};
          const float d0 = gb[k][2], diag = fmaf(lam, d0, d0);
          screen_factor<kPB, FULLP>(gq, diag, P, f);
        } else {
#pragma unroll
          for (int c = 0; c < kFacLen; ++c) f[c] = fv[k][c >> 2][c & 3];
        }
        const float b[kPB] = {bq[k][0], bq[k][1], bq[k][2], bq[k][3]};
        bool edge;
        float gain = screen_score_ldl<kPB, POW2, 0>(b, f, qmax, inv_qmax, &edge);
        constexpr int E0 = LS + kPB;  // the pivots (1 in padded columns)
        float least = f[E0];
#pragma unroll
        for (int p = 1; p < kPB; ++p) least = FULLP || p < P ? fminf(least, f[E0 + p]) : least;
        const bool ill = least < kIll * f[E0];
        const bool general = (int)(edge | ill) & (int)(s < a.S);
        edge = false;  // as the general score finds it
        if (__ballot(general) != 0) {
          if (general) {
            const int at = (32 * i + 16 * k + n) * kRow;
            gain = general_score<POW2, PE>(a, info[s], rsh + at, dsh + at, f, qmax, inv_qmax, &edge);
          }
        }
        top[k].add(s < a.S ? gain : -INFINITY, (uint32_t)s | (edge ? kEdge : 0u));
      }
    }
    // the tile's four lanes (n, n + 16, n + 32, n + 48) merge their lists
#pragma unroll
    for (int k = 0; k < 2; ++k) {
#pragma unroll
      for (int x = 16; x <= 32; x <<= 1)
        top[k].merge(__shfl_xor(top[k].g0, x, 64), __shfl_xor(top[k].g1, x, 64),
                     (uint32_t)__shfl_xor((int)top[k].s0, x, 64), (uint32_t)__shfl_xor((int)top[k].s1, x, 64));
      if (g == 0) {
        const int tl = 32 * i + 16 * k + n;
        tgs[0][tl] = top[k].g0;
        tgs[1][tl] = top[k].g1;
        tss[0][tl] = top[k].s0;
        tss[1][tl] = top[k].s1;
      }
    }
  }
  wave_sync();

  // fp64 re-score, one lane per tile
  const int64_t t = t0 + lane;
  const float tg0 = tgs[0][lane], tg1 = tgs[1][lane];
  const uint32_t ts0 = tss[0][lane], ts1 = tss[1][lane];
  float rr[kC], dd[kC];
  float e32 = 0.0f;
  double sumd = 0.0;
#pragma unroll
  for (int j = 0; j < kC; j += 4) {
    const f32x4 x = *reinterpret_cast<const f32x4*>(rsh + lane * kRow + j);
    const f32x4 y = *reinterpret_cast<const f32x4*>(dsh + lane * kRow + j);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      rr[j + k] = x[k];
      dd[j + k] = y[k];
      e32 = fmaf(y[k] * x[k], x[k], e32);
      sumd += (double)y[k];
    }
  }
  const double eps = a.lambda * (sumd / kC);
  const int iqmax = (1 << (a.b - 1)) - 1;
  auto score64 = [&](int s, int (&q)[kPB], double (&al)[kPB], uint16_t* bits) -> double {
    const uint2 mw = *reinterpret_cast<const uint2*>(info[s].mask);
    const uint32_t m[kPB] = {mw.x & 0xFFFFu, mw.x >> 16, mw.y & 0xFFFFu, mw.y >> 16};
    double bv[kPB], gr[kPB * (kPB + 1) / 2];
#pragma unroll
    for (int p = 0; p < kPB; ++p) {
      bv[p] = 0.0;
#pragma unroll
      for (int r = 0; r < p; ++r) gr[p * (p + 1) / 2 + r] = 0.0;
      gr[p * (p + 1) / 2 + p] = sumd;
    }
#pragma unroll
    for (int j = 0; j < kC; ++j) {
      const double dj = (double)dd[j], uj = dj * (double)rr[j];
#pragma unroll
      for (int p = 0; p < kPB; ++p) {
        bv[p] += flip(uj, m[p], j);
#pragma unroll
        for (int r = 0; r < p; ++r) gr[p * (p + 1) / 2 + r] += flip(dj, m[p] ^ m[r], j);
      }
    }
#pragma unroll
    for (int p = 0; p < kPB; ++p) bv[p] = p < P ? bv[p] * 0.25 : 0.0;
    double L[LS], e[kPB], inv[kPB];
    ldl64<kC, kPB>(P, gr, eps, L, e, inv);
    return solve_score_ldl<kPB>(a, bv, L, e, inv, eps, iqmax, q, al, bits);
  };
  int best_s = list_seed(ts0);
  int q[kPB];
  double al[kPB];
  uint16_t bits;
  double best = score64(best_s, q, al, &bits);
  const float thr = tg0 - rescore_window(tg0, e32, ((ts0 | ts1) & kEdge) != 0);
  const bool need = t < T && tg1 >= thr && tg1 > -INFINITY;
  if (__ballot(need) != 0) {
    int q2[kPB];
    double al2[kPB];
    uint16_t bits2;
    const int s2 = list_seed(ts1);
    const double g2 = score64(s2, q2, al2, &bits2);
    if (need && !(g2 < best) && (g2 != best || s2 < best_s)) {
      best = g2;
      best_s = s2;
      bits = bits2;
#pragma unroll
      for (int p = 0; p < kPB; ++p) { q[p] = q2[p]; al[p] = al2[p]; }
    }
  }
  if (t >= T) return;
  const int64_t to = md.tile_off + t;
  // a gain that is not a number (infinite or NaN inputs): the empty record of the general re-score
  const bool none = !(best > -INFINITY);
  a.seed_out[to] = none ? 0xFFFFu : (uint16_t)best_s;
  a.scale_out[to] = none ? 0u : bits;
  a.gain_out[to] = none ? -INFINITY : best;
  int8_t* cp = a.code_out + to * P;
  if (FULLP && (reinterpret_cast<uintptr_t>(cp) & 3) == 0) {
    uint32_t w = 0;
#pragma unroll
    for (int p = 0; p < kPB; ++p) w |= (uint32_t)(uint8_t)q[p] << (8 * p);
    *reinterpret_cast<uint32_t*>(cp) = none ? 0u : w;
  } else {
#pragma unroll
    for (int p = 0; p < kPB; ++p)
      if (p < P) cp[p] = none ? 0 : (int8_t)q[p];
  }
  if (a.alpha_out) {
#pragma unroll
    for (int p = 0; p < kPB; ++p)
      if (p < P) a.alpha_out[to * P + p] = none ? 0.0f : (float)al[p];
  }
  if (a.top_gain) {
    *reinterpret_cast<float2*>(a.top_gain + t * kTop) = make_float2(tg0, tg1);
    *reinterpret_cast<uint2*>(a.top_seed + t * kTop) = make_uint2(ts0, ts1);
  }
}

bool c16_supported(int C, int P) { return C == kC && P <= kPB; }
int64_t c16_items(int64_t tiles) { return (tiles + kNT - 1) / kNT; }
size_t c16_frag_bytes(int S) { return (size_t)((S + 3) / 4) * kBlocks * 32 * 16; }
size_t c16_info_bytes(int S) { return (size_t)S * sizeof(SeedInfo); }
size_t c16_fac_bytes(int S, int64_t blocks) { return (size_t)blocks * S * kFac * 4; }

hipError_t launch_c16_tables(const EncodeArgs& a, uint64_t key, unsigned long long candidates, void* frag, void* info,
                             hipStream_t st) {
  hipLaunchKernelGGL(k_c16_tables, dim3((unsigned)((a.S + 3) / 4)), dim3(64), 0, st, key, a.P, a.S, a.gen_version,
                     static_cast<u32x4*>(frag), static_cast<SeedInfo*>(info), a.scored, candidates);
  return hipGetLastError();
}

template <bool POW2, bool FULLP>
static void run_c16(const EncodeArgs& a, const ModEntry& one, const ModEntry* mods, int n_mods, int64_t items,
                    const u32x4* fr, const SeedInfo* mk, hipStream_t st) {
  const dim3 grid((unsigned)items), blk(64);
  if (a.d_mode == AWSRC_D_PER_ELEM)
    hipLaunchKernelGGL((k_encode_c16<POW2, FULLP, true>), grid, blk, 0, st, a, one, mods, n_mods, fr, mk);
  else
    hipLaunchKernelGGL((k_encode_c16<POW2, FULLP, false>), grid, blk, 0, st, a, one, mods, n_mods, fr, mk);
}

hipError_t launch_encode_c16(const EncodeArgs& a, const ModEntry& one, const ModEntry* mods, int n_mods, int64_t items,
                             int64_t blocks, const void* frag, const void* info, hipStream_t st) {
  const u32x4* fr = static_cast<const u32x4*>(frag);
  const SeedInfo* mk = static_cast<const SeedInfo*>(info);
  if (a.d_mode != AWSRC_D_PER_ELEM)
    hipLaunchKernelGGL(k_c16_factors, dim3((unsigned)((blocks * a.S + 255) / 256)), dim3(256), 0, st, a, one, mods, n_mods,
                       mk, blocks);
  if (a.scale_fmt == AWSRC_SCALE_POW2) {
    if (a.P == kPB) run_c16<true, true>(a, one, mods, n_mods, items, fr, mk, st);
    else run_c16<true, false>(a, one, mods, n_mods, items, fr, mk, st);
  } else {
    if (a.P == kPB) run_c16<false, true>(a, one, mods, n_mods, items, fr, mk, st);
    else run_c16<false, false>(a, one, mods, n_mods, items, fr, mk, st);
  }
  return hipGetLastError();
}

}  // namespace awsrc
