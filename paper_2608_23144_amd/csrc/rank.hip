// Gain-ranked record selection and serialization (Eq. (4), Sec. 3.3, Eq. (5)).
//
// With a fixed record size, ordering by rho_t = gain_t / L_rec is ordering by
// gain.  The positive fp64 gains are mapped to their IEEE bit patterns, which
// order like the values.  For a segment of tiles:
//  0. the eligible tiles are counted and K = min(cap, eligible) is formed on
//     the device (the host never waits for it);
//  1. radix select (12-bit digits, most significant first) finds the K-th
//     largest key k* and how many records equal to k* are taken;
//  2. a stable compaction keeps every key > k* and the first such equal keys
//     in tile order (so equal gains keep the lower tile index);
//  3. the K survivors are sorted by (decreasing key, increasing tile): chunks
//     of 256 by a bitonic network in LDS, then multiway merge passes that
//     place each item by searches in the other runs of its group;
//  4. records are bit-packed at fixed offsets h + (first slot of the segment
//     + i) * L_rec.
// Cross-block results only pass between launches.  Each select pass finishes
// the previous pass itself: every block repeats the pick of the bin holding
// the K-th key from the previous histogram (4096 bins, a block scan), so a
// pass is one launch; histograms rotate over three buffers and the pick
// state over two, so no launch overwrites what another block of the same
// launch still reads.  A segment is a chain of launches with no host round
// trip and one read of the totals ends the call.
//
// That is the exact path, which takes any number of equal gains.  The fast
// path, tried first, stops the select after two digits and sorts a few more
// keys than it keeps; small segments are ranked whole by one workgroup each.
// The fast path gives up where too many gains are equal.  Mostly it finds that
// before it sorts (a look at 4096 gains, the size of the K-th key's bin), and the
// exact path goes on from there: gains rounded to bf16, 43 M of them, 2.55 ms
// (with the whole fast path in front 4.1; the exact path alone,
// as it was before there was a fast one, 2.7).  One value many thousand times
// among distinct ones can still cost both paths, 3.1 ms there.
#include <string.h>

#include "awsrc_internal.h"

namespace awsrc {

constexpr int kThreads = 256;
constexpr int kRounds = 16;
constexpr int kItems = kThreads * kRounds;  // items per block in the compaction
constexpr int kChunk = 256;                 // items per LDS-sorted chunk
constexpr int kChunkThreads = 128;
constexpr int kLogChunk = 8;
constexpr int kFan = 16;                    // runs per multiway merge
constexpr int kLogFan = 4;
constexpr int kSelBits = 12;                // radix-select digit width
constexpr int kSelBins = 1 << kSelBits;
constexpr int kCellBits = 27;               // leading bits that the fast path sorts by (three 9-bit digits)

// Words of RankWs::state.
enum : int {
  kPrefix = 0, kMask = 1, kRem = 2, kDone = 3,  // radix select result of the current segment
  kSegK = 4, kSegOff = 5,                       // records of the segment, its first record slot
  kElig = 6, kArrive = 7,                       // per-launch accumulators, reset after use
  kTotK = 8, kTotElig = 9, kNoSpace = 10,       // totals over the segments of one call
  kAgain = 11,                                  // the fast path could not finish (kAgain* below)
  kCnt = 12,                                    // survivors of the segment (fast path)
  kBase = 13, kShift = 14,                      // fast path: smallest ~key of the segment, cell width
  kBig = 15,                                    // fast path: cells left to k_sort_cells
  kSel = 16,                                    // [2][4] pick state of alternate passes
  kOver = 24,                                   // the survivors do not fit the fast path's items
  kHist = 32                                    // [3][kSelBins] histograms of rotating passes
};
static_assert(kHist + 3 * kSelBins == kStateWords, "rank state size");
// kAgain: before anything was sorted (the select's first pass still stands), or after
constexpr uint64_t kAgainEarly = 1, kAgainLate = 2;

// Positive doubles order like their bit patterns; the top (sign) bit is set on
// eligible keys so that every eligible key exceeds every ineligible (zero) key.
__device__ __forceinline__ uint64_t gain_key(double g) {
  return g > 0.0 ? ((uint64_t)__double_as_longlong(g) | (1ull << 63)) : 0ull;
}

__device__ __forceinline__ uint64_t lanemask_lt() {
  const int lane = threadIdx.x & 63;
  return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Exclusive block scan of a 0/1 flag over kThreads threads; returns the
// exclusive prefix for this thread and the block total in *total.
__device__ __forceinline__ uint32_t block_scan_flag(bool f, uint32_t* sh_w, uint32_t* total) {
  const int lane = threadIdx.x & 63;
  const int w = threadIdx.x >> 6;
  const uint64_t bal = __ballot(f);
  const uint32_t in_wave = __popcll(bal & lanemask_lt());
  if (lane == 0) sh_w[w] = __popcll(bal);
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kThreads / 64; ++k) {
    const uint32_t c = sh_w[k];
    before += (k < w) ? c : 0u;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return before + in_wave;
}

// Clears the state and writes a piece of the stream header (passed by value,
// so the call needs no host copy).
__global__ void k_rank_init(uint64_t* state, HeaderChunk hc, int n, uint8_t* __restrict__ out) {
  if (state)
    for (int i = threadIdx.x; i < kStateWords; i += blockDim.x) state[i] = 0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) out[i] = hc.b[i];
}

// The totals of a call (records, eligible tiles, no-space and run-again
// flags) for the host.
__global__ void k_rank_totals(const uint64_t* state, uint64_t* dst) {
  if (threadIdx.x < kRankTotals) {
    uint64_t v = state[kTotK + threadIdx.x];
    if (threadIdx.x == kAgain - kTotK && state[kOver]) v = v > kAgainEarly ? v : kAgainEarly;
    dst[threadIdx.x] = v;
  }
}

// After a fast attempt that ended early, on the one segment of a call: the exact
// path goes on from the first select pass (its pick, the second histogram and the
// eligible count stand).
__global__ void k_rank_resume(uint64_t* state) {
  if ((threadIdx.x >= kTotK && threadIdx.x <= kAgain) || threadIdx.x == kOver) state[threadIdx.x] = 0;
}

// ---------------------------------------------------------------- radix select
// Each pass histograms the next digit of the keys that match the prefix so
// far; the next launch picks the bin holding the remaining-th largest key.
// When that whole bin is taken the search stops early: every key in it is
// selected, so the lower digits no longer matter.

// First pass of a segment, fused with the eligibility count: the top digit
// (eligible flag and exponent) of every key, into histogram 0.
__global__ __launch_bounds__(kThreads) void k_count_hist(const double* __restrict__ gain, int64_t n,
                                                         uint64_t* state) {
  __shared__ uint32_t h[kSelBins];
  __shared__ uint32_t sw[kThreads / 64];
  for (int b = threadIdx.x; b < kSelBins; b += kThreads) h[b] = 0;
  __syncthreads();
  uint32_t c = 0;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (; i + 7 * stride < n; i += 8 * stride) {
    double gv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) gv[u] = gain[i + u * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t k = gain_key(gv[u]);
      c += k != 0;
      atomicAdd(&h[k >> (64 - kSelBits)], 1u);
    }
  }
  for (; i < n; i += stride) {
    const uint64_t k = gain_key(gain[i]);
    c += k != 0;
    atomicAdd(&h[k >> (64 - kSelBits)], 1u);
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t t = 0;
    for (int k = 0; k < kThreads / 64; ++k) t += sw[k];
    if (t) atomicAdd((unsigned long long*)&state[kElig], (unsigned long long)t);
  }
  for (int b = threadIdx.x; b < kSelBins; b += kThreads)
    if (h[b]) atomicAdd((unsigned long long*)&state[kHist + b], (unsigned long long)h[b]);
}

struct SelState {
  uint64_t prefix, mask, rem, done;
  uint64_t bin;  // keys in the bin just picked (pick_bin)
};

// One block of kThreads: the bin of histogram `hist` (digit at `shift`,
// `width` bits) holding the rem-th largest key; thread t owns bpt consecutive
// bins counted from the top.  Every thread returns the same state.
__device__ SelState pick_bin(const uint64_t* hist, SelState in, int shift, int width) {
  __shared__ uint64_t s_wave[kThreads / 64];
  __shared__ uint64_t found[4];
  constexpr int kMaxBpt = kSelBins / kThreads;
  const int nbins = 1 << width;
  const int bpt = nbins >= kThreads ? nbins / kThreads : 1;
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  // this thread's bins, counted from the top, kept in registers for the search
  uint64_t v[kMaxBpt];
  uint64_t local = 0;
#pragma unroll
  for (int i = 0; i < kMaxBpt; ++i) {
    const int r = t * bpt + i;
    v[i] = (i < bpt && r < nbins) ? hist[nbins - 1 - r] : 0ull;
    local += v[i];
  }
  if (t < 4) found[t] = 0;
  // inclusive scan: within the wavefront by shuffles, then across the four
  uint64_t x = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_wave[wv] = x;
  __syncthreads();
  uint64_t before = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) before += w < wv ? s_wave[w] : 0ull;
  const uint64_t incl = before + x;
  const uint64_t excl = incl - local;
  if (excl < in.rem && in.rem <= incl) {
    uint64_t cum = excl;
    bool hit = false;
#pragma unroll
    for (int i = 0; i < kMaxBpt; ++i) {
      const uint64_t c = v[i];
      if (!hit && i < bpt && cum + c >= in.rem) {
        found[0] = (uint64_t)(nbins - 1 - (t * bpt + i));
        found[1] = in.rem - cum;
        found[2] = (c == in.rem - cum) ? 1ull : 0ull;
        found[3] = c;
        hit = true;
      }
      cum += c;
    }
  }
  __syncthreads();
  SelState out;
  out.prefix = in.prefix | (found[0] << shift);
  out.mask = in.mask | (((1ull << width) - 1ull) << shift);
  out.rem = found[1];
  out.done = found[2];
  out.bin = found[3];
  __syncthreads();
  return out;
}

// The fast path's look ahead at how many gains are equal: 4096 gains spread over
// the segment, those at or above the K-th key's first digit (some 950 where a
// quarter is kept, kTieSlots - 512 at most) entered in a hash table of kTieSlots
// keys; returns how many were in it already.  With gains rounded to bf16 or
// fp16, or of a thousand values, these are hundreds; groups of equal gains that
// k_sort_cells takes (up to kCellSort, 2% of the records in groups of 2000)
// give one or two.
constexpr int kTieSlots = kSelBins / 2;  // 2^11
constexpr int kTieProbe = 8;
__device__ int tie_probe(const double* __restrict__ gain, int64_t n, const SelState& sel, unsigned long long* table) {
  __shared__ int s_in, s_dup;
  for (int b = threadIdx.x; b < kTieSlots; b += kThreads) table[b] = 0ull;
  if (threadIdx.x == 0) s_in = s_dup = 0;
  __syncthreads();
  constexpr int kRows = 4096 / kThreads;
  const uint32_t step = (uint32_t)(n / 4096);  // (n <= 2^32)
  double gv[kRows];
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const uint32_t j = r * kThreads + threadIdx.x;
    gv[r] = gain[(int64_t)j * step + __umulhi(j * 0x9E3779B1u, step)];
  }
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    const uint64_t k = gain_key(gv[r]);
    if (k != 0 && (k & sel.mask) >= sel.prefix && atomicAdd(&s_in, 1) < kTieSlots - 512) {
      // at most kTieSlots - 512 keys: an empty slot always ends the search
      for (uint32_t at = ((uint32_t)(k >> 32) * 0x85EBCA6Bu ^ (uint32_t)k * 0x9E3779B1u) >> 21;; at = (at + 1) & (kTieSlots - 1)) {
        const unsigned long long old = atomicCAS(&table[at], 0ull, (unsigned long long)k);
        if (old == k) atomicAdd(&s_dup, 1);
        if (old == 0ull || old == k) break;
      }
    }
  }
  __syncthreads();
  return s_dup;
}

// Pass `pass` (1..5) of a segment: pick from the previous pass's histogram
// (digit at prev_shift), then histogram the next digit (at shift) of the keys
// under the new prefix.  Pass 1 forms K = min(cap, eligible) itself.
__global__ __launch_bounds__(kThreads) void k_select_pass(const double* __restrict__ gain, int64_t n,
                                                          uint64_t* state, int64_t cap, int pass, int prev_shift,
                                                          int prev_width, int shift, int width, int fast, int probe) {
  __shared__ __attribute__((aligned(8))) uint32_t h[kSelBins];
  SelState cur;
  if (fast && blockIdx.x == 0) {
    // the fast path's segment bookkeeping (no other block reads these words)
    __shared__ int top;
    if (threadIdx.x == 0) top = 0;
    __syncthreads();
    for (int b = threadIdx.x; b < kSelBins; b += kThreads)
      if (state[kHist + b]) atomicMax(&top, b);
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint64_t ne = state[kElig];
      state[kSegOff] = state[kTotK];
      state[kTotK] += ne < (uint64_t)cap ? ne : (uint64_t)cap;
      state[kTotElig] += ne;
      state[kCnt] = 0;
      state[kBig] = 0;
      state[kBase] = ~(((uint64_t)top << (64 - kSelBits)) | ((1ull << (64 - kSelBits)) - 1ull));
    }
  }
  if (pass == 1) {
    const uint64_t ne = state[kElig];
    const uint64_t K = ne < (uint64_t)cap ? ne : (uint64_t)cap;
    cur = SelState{0ull, 0ull, K, K == 0 ? 1ull : 0ull, 0ull};
    if (blockIdx.x == 0 && threadIdx.x == 0) state[kSegK] = K;
  } else {
    const uint64_t* sp = state + kSel + 4 * ((pass - 1) & 1);
    cur = SelState{sp[0], sp[1], sp[2], sp[3], 0ull};
  }
  // the histogram two passes back has been read by the previous launch
  uint64_t* hclr = state + kHist + kSelBins * ((pass + 1) % 3);
  for (int b = blockIdx.x * kThreads + threadIdx.x; b < kSelBins; b += gridDim.x * kThreads) hclr[b] = 0;
  SelState nw = cur;
  if (!cur.done) nw = pick_bin(state + kHist + kSelBins * ((pass - 1) % 3), cur, prev_shift, prev_width);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    uint64_t* so = state + kSel + 4 * (pass & 1);
    so[0] = nw.prefix; so[1] = nw.mask; so[2] = nw.rem; so[3] = nw.done;
    if (fast) {
      // cells of the fast path's sort: the 2^kCellBits top values of ~key - base
      // over the bins from the topmost one down to the K-th key's
      const uint64_t bins = ((~state[kBase]) >> (64 - kSelBits)) - (nw.prefix >> (64 - kSelBits)) + 1;
      int lg = 0;
      while ((1ull << lg) < bins) ++lg;
      state[kShift] = (uint64_t)(64 - kSelBits + lg - kCellBits);
    }
  }
  if (probe && blockIdx.x == gridDim.x - 1) {  // one block for this, the others for the pass
    if (tie_probe(gain, n, nw, reinterpret_cast<unsigned long long*>(h)) >= kTieProbe && threadIdx.x == 0)
      state[kAgain] = kAgainEarly;
    return;
  }
  if (nw.done) return;  // uniform
  for (int b = threadIdx.x; b < kSelBins; b += kThreads) h[b] = 0;
  __syncthreads();
  const uint64_t dm = (1ull << width) - 1ull;
  // eight independent loads per thread in flight (the grid is small: each
  // block ends with up to 4096 global atomics)
  const int64_t stride = (int64_t)(gridDim.x - probe) * kThreads;
  int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  for (; i + 7 * stride < n; i += 8 * stride) {
    double gv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) gv[u] = gain[i + u * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint64_t k = gain_key(gv[u]);
      if ((k & nw.mask) == nw.prefix) atomicAdd(&h[(k >> shift) & dm], 1u);
    }
  }
  for (; i < n; i += stride) {
    const uint64_t k = gain_key(gain[i]);
    if ((k & nw.mask) == nw.prefix) atomicAdd(&h[(k >> shift) & dm], 1u);
  }
  __syncthreads();
  uint64_t* hout = state + kHist + kSelBins * (pass % 3);
  for (int b = threadIdx.x; b < (1 << width); b += kThreads)
    if (h[b]) atomicAdd((unsigned long long*)&hout[b], (unsigned long long)h[b]);
}

// The select result after the last pass (pass 6's pick), as every block of the
// first compaction launch computes it.
__device__ SelState final_select(const uint64_t* state) {
  const uint64_t* sp = state + kSel + 4 * (5 & 1);
  SelState cur = SelState{sp[0], sp[1], sp[2], sp[3], 0ull};
  if (!cur.done) cur = pick_bin(state + kHist + kSelBins * (5 % 3), cur, 0, 4);
  return cur;
}

// ---------------------------------------------------------------- compaction
// Every block finishes the select itself (the last pick); block 0 records the
// result, the segment's first record slot and the running totals.
__global__ __launch_bounds__(kThreads) void k_compact_count(const double* __restrict__ gain, int64_t n,
                                                            uint64_t* state, uint64_t* blk_gt, uint64_t* blk_eq) {
  const uint64_t K = state[kSegK];
  const SelState fin = final_select(state);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    state[kPrefix] = fin.prefix;
    state[kMask] = fin.mask;
    state[kRem] = fin.rem;
    state[kDone] = fin.done;
    state[kSegOff] = state[kTotK];
    state[kTotK] += K;
    state[kTotElig] += state[kElig];
    state[kElig] = 0;
  }
  if (K == 0) return;  // uniform
  const uint64_t prefix = fin.prefix, mask = fin.mask;
  uint32_t gt = 0, eq = 0;
  const int64_t base = (int64_t)blockIdx.x * kItems;
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kThreads + threadIdx.x;
    if (i < n) {
      const uint64_t k = gain_key(gain[i]) & mask;
      gt += k > prefix;
      eq += k == prefix;
    }
  }
  __shared__ uint32_t s_gt[kThreads / 64], s_eq[kThreads / 64];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    gt += __shfl_xor(gt, off, 64);
    eq += __shfl_xor(eq, off, 64);
  }
  if ((threadIdx.x & 63) == 0) { s_gt[threadIdx.x >> 6] = gt; s_eq[threadIdx.x >> 6] = eq; }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t a = 0, b = 0;
    for (int k = 0; k < kThreads / 64; ++k) { a += s_gt[k]; b += s_eq[k]; }
    blk_gt[blockIdx.x] = a;
    blk_eq[blockIdx.x] = b;
  }
}

// Inclusive scan over the 1024 threads of a block: shuffles within each
// wavefront, then the 16 wavefront totals; *total gets the block sum.
__device__ __forceinline__ uint64_t scan1024(uint64_t v, uint64_t* s_wave, uint64_t* total) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  uint64_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint64_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) s_wave[wv] = x;
  __syncthreads();
  uint64_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const uint64_t t = s_wave[w];
    before += w < wv ? t : 0ull;
    tot += t;
  }
  __syncthreads();
  *total = tot;
  return before + x;
}

// Single block: eq offsets (exclusive scan of blk_eq) and selected offsets.
// On exit blk_gt[b] = first output slot of block b, blk_eq[b] = number of
// equal keys in earlier blocks.
__global__ __launch_bounds__(1024) void k_compact_scan(uint64_t* blk_gt, uint64_t* blk_eq, int64_t nblk,
                                                       uint64_t* state) {
  // every histogram has been read: leave them cleared for the next segment
  for (int b = threadIdx.x; b < 3 * kSelBins; b += 1024) state[kHist + b] = 0;
  if (threadIdx.x == 0) state[kCnt] = state[kSegK];  // exactly K items to sort
  if (state[kSegK] == 0) return;
  __shared__ uint64_t s_wave[16];
  const uint64_t rem = state[kRem];
  uint64_t carry_eq = 0, carry_sel = 0;
  for (int64_t c0 = 0; c0 < nblk; c0 += 1024) {
    const int64_t i = c0 + threadIdx.x;
    const uint64_t gt = i < nblk ? blk_gt[i] : 0, eq = i < nblk ? blk_eq[i] : 0;
    uint64_t eq_tot, sel_tot;
    const uint64_t eq_excl = carry_eq + scan1024(eq, s_wave, &eq_tot) - eq;
    uint64_t take_eq = 0;
    if (rem > eq_excl) take_eq = (rem - eq_excl) < eq ? (rem - eq_excl) : eq;
    const uint64_t sel = gt + take_eq;
    const uint64_t sel_excl = carry_sel + scan1024(sel, s_wave, &sel_tot) - sel;
    if (i < nblk) { blk_gt[i] = sel_excl; blk_eq[i] = eq_excl; }
    carry_eq += eq_tot;
    carry_sel += sel_tot;
  }
}

// gain: the segment's gains (from tile t0); seed, scale: every tile's
__global__ __launch_bounds__(kThreads) void k_compact_write(const double* __restrict__ gain,
                                                            const uint16_t* __restrict__ seed,
                                                            const uint16_t* __restrict__ scale, int64_t t0, int64_t n,
                                                            const uint64_t* __restrict__ state,
                                                            const uint64_t* __restrict__ sel_off,
                                                            const uint64_t* __restrict__ eq_off,
                                                            SortItem* __restrict__ items_out) {
  if (state[kSegK] == 0) return;  // uniform
  __shared__ uint32_t sh_w[kThreads / 64];
  const uint64_t prefix = state[kPrefix], mask = state[kMask];
  const uint64_t rem = state[kRem];
  uint64_t eq_run = eq_off[blockIdx.x];
  uint64_t sel_run = sel_off[blockIdx.x];
  const int64_t base = (int64_t)blockIdx.x * kItems;
  for (int r = 0; r < kRounds; ++r) {
    const int64_t i = base + r * kThreads + threadIdx.x;
    uint64_t k = 0;
    if (i < n) k = gain_key(gain[i]);
    const bool gt = (i < n) && (k & mask) > prefix;
    const bool eq = (i < n) && (k & mask) == prefix;
    uint32_t eq_tot, sel_tot;
    const uint32_t eq_rank = block_scan_flag(eq, sh_w, &eq_tot);
    const bool take = gt || (eq && (eq_run + eq_rank) < rem);
    const uint32_t pos = block_scan_flag(take, sh_w, &sel_tot);
    if (take) {
      SortItem it;
      it.key = ~k;  // ascending ~key = descending gain
      it.tile = (uint32_t)(t0 + i);
      it.aux = (uint32_t)seed[t0 + i] | ((uint32_t)scale[t0 + i] << 16);
      items_out[sel_run + pos] = it;
    }
    eq_run += eq_tot;
    sel_run += sel_tot;
  }
}

// ---------------------------------------------------------------- fast selection
// Two digits (24 bits) of the select leave the K-th key's bin a few keys wide
// (its keys agree in 12 mantissa bits), so the fast path stops there: it takes
// every key of that bin and above, a few more than K, sorts them by the total
// order (key, tile) and packs the first K.  That leaves out three select
// passes over the gains, the counting pass of the stable compaction and its
// scan (43 M gains: 5 x 60, 71 and 31 of 2,089 us; here one of 60).  The
// order of the survivors is free (slots are reserved by block), since the
// sort breaks ties by tile.  More survivors than the items hold (many equal
// gains) sets kAgain and the call runs the exact path instead, from the pass of
// the select that is done.
template <int ROUNDS>
__global__ __launch_bounds__(kThreads) void k_compact_fast(const double* __restrict__ gain,
                                                           const uint16_t* __restrict__ seed,
                                                           const uint16_t* __restrict__ scale, int64_t t0, int64_t n,
                                                           uint64_t* state, uint64_t cap_items,
                                                           SortItem* __restrict__ items_out) {
  __shared__ uint32_t s_cnt[kThreads / 64];
  __shared__ uint64_t s_base;
  const uint64_t K = state[kSegK];
  const uint64_t* sp = state + kSel + 4;  // the pick of pass 1
  SelState fin = SelState{sp[0], sp[1], sp[2], sp[3], 0ull};
  if (state[kAgain]) return;  // (not set in this launch)
  if (!fin.done) {
    fin = pick_bin(state + kHist + kSelBins, fin, 64 - 2 * kSelBits, kSelBits);
    if (K - fin.rem + fin.bin > cap_items) {  // uniform
      if (blockIdx.x == 0 && threadIdx.x == 0) state[kOver] = 1;
      return;
    }
  }
  if (blockIdx.x == 0) {  // the first histogram has been read: clear it and the count for the next segment
    for (int b = threadIdx.x; b < kSelBins; b += kThreads) state[kHist + b] = 0;
    if (threadIdx.x == 0) state[kElig] = 0;
  }
  if (K == 0) return;  // uniform
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint64_t lt = lanemask_lt();
  constexpr int kBlock = kThreads * ROUNDS;
  for (int64_t base = (int64_t)blockIdx.x * kBlock; base < n; base += (int64_t)gridDim.x * kBlock) {
    double gv[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int64_t i = base + r * kThreads + threadIdx.x;
      gv[r] = i < n ? gain[i] : 0.0;
    }
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const uint64_t k = gain_key(gv[r]);
      cnt += __popcll(__ballot(k != 0 && (k & fin.mask) >= fin.prefix));
    }
    if (lane == 0) s_cnt[wv] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t tot = 0;
      for (int w = 0; w < kThreads / 64; ++w) tot += s_cnt[w];
      s_base = tot ? atomicAdd((unsigned long long*)&state[kCnt], (unsigned long long)tot) : 0;
    }
    __syncthreads();
    uint64_t at = s_base;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) at += w < wv ? s_cnt[w] : 0u;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
      const int64_t i = base + r * kThreads + threadIdx.x;
      const uint64_t k = gain_key(gv[r]);
      const bool take = k != 0 && (k & fin.mask) >= fin.prefix;
      const uint64_t bal = __ballot(take);
      const uint64_t slot = at + (uint64_t)__popcll(bal & lt);
      if (take && slot < cap_items) {
        SortItem it;
        it.key = ~k;  // ascending ~key = descending gain
        it.tile = (uint32_t)(t0 + i);
        it.aux = (uint32_t)seed[t0 + i] | ((uint32_t)scale[t0 + i] << 16);
        items_out[slot] = it;
      }
      at += (uint64_t)__popcll(bal);
    }
    __syncthreads();  // s_cnt and s_base are reused
  }
}

// Items to sort in the current segment.
__device__ __forceinline__ int64_t sort_count(const uint64_t* state, int64_t cap_items) {
  const int64_t c = (int64_t)state[kCnt];
  return c < cap_items ? c : cap_items;
}

// ---------------------------------------------------------------- packing
__device__ __forceinline__ void put_bits(uint64_t (&w)[3], int& pos, uint64_t v, int nbits) {
  if (nbits <= 0) return;
  const int o = pos & 63, k = pos >> 6;
  w[k] |= v << o;
  if (o + nbits > 64) w[k + 1] |= v >> (64 - o);
  pos += nbits;
}

// The P codes of tile t as bytes (code p in byte p), in one load where they
// fill an aligned word.
struct Codes {
  uint64_t w[2];
};
__device__ __forceinline__ Codes load_codes(const PackArgs& pa, uint32_t t) {
  const int8_t* c = pa.code + (int64_t)t * pa.P;
  Codes r = {{0, 0}};
  if (pa.P == 8 && (reinterpret_cast<uintptr_t>(pa.code) & 7) == 0) {
    r.w[0] = *reinterpret_cast<const uint64_t*>(c);
  } else if (pa.P == 4 && (reinterpret_cast<uintptr_t>(pa.code) & 3) == 0) {
    r.w[0] = *reinterpret_cast<const uint32_t*>(c);
  } else {
#pragma unroll
    for (int p = 0; p < kMaxP; ++p)
      if (p < pa.P) r.w[p >> 3] |= (uint64_t)(uint8_t)c[p] << (8 * (p & 7));
  }
  return r;
}

// Record of tile t (aux = its seed | scale << 16) into a slot of the stream.
// A record at a 4-byte aligned place whose size is a multiple of 4 goes out
// as whole words.
__device__ __forceinline__ void write_record(const PackArgs& pa, uint64_t slot, uint32_t t, uint32_t aux,
                                             const Codes& codes) {
  uint64_t w[3] = {0, 0, 0};
  int pos = 0;
  put_bits(w, pos, (uint64_t)t, pa.idx_bits);
  put_bits(w, pos, (uint64_t)(aux & 0xFFFFu), pa.seed_bits);
  const uint64_t cm = (1ull << pa.b) - 1ull;
#pragma unroll
  for (int p = 0; p < kMaxP; ++p)
    if (p < pa.P) put_bits(w, pos, (codes.w[p >> 3] >> (8 * (p & 7))) & cm, pa.b);
  put_bits(w, pos, (uint64_t)(aux >> 16) & ((1ull << pa.scale_bits) - 1ull), pa.scale_bits);
  uint8_t* o = pa.out + pa.h + slot * (uint64_t)pa.L;
  if (((reinterpret_cast<uintptr_t>(o) | (uintptr_t)pa.L) & 3) == 0) {
    uint32_t* o32 = reinterpret_cast<uint32_t*>(o);
    for (int k = 0; k < pa.L / 4; ++k) o32[k] = (uint32_t)(w[k >> 1] >> (32 * (k & 1)));
  } else {
    for (int k = 0; k < pa.L; ++k) o[k] = (uint8_t)(w[k >> 3] >> (8 * (k & 7)));
  }
}

// Record i of the segment (tile t) goes to byte h + (first slot + i) * L of
// the stream; a stream buffer too small for the running total raises the
// no-space flag instead.
__device__ __forceinline__ void pack_record(const PackArgs& pa, uint64_t* state, int64_t i, uint32_t t, uint32_t aux,
                                            const Codes& codes) {
  const uint64_t K = state[kSegK], off = state[kSegOff];
  if ((uint64_t)i >= K) return;  // the fast path sorts a few more items than it keeps
  if (pa.h + (off + K) * (uint64_t)pa.L > pa.cap) {
    if (i == 0) state[kNoSpace] = 1;
    return;
  }
  write_record(pa, off + (uint64_t)i, t, aux, codes);
}

// the same, with the seed and scale read from the encoder outputs
__device__ __forceinline__ void pack_record(const PackArgs& pa, uint64_t* state, int64_t i, uint32_t t) {
  pack_record(pa, state, i, t, (uint32_t)pa.seed[t] | ((uint32_t)pa.scale[t] << 16), load_codes(pa, t));
}

// ---------------------------------------------------------------- sort of the survivors
// Items are (key, tile) pairs; tiles are distinct, so the lexicographic order
// on the pair is a total order and equal gains come out in increasing tile
// order without any stability argument.
__device__ __forceinline__ bool kv_less(const SortItem& a, const SortItem& b) {
  return (a.key < b.key) | ((a.key == b.key) & (a.tile < b.tile));  // no short-circuit branches
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Bitonic sort of M (key, tile) pairs in LDS by THREADS threads.  Pair q of a
// stage with distance j compares elements i = (q with a zero inserted at bit
// log2 j) and i + j; thread t takes pairs t + r THREADS, so for j <= 64 every
// wavefront works inside its own 128-element windows and a wavefront-level
// barrier suffices between stages.
template <int M, int THREADS>
__device__ __forceinline__ void bitonic_lds(uint64_t* sk, uint32_t* st) {
  int prev = M;
  for (int k = 2; k <= M; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j > 64 || prev > 64) __syncthreads(); else wave_sync();
#pragma unroll
      for (int r = 0; r < M / (2 * THREADS); ++r) {
        const int q = r * THREADS + threadIdx.x;
        const int i = ((q & ~(j - 1)) << 1) | (q & (j - 1));
        const uint64_t ka = sk[i], kb = sk[i + j];
        const uint32_t ta = st[i], tb = st[i + j];
        const bool b_first = kb < ka || (kb == ka && tb < ta);
        const bool sw = ((i & k) == 0) == b_first;  // ascending half: swap if b < a
        sk[i] = sw ? kb : ka;
        sk[i + j] = sw ? ka : kb;
        st[i] = sw ? tb : ta;
        st[i + j] = sw ? ta : tb;
      }
      prev = j;
    }
  }
  __syncthreads();
}

// In-place sort of each chunk of kChunk items; the tail chunk is padded with
// sentinels that sort last and are not written back.  With `pack` set (the
// final pass) the sorted items are packed as records.  clear_hist: the fast
// path's second histogram has been read by now and is cleared here.
__global__ __launch_bounds__(kChunkThreads) void k_sort_chunks(SortItem* __restrict__ items, uint64_t* state,
                                                               int64_t cap_items, int clear_hist, int pack,
                                                               PackArgs pa) {
  __shared__ uint64_t sk[kChunk];
  __shared__ uint32_t st[kChunk];
  const int64_t n = sort_count(state, cap_items);
  if (clear_hist && blockIdx.x == 0 && n > 0)  // (an attempt given up needs it again)
    for (int b = threadIdx.x; b < kSelBins; b += kChunkThreads) state[kHist + kSelBins + b] = 0;
  const int64_t base = (int64_t)blockIdx.x * kChunk;
  if (base >= n) return;  // uniform per block
#pragma unroll
  for (int r = 0; r < kChunk / kChunkThreads; ++r) {
    const int j = r * kChunkThreads + threadIdx.x;
    const int64_t i = base + j;
    uint64_t key = ~0ull;
    uint32_t tile = 0xFFFFFFFFu;
    if (i < n) { key = items[i].key; tile = items[i].tile; }
    sk[j] = key;
    st[j] = tile;
  }
  bitonic_lds<kChunk, kChunkThreads>(sk, st);
#pragma unroll
  for (int r = 0; r < kChunk / kChunkThreads; ++r) {
    const int j = r * kChunkThreads + threadIdx.x;
    const int64_t i = base + j;
    if (i < n) {
      if (pack) {
        pack_record(pa, state, i, st[j]);
      } else {
        SortItem x;
        x.key = sk[j];
        x.tile = st[j];
        x.aux = 0u;  // the merge passes pack from the encoder outputs
        items[i] = x;
      }
    }
  }
}

// ---------------------------------------------------------------- small segments
// Segments of at most kSmallMax tiles: one workgroup sorts all of a segment's
// keys in LDS and packs the first K, so a call over small modules is one
// launch (two with several segments) instead of a dozen for each.  The path
// above costs about 70 us of launches and their latencies whatever the size;
// this one 10 to 25.
struct SmallSeg {
  int64_t t0, n, cap;
};
__device__ __forceinline__ SmallSeg small_seg(const SmallTable& tb, int i) {
  return SmallSeg{tb.t0[i], tb.t0[i + 1] - tb.t0[i], tb.cap[i]};
}

// K and the eligible tiles of every segment.
__global__ __launch_bounds__(256) void k_small_count(const double* __restrict__ gain, SmallTable tb, uint64_t* kseg) {
  __shared__ uint32_t sw[4];
  const SmallSeg sg = small_seg(tb, blockIdx.x);
  uint32_t c = 0;
  for (int64_t i = threadIdx.x; i < sg.n; i += 256) c += gain_key(gain[sg.t0 + i]) != 0;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint64_t e = (uint64_t)sw[0] + sw[1] + sw[2] + sw[3];
    kseg[2 * blockIdx.x] = e < (uint64_t)sg.cap ? e : (uint64_t)sg.cap;
    kseg[2 * blockIdx.x + 1] = e;
  }
}

template <int M>
__global__ __launch_bounds__(M / 2 < 1024 ? M / 2 : 1024) void k_small_rank(const double* __restrict__ gain, SmallTable tb, int n_seg,
                                                     const uint64_t* __restrict__ kseg, HeaderChunk hc,
                                                     int n_hdr, PackArgs pa, uint64_t* __restrict__ totals) {
  constexpr int THREADS = M / 2 < 1024 ? M / 2 : 1024;
  __shared__ uint64_t sk[M];
  __shared__ uint32_t st[M];
  __shared__ uint64_t s_sum[2];
  __shared__ uint32_t s_el;
  const SmallSeg sg = small_seg(tb, blockIdx.x);
  const bool last = (int)blockIdx.x == n_seg - 1;
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < n_hdr; i += THREADS) pa.out[i] = hc.b[i];
  if (threadIdx.x < 2) s_sum[threadIdx.x] = 0;
  if (threadIdx.x == 0) s_el = 0;
  __syncthreads();
  // records and eligible tiles of the earlier segments
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += THREADS) {
    atomicAdd((unsigned long long*)&s_sum[0], (unsigned long long)kseg[2 * i]);
    atomicAdd((unsigned long long*)&s_sum[1], (unsigned long long)kseg[2 * i + 1]);
  }
  uint32_t c = 0;
  for (int i = threadIdx.x; i < M; i += THREADS) {
    const uint64_t k = i < sg.n ? gain_key(gain[sg.t0 + i]) : 0ull;
    c += k != 0;
    sk[i] = ~k;  // ineligible tiles and padding sort last
    st[i] = (uint32_t)i;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) c += __shfl_xor(c, off, 64);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(&s_el, c);
  bitonic_lds<M, THREADS>(sk, st);
  const uint64_t elig = s_el, off = s_sum[0];
  const uint64_t K = elig < (uint64_t)sg.cap ? elig : (uint64_t)sg.cap;
  const bool fits = pa.h + (off + K) * (uint64_t)pa.L <= pa.cap;
  if (fits)
    for (int i = threadIdx.x; i < (int)K; i += THREADS) {
      const uint32_t t = (uint32_t)sg.t0 + st[i];
      write_record(pa, off + (uint64_t)i, t, (uint32_t)pa.seed[t] | ((uint32_t)pa.scale[t] << 16), load_codes(pa, t));
    }
  if (last && threadIdx.x == 0) {
    totals[0] = off + K;
    totals[1] = s_sum[1] + elig;
    totals[2] = fits ? 0 : 1;  // the totals only grow, so the last segment knows
    totals[3] = 0;
  }
}

// One multiway merge pass: runs of 2^logw sorted items, groups of F runs.
// An item's output slot is the first slot of its group, plus its index in its
// own run, plus, for every other run of the group, the number of that run's
// items that order before it.  That count is found digit by digit in radix
// 2^LOGR: each level probes 2^LOGR - 1 positions of every run, all loads
// independent and issued together (addresses clamped in range, results
// masked), so a level costs one memory round trip.  Wide groups use binary
// digits (F loads per level); the last pass over a few long runs uses base-8
// digits, which cuts the number of round trips by three.
template <int LOGR, int F>
__global__ __launch_bounds__(256) void k_merge_runs(const SortItem* __restrict__ in, uint64_t* state,
                                                    int64_t cap_items, int logw, SortItem* __restrict__ out, int pack,
                                                    PackArgs pa) {
  constexpr int NP = (1 << LOGR) - 1;  // probes per run per level
  const int64_t n = sort_count(state, cap_items);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const SortItem x = in[i];
  const int64_t w = (int64_t)1 << logw;
  const int64_t run = i >> logw;
  const int64_t g0 = run - run % F;
  int64_t len[F];
  int64_t cnt[F];
#pragma unroll
  for (int r = 0; r < F; ++r) {
    const int64_t rem = n - ((g0 + r) << logw);
    len[r] = (g0 + r == run || rem <= 0) ? 0 : (rem < w ? rem : w);
    cnt[r] = 0;
  }
  // largest power of 2^LOGR not above w: the count's top digit is then at most
  // w / top < 2^LOGR
  for (int64_t step = (int64_t)1 << (LOGR * (logw / LOGR)); step >= 1; step >>= LOGR) {
    SortItem y[F][NP];
#pragma unroll
    for (int r = 0; r < F; ++r) {
      const int64_t st = (g0 + r) << logw;
#pragma unroll
      for (int j = 1; j <= NP; ++j) {
        const int64_t probe = cnt[r] + j * step;
        y[r][j - 1] = in[len[r] > 0 ? st + (probe <= len[r] ? probe : len[r]) - 1 : i];
      }
    }
#pragma unroll
    for (int r = 0; r < F; ++r) {
      int c = 0;
#pragma unroll
      for (int j = 1; j <= NP; ++j) c += (int)((cnt[r] + j * step <= len[r]) & kv_less(y[r][j - 1], x));
      cnt[r] += c * step;
    }
  }
  int64_t pos = (g0 << logw) + (i - (run << logw));
#pragma unroll
  for (int r = 0; r < F; ++r) pos += cnt[r];
  if (pack) pack_record(pa, state, pos, x.tile);
  else out[pos] = x;
}

// ---------------------------------------------------------------- radix sort of large survivor sets
// Least-significant-digit radix sort.  A pass is a block histogram (kRsItems
// items per block), a scan per digit over the blocks, and a scatter in which
// every block first orders its items by digit in LDS (index order within a
// digit: within a wavefront by matching digits with ballots, across the
// block's four wavefronts and its rounds through LDS counters) and then writes
// them in that order, so that each digit's run of the block goes out as
// adjacent stores rather than one scattered 16-byte store per lane.
//
// The exact path sorts the whole 64-bit key, eight stable passes of 8 bits
// (the items enter in tile order, so equal keys keep increasing tiles, the
// same total order as the merge path), and packs in the last one.  The fast
// path (CELL) sorts by the 27 leading bits of the range the survivors span,
// three passes of 9 bits; items that share those bits (a handful: 9.2 M
// records of 43 M log-normal gains spread over more cells than there are
// records) are put in order by k_pack_cells.  Each pass moves every item once,
// 0.17 ms for 9.2 M, so the five passes left out are worth 0.85 ms.
constexpr int kRsThreads = 256;
constexpr int kRsRounds = 16;
constexpr int kRsItems = kRsThreads * kRsRounds;
constexpr int kRsMaxBins = 512;
constexpr int64_t kRadixMin = int64_t(1) << 20;  // record caps above this use the radix sort

// An item's sort value: the whole key, or its cell.
template <bool CELL>
__device__ __forceinline__ uint64_t sort_value(const uint64_t key, uint64_t base, int shift0) {
  return CELL ? (key - base) >> shift0 : key;
}

template <int BITS, bool CELL>
__global__ __launch_bounds__(kRsThreads) void k_rs_hist(const SortItem* __restrict__ in, uint64_t* state,
                                                        int64_t cap_items, int clear_hist, int shift,
                                                        uint32_t* __restrict__ hist, int nblk) {
  constexpr int BINS = 1 << BITS;
  __shared__ uint32_t h[BINS];
  for (int d = threadIdx.x; d < BINS; d += kRsThreads) h[d] = 0;
  const int64_t n = sort_count(state, cap_items);
  if (clear_hist && blockIdx.x == 0 && n > 0)  // the fast path's second histogram has been read by now
    for (int b = threadIdx.x; b < kSelBins; b += kRsThreads) state[kHist + kSelBins + b] = 0;
  __syncthreads();
  const uint64_t kb = state[kBase];
  const int s0 = (int)state[kShift];
  const int64_t base = (int64_t)blockIdx.x * kRsItems;
  uint64_t keys[kRsRounds];  // every load issued before the first count
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    const int64_t i = base + r * kRsThreads + threadIdx.x;
    keys[r] = i < n ? in[i].key : 0;
  }
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    const int64_t i = base + r * kRsThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(uint32_t)(sort_value<CELL>(keys[r], kb, s0) >> shift) & (BINS - 1)], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < BINS; d += kRsThreads) hist[(int64_t)d * nblk + blockIdx.x] = h[d];
}

// One block per digit: exclusive scan of the digit's counts over the blocks
// (in place), and the digit's total.
__global__ __launch_bounds__(1024) void k_rs_scan(uint32_t* __restrict__ hist, int nblk, uint32_t* __restrict__ tot) {
  __shared__ uint64_t s_wave[16];
  uint32_t* row = hist + (int64_t)blockIdx.x * nblk;
  uint64_t carry = 0;
  for (int c0 = 0; c0 < nblk; c0 += 1024) {
    const int i = c0 + threadIdx.x;
    const uint64_t v = i < nblk ? row[i] : 0;
    uint64_t t;
    const uint64_t incl = scan1024(v, s_wave, &t);
    if (i < nblk) row[i] = (uint32_t)(carry + incl - v);
    carry += t;
  }
  if (threadIdx.x == 0) tot[blockIdx.x] = (uint32_t)carry;
}

template <int BITS, bool CELL>
__global__ __launch_bounds__(kRsThreads) void k_rs_scatter(const SortItem* __restrict__ in, SortItem* __restrict__ out,
                                                           uint64_t* state, int64_t cap_items, int shift,
                                                           const uint32_t* __restrict__ hist, int nblk,
                                                           const uint32_t* __restrict__ tot, int pack, PackArgs pa) {
  constexpr int BINS = 1 << BITS;
  constexpr int NB = BINS / kRsThreads;       // digits per thread: NB t .. NB t + NB - 1
  __shared__ uint32_t dbase[BINS];            // first slot of each digit for this block
  __shared__ uint32_t lstart[BINS];           // first place of each digit in the block's digit order
  __shared__ uint32_t lcur[BINS];             // next place of each digit in that order
  __shared__ uint32_t wc[kRsThreads / 64][BINS];  // items per digit of each wavefront in the round
  __shared__ uint32_t s_wave[kRsThreads / 64];
  __shared__ SortItem s_items[kRsItems];      // the block's items in digit order (stable within a digit)
  const int64_t n = sort_count(state, cap_items);
  const int64_t base = (int64_t)blockIdx.x * kRsItems;
  if (base >= n) return;  // uniform per block
  const uint64_t kb = state[kBase];
  const int s0 = (int)state[kShift];
  auto digit = [&](uint64_t key) -> uint32_t {
    return (uint32_t)(sort_value<CELL>(key, kb, s0) >> shift) & (BINS - 1);
  };
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // exclusive scan of the digits' values (thread t holds digits NB t ..) over
  // the block's threads, in place
  auto scan_digits = [&](uint32_t (&v)[NB]) {
    uint32_t own = 0;
#pragma unroll
    for (int q = 0; q < NB; ++q) own += v[q];
    uint32_t x = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if (lane >= o) x += y;
    }
    if (lane == 63) s_wave[w] = x;
    __syncthreads();
    uint32_t run = x - own;
#pragma unroll
    for (int k = 0; k < kRsThreads / 64; ++k) run += k < w ? s_wave[k] : 0u;
    __syncthreads();  // s_wave is reused by the next scan
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      const uint32_t c = v[q];
      v[q] = run;
      run += c;
    }
  };
  // digit bases: exclusive scan of the digit totals, plus this block's prefix
  uint32_t dv[NB];
#pragma unroll
  for (int q = 0; q < NB; ++q) dv[q] = tot[NB * t + q];
  scan_digits(dv);
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    dbase[NB * t + q] = dv[q] + hist[(int64_t)(NB * t + q) * nblk + blockIdx.x];
    lcur[NB * t + q] = 0;
  }
  const uint64_t lt = lanemask_lt();
  // every round's item is loaded before the first round (one wait, not one
  // per round)
  SortItem xs[kRsRounds];
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
    const int64_t i = base + r * kRsThreads + t;
    xs[r].key = 0; xs[r].tile = 0; xs[r].aux = 0;
    if (i < n) xs[r] = in[i];
  }
  // the block's count of each digit, then where each digit's run starts in
  // the block's digit order
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r)
    if (base + r * kRsThreads + t < n) atomicAdd(&lcur[digit(xs[r].key)], 1u);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NB; ++q) dv[q] = lcur[NB * t + q];
  scan_digits(dv);
#pragma unroll
  for (int q = 0; q < NB; ++q) {
    lstart[NB * t + q] = dv[q];
    lcur[NB * t + q] = dv[q];
  }
  // place every item in the block's digit order: within a wavefront by
  // matching digits with ballots, across the block's wavefronts and its
  // rounds through LDS counters (index order within a digit)
#pragma unroll
  for (int r = 0; r < kRsRounds; ++r) {
#pragma unroll
    for (int k = 0; k < kRsThreads / 64; ++k)
#pragma unroll
      for (int q = 0; q < NB; ++q) wc[k][NB * t + q] = 0;
    __syncthreads();
    const int64_t i = base + r * kRsThreads + t;
    const bool valid = i < n;
    const SortItem x = xs[r];
    const uint32_t d = digit(x.key);
    // lanes of this wavefront holding the same digit
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const uint64_t bal = __ballot((d >> b) & 1u);
      same &= ((d >> b) & 1u) ? bal : ~bal;
    }
    const uint32_t rank = (uint32_t)__popcll(same & lt);
    if (valid && rank == 0) wc[w][d] = (uint32_t)__popcll(same);
    __syncthreads();
    if (valid) {
      uint32_t lp = lcur[d] + rank;
#pragma unroll
      for (int k = 0; k < kRsThreads / 64; ++k) lp += k < w ? wc[k][d] : 0u;
      s_items[lp] = x;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NB; ++q) {
      uint32_t add = 0;
#pragma unroll
      for (int k = 0; k < kRsThreads / 64; ++k) add += wc[k][NB * t + q];
      lcur[NB * t + q] += add;
    }
  }
  __syncthreads();
  // write the block's items in digit order: consecutive threads take
  // consecutive items, so each digit's run goes out as adjacent stores
  const int64_t m = n - base < kRsItems ? n - base : kRsItems;
#pragma unroll 4
  for (int r = 0; r < kRsRounds; ++r) {
    const int j = r * kRsThreads + t;
    if (j < m) {
      const SortItem x = s_items[j];
      const uint32_t d = digit(x.key);
      const uint32_t off = dbase[d] + ((uint32_t)j - lstart[d]);
      if (pack) pack_record(pa, state, (int64_t)off, x.tile, x.aux, load_codes(pa, x.tile));
      else out[off] = x;
    }
  }
}

// Last step of the fast path's radix sort: the items are in cell order; each
// finds its place among the items of its own cell (by key, then tile) and is
// packed.  A cell of more than kCellMax items (equal gains, or gains that agree
// in more than 20 mantissa bits) goes to `big`, as its first item's place.
// A block's keys (and kCellMax to either side) are compared in LDS, while the
// gathers of its tiles' codes, the bulk of the memory time, are in flight.
constexpr int kCellMax = 64;
constexpr int kPcRounds = 4;
constexpr int kPcItems = 256 * kPcRounds;
__global__ __launch_bounds__(256) void k_pack_cells(const SortItem* __restrict__ in, uint64_t* state, int64_t cap_items,
                                                    uint32_t* __restrict__ big, PackArgs pa) {
  __shared__ uint64_t sk[kPcItems + 2 * kCellMax];
  __shared__ uint32_t st[kPcItems + 2 * kCellMax];
  const int64_t n = sort_count(state, cap_items);
  const int64_t base = (int64_t)blockIdx.x * kPcItems;
  if (base >= n) return;  // uniform per block
  const uint64_t kb = state[kBase];
  const int s0 = (int)state[kShift];
  SortItem x[kPcRounds];
#pragma unroll
  for (int r = 0; r < kPcRounds; ++r) {
    const int64_t i = base + r * 256 + threadIdx.x;
    x[r] = in[i < n ? i : n - 1];
  }
  if (threadIdx.x < 2 * kCellMax) {  // the halo; places outside [0, n) are never compared
    const int j = threadIdx.x < kCellMax ? (int)threadIdx.x : kPcItems + (int)threadIdx.x;
    const int64_t i = base + j - kCellMax;
    if (i >= 0 && i < n) { sk[j] = in[i].key; st[j] = in[i].tile; }
  }
  Codes c[kPcRounds];
#pragma unroll
  for (int r = 0; r < kPcRounds; ++r) c[r] = load_codes(pa, x[r].tile);
#pragma unroll
  for (int r = 0; r < kPcRounds; ++r) {
    sk[kCellMax + r * 256 + threadIdx.x] = x[r].key;
    st[kCellMax + r * 256 + threadIdx.x] = x[r].tile;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPcRounds; ++r) {
    const int64_t i = base + r * 256 + threadIdx.x;
    if (i >= n) break;
    const int at = kCellMax + r * 256 + threadIdx.x;
    const uint64_t cell = sort_value<true>(x[r].key, kb, s0);
    const int lo = i < kCellMax ? (int)i : kCellMax;                 // items before and after this one in reach
    const int hi = n - 1 - i < kCellMax ? (int)(n - 1 - i) : kCellMax;
    int64_t pos = i;
    int d = 1;
    for (; d <= lo; ++d) {
      const SortItem y{sk[at - d], st[at - d], 0u};
      if (sort_value<true>(y.key, kb, s0) != cell) break;
      pos -= kv_less(x[r], y);
    }
    int e = 1;
    for (; e <= hi; ++e) {
      const SortItem y{sk[at + e], st[at + e], 0u};
      if (sort_value<true>(y.key, kb, s0) != cell) break;
      pos += kv_less(y, x[r]);
    }
    if (d - 1 + e - 1 < kCellMax)
      pack_record(pa, state, pos, x[r].tile, x[r].aux, c[r]);
    else if (d == 1)  // at most n / kCellMax of them, and `big` has room for n / 8
      big[atomicAdd((unsigned long long*)&state[kBig], 1ull)] = (uint32_t)i;
  }
}

// The cells that k_pack_cells left, one workgroup each: up to kCellSort items
// are sorted in LDS and packed, a larger cell sets kAgain.  10 M records of 43 M
// gains, 2% of these in groups of 128 equal ones: 1.4 ms, 3.2 when such a call
// ran both paths; none to sort: 5 us.
constexpr int kCellSort = 4096;
constexpr int kCellBlocks = 128;
__global__ __launch_bounds__(256) void k_sort_cells(const SortItem* __restrict__ in, uint64_t* state, int64_t cap_items,
                                                    const uint32_t* __restrict__ big, PackArgs pa) {
  __shared__ uint64_t sk[kCellSort];
  __shared__ uint32_t st[kCellSort];
  __shared__ int s_m;
  const int64_t n = sort_count(state, cap_items);
  const uint64_t n_big = state[kBig], kb = state[kBase];
  const int s0 = (int)state[kShift];
  for (uint64_t c = blockIdx.x; c < n_big; c += gridDim.x) {
    const int64_t i0 = big[c];
    const uint64_t cell = sort_value<true>(in[i0].key, kb, s0);
    if (threadIdx.x == 0) s_m = 0;
    __syncthreads();
    int m = 0;  // items of the cell among the next kCellSort + 256 (they are adjacent)
    for (int k = threadIdx.x; k < kCellSort + 256; k += 256) {
      if (i0 + k >= n) break;
      const SortItem x = in[i0 + k];
      if (sort_value<true>(x.key, kb, s0) != cell) break;
      if (k < kCellSort) {
        sk[k] = x.key;
        st[k] = x.tile;
      }
      ++m;
    }
    if (m) atomicAdd(&s_m, m);
    __syncthreads();
    m = s_m;
    if (m > kCellSort) {  // uniform
      if (threadIdx.x == 0) state[kAgain] = kAgainLate;
      __syncthreads();
      continue;
    }
    const int M = m <= 512 ? 512 : kCellSort;
    for (int k = m + threadIdx.x; k < M; k += 256) {  // sorts behind every item
      sk[k] = ~0ull;
      st[k] = 0xFFFFFFFFu;
    }
    if (M == 512) bitonic_lds<512, 256>(sk, st);
    else bitonic_lds<kCellSort, 256>(sk, st);
    for (int k = threadIdx.x; k < m; k += 256) pack_record(pa, state, i0 + k, st[k]);
    __syncthreads();  // sk, st and s_m are used again
  }
}

// ---------------------------------------------------------------- workspace
// Items beyond the record cap that the fast path may sort: the keys that share
// the K-th key's 24 leading bits (about n 2^-12 times the density of the gains'
// logarithms there).
static size_t cap_slack(size_t n_tiles) { return 4096 + n_tiles / 256; }

size_t rank_ws_bytes(size_t n_tiles, size_t k_cap, size_t n_seg) {
  const size_t cap = k_cap + cap_slack(n_tiles);
  const size_t max_blocks = (n_tiles + kItems - 1) / kItems + 1;
  const size_t rs_blocks = (cap + kRsItems - 1) / kRsItems;
  size_t b = 0;
  b += align_up(cap * sizeof(SortItem), 256) * 2;
  b += align_up((max_blocks + 1) * 8, 256) * 2;
  b += align_up((size_t)kStateWords * 8, 256);
  b += align_up(rs_blocks * kRsMaxBins * 4, 256) + align_up(kRsMaxBins * 4, 256);
  b += align_up(n_seg * 16, 256);
  return b;
}

RankWs carve_rank(void* base, size_t n_tiles, size_t k_cap, size_t n_seg) {
  const size_t cap = k_cap + cap_slack(n_tiles);
  const size_t max_blocks = (n_tiles + kItems - 1) / kItems + 1;
  char* p = static_cast<char*>(base);
  RankWs w;
  w.items_a = reinterpret_cast<SortItem*>(p); p += align_up(cap * sizeof(SortItem), 256);
  w.items_b = reinterpret_cast<SortItem*>(p); p += align_up(cap * sizeof(SortItem), 256);
  w.blk_a = reinterpret_cast<uint64_t*>(p); p += align_up((max_blocks + 1) * 8, 256);
  w.blk_b = reinterpret_cast<uint64_t*>(p); p += align_up((max_blocks + 1) * 8, 256);
  w.state = reinterpret_cast<uint64_t*>(p); p += align_up((size_t)kStateWords * 8, 256);
  w.rs_nblk = (cap + kRsItems - 1) / kRsItems;
  w.rs_hist = reinterpret_cast<uint32_t*>(p); p += align_up(w.rs_nblk * kRsMaxBins * 4, 256);
  w.rs_tot = reinterpret_cast<uint32_t*>(p); p += align_up(kRsMaxBins * 4, 256);
  w.kseg = reinterpret_cast<uint64_t*>(p);
  w.cap = cap;
  w.max_blocks = max_blocks;
  (void)n_seg;
  return w;
}

hipError_t launch_rank_init(const RankWs* ws, const uint8_t* hdr, size_t n_hdr, uint8_t* stream_out, hipStream_t st) {
  for (size_t o = 0; o == 0 || o < n_hdr; o += sizeof(HeaderChunk)) {
    HeaderChunk hc;
    const size_t k = n_hdr - o < sizeof hc ? n_hdr - o : sizeof hc;
    memcpy(hc.b, hdr + o, k);
    hipLaunchKernelGGL(k_rank_init, dim3(1), dim3(256), 0, st, ws && o == 0 ? ws->state : (uint64_t*)nullptr, hc, (int)k,
                       stream_out + o);
  }
  return hipGetLastError();
}

hipError_t launch_rank_totals(const RankWs& ws, uint64_t* dst, hipStream_t st) {
  hipLaunchKernelGGL(k_rank_totals, dim3(1), dim3(64), 0, st, ws.state, dst);
  return hipGetLastError();
}

bool rank_small(int64_t max_n, size_t n_seg) { return max_n <= kSmallMax && n_seg <= (size_t)kSmallSegs; }

hipError_t launch_rank_small(const double* gain, const SmallTable& tb, int n_seg, int64_t max_n, const RankWs& ws,
                             const HeaderChunk& hc, int n_hdr, const PackArgs& pa, uint64_t* totals, hipStream_t st) {
  if (n_seg > 1) hipLaunchKernelGGL(k_small_count, dim3((unsigned)n_seg), dim3(256), 0, st, gain, tb, ws.kseg);
  if (max_n <= 1024)
    hipLaunchKernelGGL((k_small_rank<1024>), dim3((unsigned)n_seg), dim3(512), 0, st, gain, tb, n_seg, ws.kseg,
                       hc, n_hdr, pa, totals);
  else if (max_n <= 2048)
    hipLaunchKernelGGL((k_small_rank<2048>), dim3((unsigned)n_seg), dim3(1024), 0, st, gain, tb, n_seg, ws.kseg,
                       hc, n_hdr, pa, totals);
  else
    hipLaunchKernelGGL((k_small_rank<kSmallMax>), dim3((unsigned)n_seg), dim3(1024), 0, st, gain, tb, n_seg, ws.kseg,
                       hc, n_hdr, pa, totals);
  return hipGetLastError();
}

// Sort of the survivors in items_a (at most cap_items, the count in the state)
// by chunks in LDS, then multiway merges; the final pass packs the records.
static void sort_and_pack(const RankWs& ws, int64_t cap_items, int clear_hist, const PackArgs& pa, hipStream_t st) {
  int passes = 0;
  for (int logw = kLogChunk; ((int64_t)1 << logw) < cap_items;
       logw += cap_items <= ((int64_t)4 << logw) ? 2 : kLogFan)
    ++passes;
  hipLaunchKernelGGL(k_sort_chunks, dim3((unsigned)((cap_items + kChunk - 1) / kChunk)), dim3(kChunkThreads), 0, st,
                     ws.items_a, ws.state, cap_items, clear_hist, passes == 0 ? 1 : 0, pa);
  SortItem* in = ws.items_a;
  SortItem* out = ws.items_b;
  int done = 0;
  for (int logw = kLogChunk; ((int64_t)1 << logw) < cap_items;) {
    const dim3 grid((unsigned)((cap_items + 255) / 256));
    const int last = ++done == passes ? 1 : 0;
    if (cap_items <= ((int64_t)4 << logw)) {  // at most four runs left: one base-8 pass
      hipLaunchKernelGGL((k_merge_runs<3, 4>), grid, dim3(256), 0, st, in, ws.state, cap_items, logw, out, last, pa);
      logw += 2;
    } else {
      hipLaunchKernelGGL((k_merge_runs<1, kFan>), grid, dim3(256), 0, st, in, ws.state, cap_items, logw, out, last, pa);
      logw += kLogFan;
    }
    SortItem* t = in; in = out; out = t;
  }
}

// One segment: count -> select -> compact -> sort -> pack, all on the device.
// `cap` bounds K (the budget's record count, at most n); grids are sized by it
// and kernels read the actual K from the state.  exact: the path that handles
// any number of equal gains, else the fast one (see k_compact_fast).
hipError_t launch_rank_segment(const double* gain, int64_t t0, int64_t n, int64_t cap, const RankWs& ws,
                               const PackArgs& pa, RankPath path, hipStream_t st) {
  const bool exact = path != kRankFast;
  const double* g = gain + t0;
  int64_t cb = (n + kThreads - 1) / kThreads;
  if (cb > 512) cb = 512;
  if (cb < 1) cb = 1;
  if (path == kRankResume) hipLaunchKernelGGL(k_rank_resume, dim3(1), dim3(64), 0, st, ws.state);
  else hipLaunchKernelGGL(k_count_hist, dim3((unsigned)cb), dim3(kThreads), 0, st, g, n, ws.state);
  // passes 1..5 over the digits 12, 12, 12, 12 and 4 bits below the top one
  const int shifts[6] = {64 - kSelBits, 64 - 2 * kSelBits, 64 - 3 * kSelBits, 64 - 4 * kSelBits, 64 - 5 * kSelBits, 0};
  const int widths[6] = {kSelBits, kSelBits, kSelBits, kSelBits, kSelBits, 4};
  // fewer blocks than the counting pass: every block repeats the pick (a read
  // of the 32 KB histogram), and the keys under the prefix thin out fast
  int64_t sb = (n + 4 * kThreads - 1) / (4 * kThreads);
  // (the fast path's one pass reads every gain: on many, twice the machine)
  const int64_t sb_max = !exact && n > ((int64_t)1 << 22) ? 512 : 128;
  if (sb > sb_max) sb = sb_max;
  if (sb < 1) sb = 1;
  const int n_pass = exact ? 5 : 1;
  int64_t cap_items = cap + (int64_t)cap_slack((size_t)n);
  if (cap_items > n) cap_items = n;
  // (the merges of smaller caps do not mind equal gains; the look ahead has one
  // of the pass's blocks, of 128 or more)
  const int probe = !exact && cap > 0 && cap_items > kRadixMin ? 1 : 0;
  for (int pass = path == kRankResume ? 2 : 1; pass <= n_pass; ++pass)
    hipLaunchKernelGGL(k_select_pass, dim3((unsigned)sb), dim3(kThreads), 0, st, g, n, ws.state,
                       (int64_t)(cap > 0 ? cap : 0), pass, shifts[pass - 1], widths[pass - 1], shifts[pass],
                       widths[pass], exact ? 0 : 1, probe);
  if (!exact) {
    // small segments in shorter chunks, so that more blocks share them
    const int rounds = n > ((int64_t)1 << 22) ? 16 : 4;
    int64_t nb = (n + kThreads * rounds - 1) / (kThreads * rounds);
    nb = nb < 1 ? 1 : nb > 1536 ? 1536 : nb;
    if (rounds == 16)
      hipLaunchKernelGGL((k_compact_fast<16>), dim3((unsigned)nb), dim3(kThreads), 0, st, g, pa.seed, pa.scale, t0, n,
                         ws.state, (uint64_t)cap_items, ws.items_a);
    else
      hipLaunchKernelGGL((k_compact_fast<4>), dim3((unsigned)nb), dim3(kThreads), 0, st, g, pa.seed, pa.scale, t0, n,
                         ws.state, (uint64_t)cap_items, ws.items_a);
    if (cap <= 0 || n <= 0) return hipGetLastError();
    if (cap_items <= kRadixMin) {
      sort_and_pack(ws, cap_items, 1, pa, st);
      return hipGetLastError();
    }
    const int nblk = (int)((cap_items + kRsItems - 1) / kRsItems);
    SortItem* in = ws.items_a;
    SortItem* out = ws.items_b;
    for (int pass = 0; pass < 3; ++pass) {
      hipLaunchKernelGGL((k_rs_hist<9, true>), dim3((unsigned)nblk), dim3(kRsThreads), 0, st, in, ws.state, cap_items,
                         pass == 0 ? 1 : 0, 9 * pass, ws.rs_hist, nblk);
      hipLaunchKernelGGL(k_rs_scan, dim3(512), dim3(1024), 0, st, ws.rs_hist, nblk, ws.rs_tot);
      hipLaunchKernelGGL((k_rs_scatter<9, true>), dim3((unsigned)nblk), dim3(kRsThreads), 0, st, in, out, ws.state,
                         cap_items, 9 * pass, ws.rs_hist, nblk, ws.rs_tot, 0, pa);
      SortItem* tt = in; in = out; out = tt;
    }
    hipLaunchKernelGGL(k_pack_cells, dim3((unsigned)((cap_items + kPcItems - 1) / kPcItems)), dim3(256), 0, st, in, ws.state,
                       cap_items, ws.rs_hist, pa);  // (the digit counts have been read)
    hipLaunchKernelGGL(k_sort_cells, dim3(kCellBlocks), dim3(256), 0, st, in, ws.state, cap_items, ws.rs_hist, pa);
    return hipGetLastError();
  }
  // the first compaction launch finishes the select and records the totals
  int64_t nbc = (n + kItems - 1) / kItems;
  if (nbc < 1) nbc = 1;
  hipLaunchKernelGGL(k_compact_count, dim3((unsigned)nbc), dim3(kThreads), 0, st, g, n, ws.state, ws.blk_a, ws.blk_b);
  hipLaunchKernelGGL(k_compact_scan, dim3(1), dim3(1024), 0, st, ws.blk_a, ws.blk_b, nbc, ws.state);
  if (cap <= 0 || n <= 0) return hipGetLastError();
  hipLaunchKernelGGL(k_compact_write, dim3((unsigned)nbc), dim3(kThreads), 0, st, g, pa.seed, pa.scale, t0, n, ws.state,
                     ws.blk_a, ws.blk_b, ws.items_a);
  // sort the survivors ascending on (~key, tile)
  if (cap > kRadixMin) {
    const int nblk = (int)((cap + kRsItems - 1) / kRsItems);
    SortItem* in = ws.items_a;
    SortItem* out = ws.items_b;
    for (int pass = 0; pass < 8; ++pass) {
      hipLaunchKernelGGL((k_rs_hist<8, false>), dim3((unsigned)nblk), dim3(kRsThreads), 0, st, in, ws.state, cap, 0,
                         8 * pass, ws.rs_hist, nblk);
      hipLaunchKernelGGL(k_rs_scan, dim3(256), dim3(1024), 0, st, ws.rs_hist, nblk, ws.rs_tot);
      hipLaunchKernelGGL((k_rs_scatter<8, false>), dim3((unsigned)nblk), dim3(kRsThreads), 0, st, in, out, ws.state, cap,
                         8 * pass, ws.rs_hist, nblk, ws.rs_tot, pass == 7 ? 1 : 0, pa);
      SortItem* tt = in; in = out; out = tt;
    }
    return hipGetLastError();
  }
  sort_and_pack(ws, cap, 0, pa, st);
  return hipGetLastError();
}

}  // namespace awsrc
