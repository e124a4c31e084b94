// selkv_select: per-head top-m_s selection of Sec. 3.3 (Eq. 2).
//
// A head is handled by `split` workgroups of 16 waves (one when the call has
// heads enough to fill the chip).  Each of them finds, from the whole head,
// the m_s-th largest score T and how many scores equal to T must be taken
// (`need`), the same in every workgroup, and compacts its own share of the
// positions: no scratch memory and no hand-over between workgroups.
//
// Threshold, heads of at most kColumnsMax candidates (column path):
//   sample   4096 scores at evenly spaced positions; a histogram of those
//            above -inf over their own key range gives a band of scores
//            around the sample rank where T is expected (128 sample ranks on
//            either side).  Short heads skip this: their band is every
//            score.
//   band     one pass over the scores, as floats: scores above the band are
//            counted per wave, scores inside it go to the thread's own column
//            in LDS (an unconditional store at the column's end, which moves
//            up when the score was in the band: no atomics, ballots or
//            branches).  The waves take steps of 64 candidates in turn, so
//            that scores which rise or fall along the sequence fill all
//            columns alike: with one contiguous run per wave, a band whose
//            scores lie together filled the columns of one wave, and a
//            102384-candidate head whose scores grow tenfold took 193 us
//            instead of 27
//   resolve  T is located among the staged scores by one histogram of their
//            order-preserving keys and a ranking of the few in its bin; the
//            staged scores then complete the counts before the share
// Where the band misses T, a column overflows (many equal scores) or a NaN
// turns up, and for longer heads, each workgroup works on order keys instead:
//   band     unless it missed T or, by the sample, would overflow too: one
//            pass with wave-aggregated appends to one list
//   pass 0   the head's smallest and largest key above that of -inf, and
//            how many keys lie above it (-inf marks candidates that must not
//            be chosen; when fewer than m_s keys lie above, every key and
//            the whole key range are used instead)
//   pass 1   histogram of d >> s over 4096 LDS bins (integer atomics), d the
//            offset from the smallest key and s the smallest shift that fits
//            the key range into them, so the bins span the scores present
//   pass 2   the keys of the bin holding T are copied into LDS and the s low
//            bits are resolved there in passes of at most 10 bits; a bin too
//            large for LDS is resolved with global passes instead
//   count    keys > T and == T before the share
// Either way the result is the exact m_s-th largest key: the paths differ
// only in cost.  Compaction: the share is walked in rounds of one block of up
// to 1024 candidates per wave.  A block is held in registers; its counts meet
// those of the other waves in LDS, and the wave keeps every key > T and the
// first `need` keys == T (lowest positions win ties), ranking them with
// ballots, so kept and evicted positions come out ascending.  The m_r' recent
// positions are appended to the kept list.  Outputs do not depend on
// scheduling: bitwise deterministic.
//
// What it took with one workgroup per head and staging through ballots and
// atomics, and now: 8 heads of 102384 candidates 80 -> 27 us (16 workgroups
// per head; the sample's loads take 5 us of it, the band pass 9 us), 8 heads
// of 8176 20 -> 13 us, 256 heads of 32752 39 -> 30 us (a 34 MB read and as
// much written take 14 us) and of 102384 105 -> 71 us; past the columns, 4
// heads of 299984 349 -> 134 us.
#include <type_traits>

#include "common.hpp"
#include "internal.hpp"

namespace selkv {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / 64;
constexpr int kIter = 256;        // keys of one wave step (four per lane: positions e * 64 + lane)
constexpr int kRing = 8;          // wave steps whose loads are in flight together
constexpr int kSample = 4096;     // sampled keys (four per thread)
constexpr int kBandRanks = 128;   // sample ranks on either side of T's expected rank
constexpr int kHistBatch = 16;    // score loads in flight per thread
constexpr int kTopBits = 12;
constexpr int kTopBins = 1 << kTopBits;
constexpr int kLowBits = 10;      // bits per pass below the top bins
constexpr int kCandCap = 32768;   // whole-head path: staged keys (128 KB)
constexpr int kColumn = 32;       // column path: LDS slots per thread (128 KB in all)
constexpr int kColumnFull = 24;   // entries a column may hold at the end of a batch of 8
// Heads of at most so many steps of 64 candidates per wave are staged in full:
// beyond, the passes over what is staged cost more than the sample (9000
// candidates, 8 heads 13.2 us with the sample and 13.7 without, 600 heads 39.9
// and 40.6; 16400: 14.4 and 17.4; 24000: 16.1 and 21.8; 6000: 13.0 and 12.2)
constexpr int kAllSteps = 8;
// a band of 256 sample ranks holds 1/16 of the candidates: 8 per column at kColumnsMax
constexpr int kColumnsMax = 128 * 1024;
constexpr int kMaxSplit = 16;     // workgroups per head
// a key range of up to 2^32 - 1 fits the top bins at a shift of at most 20,
// which two low passes resolve
static_assert(kAllSteps <= kColumnFull, "short heads fit the columns");
static_assert(kTopBits + 2 * kLowBits == 32, "two low passes cover the bits below the top bins");

constexpr uint32_t kNegInfKey = 0x007fffffu;   // order_key(-inf)

__device__ __forceinline__ uint32_t order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if (u == 0x80000000u) u = 0u;  // -0 ranks with +0
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// The score of an order key (order_key's inverse; keys above that of +inf and
// below that of -inf give NaN, which compares false).
__device__ __forceinline__ float key_score(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Exclusive prefix sum over the block; `total` receives the block sum.
__device__ __forceinline__ int block_exclusive_scan(int v, int* lds_waves, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int incl = wave_inclusive_scan(v, lane);
  if (lane == 63) lds_waves[wave] = incl;
  __syncthreads();
  if (wave == 0) {
    int w = lane < kWaves ? lds_waves[lane] : 0;
    const int wi = wave_inclusive_scan(w, lane);
    if (lane < kWaves) lds_waves[kWaves + lane] = wi - w;   // exclusive wave offsets
    if (lane == kWaves - 1) lds_waves[2 * kWaves] = wi;
  }
  __syncthreads();
  const int r = lds_waves[kWaves + wave] + incl - v;
  total = lds_waves[2 * kWaves];
  __syncthreads();
  return r;
}

struct Pick {
  uint32_t bin;   // the digit of the need-th largest key
  int need;       // its rank among the keys of that bin
  int count;      // keys in that bin
};

// Walks the nbins bins from the top (thread t covers nbins / kThreads
// consecutive bins, or one) and finds the bin holding the need-th largest key.
__device__ Pick find_bin(const int* hist, int nbins, int need, int* scan_lds, Pick* sh) {
  const int tid = threadIdx.x;
  const int bpt = nbins > kThreads ? nbins / kThreads : 1;
  const int top = nbins - 1 - tid * bpt;   // this thread's highest bin
  int c = 0;
  for (int k = 0; k < bpt; ++k)
    if (top - k >= 0) c += hist[top - k];
  int total;
  const int excl = block_exclusive_scan(c, scan_lds, total);
  if (excl < need && excl + c >= need) {
    int cum = excl;
    for (int k = 0; k < bpt; ++k) {
      const int h = hist[top - k];
      if (cum + h >= need) {
        sh->bin = (uint32_t)(top - k);
        sh->need = need - cum;
        sh->count = h;
        break;
      }
      cum += h;
    }
  }
  __syncthreads();
  const Pick r = *sh;
  __syncthreads();
  return r;
}

// Histogram of digit (d >> shift) & (nbins - 1), d = key - base, over the
// keys >= kfloor whose d matches prefix under mask: from the global scores
// (LDS_SRC false) or the staged offsets (which are d already, all admitted).
template <bool LDS_SRC>
__device__ void histogram(const float* s, const uint32_t* cand, int count, uint32_t kfloor, uint32_t base, int shift,
                          int nbins, uint32_t mask, uint32_t prefix, int* hist) {
  const int tid = threadIdx.x;
  for (int b = tid; b < nbins; b += kThreads) hist[b] = 0;
  __syncthreads();
  const uint32_t dmask = (uint32_t)nbins - 1u;
  if constexpr (LDS_SRC) {
    for (int j = tid; j < count; j += kThreads) {
      const uint32_t d = cand[j];
      if ((d & mask) == prefix) atomicAdd(&hist[(d >> shift) & dmask], 1);
    }
  } else {
    for (int j0 = tid; j0 < count; j0 += kThreads * kHistBatch) {
      float v[kHistBatch];
#pragma unroll
      for (int u = 0; u < kHistBatch; ++u) v[u] = s[min(j0 + u * kThreads, count - 1)];
#pragma unroll
      for (int u = 0; u < kHistBatch; ++u) {
        const uint32_t key = order_key(v[u]), d = key - base;
        if (j0 + u * kThreads < count && key >= kfloor && (d & mask) == prefix)
          atomicAdd(&hist[(d >> shift) & dmask], 1);
      }
    }
  }
  __syncthreads();
}

// Block-wide min / max / sum of the per-thread partial ranges, visible to
// every thread.
__device__ void reduce_range(uint32_t lo, uint32_t hi, int c, uint32_t* red, uint32_t& kmin, uint32_t& kmax,
                             int& count) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 32; o >= 1; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, 64));
    c += __shfl_xor(c, o, 64);
  }
  if (lane == 0) {
    red[wave] = lo;
    red[kWaves + wave] = hi;
    red[2 * kWaves + wave] = (uint32_t)c;
  }
  __syncthreads();
  lo = red[0];
  hi = red[kWaves];
  c = (int)red[2 * kWaves];
  for (int w = 1; w < kWaves; ++w) {
    lo = min(lo, red[w]);
    hi = max(hi, red[kWaves + w]);
    c += (int)red[2 * kWaves + w];
  }
  kmin = lo;
  kmax = hi;
  count = c;
  __syncthreads();
}

// Smallest and largest key above the key of -inf, and how many keys are
// above it, visible to every thread (lo > hi when there are none).
__device__ void key_range(const float* s, int count, uint32_t* red, uint32_t& kmin, uint32_t& kmax, int& above) {
  const int tid = threadIdx.x;
  uint32_t lo = 0xffffffffu, hi = 0u;
  int c = 0;
  for (int j0 = tid; j0 < count; j0 += kThreads * kHistBatch) {
    float v[kHistBatch];
#pragma unroll
    for (int u = 0; u < kHistBatch; ++u) v[u] = s[min(j0 + u * kThreads, count - 1)];
#pragma unroll
    for (int u = 0; u < kHistBatch; ++u) {
      const uint32_t key = order_key(v[u]);
      if (j0 + u * kThreads < count && key > kNegInfKey) {
        lo = min(lo, key);
        hi = max(hi, key);
        ++c;
      }
    }
  }
  reduce_range(lo, hi, c, red, kmin, kmax, above);
}

// The smallest shift that fits the key range [kmin, kmax] into the top bins.
__device__ __forceinline__ int top_shift(uint32_t kmin, uint32_t kmax) {
  int hb = 0;
  while (hb < 32 && ((kmax - kmin) >> hb) >= (uint32_t)kTopBins) ++hb;
  return hb;
}

// Walks the wave's segment [begin, end) of the scores: step t holds
// positions begin + t * kIter + e * 64 + lane (e = 0 .. 3), so every load
// instruction reads 256 contiguous bytes and the keys of a step ascend in
// (e, lane) order.  The loads of kRing steps are issued together, the next
// group's before the current group is handled.  f(t, v) gets the lane's four
// scores of step t; reads past the end are clamped (the caller masks them by
// position).
template <class F>
__device__ __forceinline__ void walk_segment(const float* s, int begin, int end, F&& f) {
  const int lane = threadIdx.x & 63;
  const int steps = (end - begin + kIter - 1) / kIter;
  if (steps <= 0) return;
  float cur[kRing][4], nxt[kRing][4];
  auto load = [&](float (&v)[kRing][4], int g) {
#pragma unroll
    for (int r = 0; r < kRing; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[r][e] = s[min(begin + (g + r) * kIter + e * 64 + lane, end - 1)];
  };
  load(cur, 0);
  for (int g = 0; g < steps; g += kRing) {
    if (g + kRing < steps) load(nxt, g + kRing);
#pragma unroll
    for (int r = 0; r < kRing; ++r)
      if (g + r < steps) f(g + r, cur[r]);
#pragma unroll
    for (int r = 0; r < kRing; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) cur[r][e] = nxt[r][e];
  }
}

// Resolves the need-th largest of the staged offsets cand[0 .. count) whose
// values lie in [0, 2^32): the offset itself, and `need` becomes its rank
// among the offsets equal to it.
__device__ uint32_t resolve_staged(const uint32_t* cand, int count, uint32_t dmax, int& need, int* hist, int* scan_lds,
                                   Pick* sh) {
  int hb = top_shift(0u, dmax);
  histogram<true>(nullptr, cand, count, 0u, 0u, hb, kTopBins, 0u, 0u, hist);
  const Pick pk = find_bin(hist, kTopBins, need, scan_lds, sh);
  uint32_t prefix = pk.bin << hb;
  uint32_t mask = hb >= 32 ? 0u : ~0u << hb;
  need = pk.need;
  while (hb > 0) {
    const int shift = hb > kLowBits ? hb - kLowBits : 0;
    const int nbins = 1 << (hb - shift);
    histogram<true>(nullptr, cand, count, 0u, 0u, shift, nbins, mask, prefix, hist);
    const Pick q = find_bin(hist, nbins, need, scan_lds, sh);
    prefix |= q.bin << shift;
    mask |= ((uint32_t)nbins - 1u) << shift;
    need = q.need;
    hb = shift;
  }
  return prefix;
}

// LDS of a workgroup.
struct SelectLds {
  alignas(16) int hist[kTopBins];
  uint32_t buf[kColumn * kThreads];
  int scan[2 * kWaves + 1];
  uint32_t red[2][4 * kWaves];    // of the sample's reduction and of the band's: no barrier need lie between them
  int wgt[kWaves], weq[kWaves];   // per wave: keys > T, keys == T it counted before the workgroup's share
  int ties[kWaves];               // per wave, for kFlags: keys == T in all (-1: not counted)
  uint32_t cnt[2][kWaves];        // per wave: keys > T (low half), == T (high half) of its block, two rounds
  Pick pick[2];
  int pos;
};

// What is done with a candidate once it is ranked.
enum Sink {
  kLists,   // its position goes to the head's kept or evicted list
  kFlags,   // kept: its bit in the flag words of the head's cache is set
  kShared   // as kLists, into the lists of every head of the cache
};

struct SelectArgs {
  const float* score;
  int32_t* kept;
  int32_t* evicted;
  uint64_t* flag;      // kFlags: [caches, ceil(n_cand / 64)]
  int copies;          // kFlags: heads per cache; kShared: lists per selected head
  int n, n_cand, m, mr, ms;
  int split;
};

template <Sink SINK>
struct Output {
  int32_t* kh;
  int32_t* eh;
  uint64_t* flag;
  int ms, m, ne, copies;
  __device__ __forceinline__ Output(const SelectArgs& a, int64_t head)
      : ms(a.ms), m(a.m), ne(a.n - a.m), copies(SINK == kShared ? a.copies : 1) {
    const int64_t list = head * copies;
    kh = a.kept + (SINK == kFlags ? 0 : (size_t)list * m);
    eh = a.evicted + (SINK == kFlags ? 0 : (size_t)list * ne);
    flag = SINK == kFlags ? a.flag + (size_t)(head / a.copies) * ((a.n_cand + 63) / 64) : nullptr;
  }
};

// The wave copies cnt entries from LDS to a global list of any alignment:
// 16-byte stores, and single entries before the first and after the last
// 16-byte boundary.
__device__ __forceinline__ void copy_list(const int* from, int32_t* to, int cnt, int lane) {
  const int head = min((int)((16u - ((uint32_t)(uintptr_t)to & 15u)) & 15u) / 4, cnt);
  const int full = (cnt - head) / 4, tail = cnt - head - 4 * full;
  for (int c = lane; c < full; c += 64) {
    const int* f = from + head + 4 * c;
    *reinterpret_cast<int4*>(to + head + 4 * c) = make_int4(f[0], f[1], f[2], f[3]);
  }
  const int i = lane < 4 ? lane : head + 4 * full + lane - 4;
  if (lane < 4 ? lane < head : lane < 4 + tail) to[i] = from[i];
}

// ---- column path.  Its wave-wide sums and scans run on DPP, not on LDS
// permutes, and a block-wide step costs two barriers.

// x of the lane N places down (row shift within 16 lanes), `none` where there is none.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp(int none, int x) {
  return __builtin_amdgcn_update_dpp(none, x, CTRL, ROWS, 0xf, false);
}

// op over the lanes 0 .. lane of the wave (`none` is op's identity).
template <class Op>
__device__ __forceinline__ int wave_scan(int x, int none, Op op) {
  x = op(x, dpp<0x111, 0xf>(none, x));   // row_shr 1, 2, 4, 8
  x = op(x, dpp<0x112, 0xf>(none, x));
  x = op(x, dpp<0x114, 0xf>(none, x));
  x = op(x, dpp<0x118, 0xf>(none, x));
  x = op(x, dpp<0x142, 0xa>(none, x));   // lane 15 of rows 0 and 2 to rows 1 and 3
  x = op(x, dpp<0x143, 0xc>(none, x));   // lane 31 to rows 2 and 3
  return x;
}

struct OpAdd {
  __device__ __forceinline__ int operator()(int x, int y) const { return x + y; }
};
struct OpMin {
  __device__ __forceinline__ int operator()(int x, int y) const { return (int)min((uint32_t)x, (uint32_t)y); }
};
struct OpMax {
  __device__ __forceinline__ int operator()(int x, int y) const { return (int)max((uint32_t)x, (uint32_t)y); }
};

template <class Op>
__device__ __forceinline__ int wave_reduce(int x, int none, Op op) {
  return __builtin_amdgcn_readlane(wave_scan(x, none, op), 63);
}

// Minimum of lo, maximum of hi and sum of c over the workgroup (one barrier;
// `red` may be reused after the next).
__device__ __forceinline__ void block_range(uint32_t& lo, uint32_t& hi, int& c, uint32_t* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l = wave_reduce((int)lo, -1, OpMin()), h = wave_reduce((int)hi, 0, OpMax()), s = wave_reduce(c, 0, OpAdd());
  if (lane == 0) {
    red[wave] = (uint32_t)l;
    red[kWaves + wave] = (uint32_t)h;
    red[2 * kWaves + wave] = (uint32_t)s;
  }
  __syncthreads();
  const int i = lane & (kWaves - 1);
  lo = (uint32_t)wave_reduce((int)red[i], -1, OpMin());
  hi = (uint32_t)wave_reduce((int)red[kWaves + i], 0, OpMax());
  c = wave_reduce(lane < kWaves ? (int)red[2 * kWaves + i] : 0, 0, OpAdd());
}

// The bins holding the need[i]-th largest of the keys counted in hist (kTopBins bins).
template <int N>
__device__ __forceinline__ void find_bins(const int* hist, const int (&need)[N], SelectLds& l, Pick (&out)[N]) {
  static_assert(kTopBins == 4 * kThreads, "four bins per thread");
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int low = kTopBins - 4 - 4 * tid;   // thread t walks bins low + 3 down to low
  const int4 h = *reinterpret_cast<const int4*>(hist + low);
  const int c = h.x + h.y + h.z + h.w;
  const int incl = wave_scan(c, 0, OpAdd());
  if (lane == 63) l.scan[wave] = incl;
  __syncthreads();
  const int before = wave_reduce(lane < wave ? l.scan[lane & (kWaves - 1)] : 0, 0, OpAdd());
  const int excl = before + incl - c;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (excl < need[i] && excl + c >= need[i]) {
      int q = need[i] - excl, k = 3, n = h.w;
      if (q > n) { q -= n; k = 2; n = h.z; }
      if (k == 2 && q > n) { q -= n; k = 1; n = h.y; }
      if (k == 1 && q > n) { q -= n; k = 0; n = h.x; }
      l.pick[i].bin = (uint32_t)(low + k);
      l.pick[i].need = q;
      l.pick[i].count = n;
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < N; ++i) out[i] = l.pick[i];
}

constexpr int kLoads = 16;               // steps of 64 scores in flight ahead of use
constexpr int kSpan = kWaves * 64;       // scores a step of every wave covers

// kLoads steps from `at`, `stride` scores apart; past `end` the last score again.
template <int STRIDE>
__device__ __forceinline__ void load_steps(const float* s, int at, int end, int lane, float (&v)[kLoads]) {
  if (at + (kLoads - 1) * STRIDE + 64 <= end) {   // wave-uniform
    const float* p = s + at;
#pragma unroll
    for (int r = 0; r < kLoads; ++r) v[r] = p[r * STRIDE + lane];
  } else {
#pragma unroll
    for (int r = 0; r < kLoads; ++r) v[r] = s[min(at + r * STRIDE + lane, end - 1)];
  }
}

// f(r, at, inside) for the first `steps` steps of a group, as far as they
// begin below `end`; `inside`, whether the lane's score is, is a constant true
// on whole groups.
template <int STRIDE, class F>
__device__ __forceinline__ void each_step(int at, int steps, int end, int lane, F&& f) {
  if (at + (steps - 1) * STRIDE + 64 <= end) {   // wave-uniform
#pragma unroll
    for (int r = 0; r < kLoads; ++r)
      if (r < steps) f(r, at + r * STRIDE, true);
  } else {
#pragma unroll
    for (int r = 0; r < kLoads; ++r)
      if (at + r * STRIDE < end) f(r, at + r * STRIDE, at + r * STRIDE + lane < end);
  }
}

// f(j, order key of the thread's j-th staged score), four LDS reads at a time.
template <class F>
__device__ __forceinline__ void each_staged(const float* column, int cnt, F&& f) {
  for (int j = 0; j < cnt; j += 4) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = column[(j + u) * kThreads];   // cnt <= kColumnFull, so j + u < kColumn
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (j + u < cnt) f(j + u, order_key(v[u]));
  }
}

// ---- the band [lo, hi) of order keys around T's expected place, from kSample
// evenly spaced scores: a histogram of those above -inf over their own key
// range (-inf ranks below them all and would stretch the range over the whole
// key space).  Returns how many those are: with none, there is no band.
// between() runs behind the sample's loads.  Leaves the bins cleared.
struct Band {
  uint32_t lo;
  uint64_t hi;   // 2^32: no key above
  int holds;     // about how many candidates it holds, by the sample
};

template <class Between>
__device__ __forceinline__ int sample_band(const float* s, int n_cand, int ms, SelectLds& l, Band& band,
                                           Between&& between) {
  const int tid = threadIdx.x;
  *reinterpret_cast<int4*>(l.hist + 4 * tid) = make_int4(0, 0, 0, 0);
  uint32_t key[kSample / kThreads], smin = 0xffffffffu, smax = 0u;
  int fin = 0;
#pragma unroll
  for (int e = 0; e < kSample / kThreads; ++e)
    key[e] = order_key(s[(int)(((int64_t)(e * kThreads + tid) * n_cand) / kSample)]);
  between();
#pragma unroll
  for (int e = 0; e < kSample / kThreads; ++e)
    if (key[e] > kNegInfKey) {
      smin = min(smin, key[e]);
      smax = max(smax, key[e]);
      ++fin;
    }
  block_range(smin, smax, fin, l.red[0]);   // its barrier also publishes the cleared bins
  if (fin == 0) return 0;
  const int sh = top_shift(smin, smax);
#pragma unroll
  for (int e = 0; e < kSample / kThreads; ++e)
    if (key[e] > kNegInfKey) atomicAdd(&l.hist[(key[e] - smin) >> sh], 1);
  __syncthreads();
  // T's expected rank in the sample, 1-based from the top
  const int rr = (int)(((int64_t)ms * kSample + n_cand - 1) / n_cand);
  const int ranks[2] = {max(1, min(fin, rr - kBandRanks)), min(fin, rr + kBandRanks)};
  Pick pk[2];
  find_bins(l.hist, ranks, l, pk);
  *reinterpret_cast<int4*>(l.hist + 4 * tid) = make_int4(0, 0, 0, 0);
  band.lo = smin + (pk[1].bin << sh);
  band.hi = (uint64_t)smin + ((uint64_t)(pk[0].bin + 1u) << sh);
  const int in = (ranks[1] - pk[1].need + pk[1].count) - (ranks[0] - pk[0].need);
  band.holds = (int)((int64_t)in * n_cand / kSample);
  return fin;
}

// Whether T was found, and if not whether the band may still hold it (a column
// was full or a score was NaN).
enum Found { kFound, kInBand, kNotInBand };

// ---- column path: T and need of a head of at most kColumnsMax candidates, and
// per wave the counts of the scores before `from` (a multiple of kSpan) in wgt
// and weq, with TIES the number of all scores equal to T in ties.  `all`: every score fits the columns, and is staged; else those of
// the band.  Every workgroup of a head comes to the same decision.  `cur` holds
// the wave's first group.
template <bool TIES>
__device__ __forceinline__ Found column_threshold(const float* s, int n_cand, int ms, bool all, const Band& band,
                                                  int from, SelectLds& l, float (&cur)[kLoads], float& T, int& need) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int first = wave * 64;   // step i of the wave: 64 candidates from first + i * kSpan
  uint32_t smin = 0xffffffffu, smax = 0u;   // range of the staged keys
  float lo = kNegInf, hi = __uint_as_float(0x7fc00000u);
  if (!all) {
    smin = band.lo;
    smax = (uint32_t)min<uint64_t>(band.hi - 1u, 0xffffffffull);
    lo = key_score(smin);
    if (band.hi <= 0xffffffffull) hi = key_score((uint32_t)band.hi);
  }
  // ---- one pass: count the scores above the band, stage those inside it
  float* column = reinterpret_cast<float*>(l.buf) + tid;
  int up = 0, cnt = 0;
  int up0 = 0, cnt0 = 0;   // of the scores before `from`
  uint64_t bad = 0;        // lanes with a NaN or a full column
  const int cut = from > 0 ? from + first : -1;   // the wave's first step past them (none: there are no such scores)
  for (int at = first; at < n_cand; at += kLoads * kSpan) {
    float nxt[kLoads];
    if (at + kLoads * kSpan < n_cand) load_steps<kSpan>(s, at + kLoads * kSpan, n_cand, lane, nxt);
    auto stage = [&](auto cuts, int r, int pos, bool inside) {
      if constexpr (decltype(cuts)::value) {
        up0 = pos <= cut ? up : up0;
        cnt0 = pos <= cut ? cnt : cnt0;
      }
      const float v = cur[r];
      const bool above = inside && v >= hi, in = inside && v >= lo && !(v >= hi);
      bad |= __ballot(inside && v != v);
      column[cnt * kThreads] = v;
      up += above ? 1 : 0;
      cnt += in ? 1 : 0;
      if (r % 8 == 7) {
        bad |= __ballot(cnt > kColumnFull);
        cnt = min(cnt, kColumnFull);
      }
    };
    // Only the group that holds the cut looks for it: in every step, it broke
    // up the schedule of the steps (102384 candidates: 29.2 us, 27.5 so, 25.7
    // without a cut).
    if (at <= cut && cut < at + kLoads * kSpan)   // wave-uniform
      each_step<kSpan>(at, kLoads, n_cand, lane,
                       [&](int r, int pos, bool inside) { stage(std::true_type{}, r, pos, inside); });
    else
      each_step<kSpan>(at, kLoads, n_cand, lane,
                       [&](int r, int pos, bool inside) { stage(std::false_type{}, r, pos, inside); });
    bad |= __ballot(cnt > kColumnFull);
    cnt = min(cnt, kColumnFull);
    if (bad) break;
#pragma unroll
    for (int r = 0; r < kLoads; ++r) cur[r] = nxt[r];
  }
  if (cut >= n_cand) {   // all of the wave's scores lie before the share
    up0 = up;
    cnt0 = cnt;
  }
  // ---- what was staged: how many above -inf and, if every score was, their key range
  int fin = cnt;
  if (all) {
    fin = 0;
    each_staged(column, cnt, [&](int, uint32_t k) {
      if (k > kNegInfKey) {
        smin = min(smin, k);
        smax = max(smax, k);
        ++fin;
      }
    });
  }
  const int wave_up = wave_reduce(up, 0, OpAdd());
  if (lane == 0) {
    l.wgt[wave] = wave_up;
    l.red[1][3 * kWaves + wave] = bad ? 1u : 0u;
  }
  block_range(smin, smax, fin, l.red[1]);   // its barrier also publishes wgt, red and the bins
  const int above = wave_reduce(lane < kWaves ? l.wgt[lane] : 0, 0, OpAdd());
  const int any_bad = wave_reduce((int)l.red[1][3 * kWaves + (lane & (kWaves - 1))], 0, OpMax());
  if (any_bad) return kInBand;
  if (above >= ms || (!all && above + fin < ms)) return kNotInBand;
  need = ms - above;
  uint32_t tk = kNegInfKey;
  if (fin < need) {   // staged in full, and too few above -inf: -inf itself
    need -= fin;
    __syncthreads();   // the counts are read before they are written again
  } else {
    int sh = top_shift(smin, smax);
    each_staged(column, cnt, [&](int, uint32_t k) {
      if (k > kNegInfKey) atomicAdd(&l.hist[(k - smin) >> sh], 1);
    });
    if (tid == 0) l.pos = 0;
    __syncthreads();
    const int needs[1] = {need};
    Pick pk[1];
    find_bins(l.hist, needs, l, pk);
    uint32_t prefix = pk[0].bin << sh, mask = sh >= 32 ? 0u : ~0u << sh;
    need = pk[0].need;
    if (sh > 0 && pk[0].count <= 64) {
      // the few keys of the bin are ranked by every wave
      uint32_t* list = reinterpret_cast<uint32_t*>(l.hist);
      each_staged(column, cnt, [&](int, uint32_t k) {
        if (k > kNegInfKey && ((k - smin) & mask) == prefix) list[atomicAdd(&l.pos, 1)] = k - smin;
      });
      __syncthreads();
      const uint32_t mine = lane < pk[0].count ? list[lane] : 0u;
      int gt = 0, eq = 0;
      for (int j = 0; j < pk[0].count; ++j) {
        const uint32_t d = (uint32_t)__builtin_amdgcn_readlane((int)mine, j);
        gt += d > mine ? 1 : 0;
        eq += d == mine ? 1 : 0;
      }
      const uint64_t hit = __ballot(lane < pk[0].count && gt < need && gt + eq >= need);
      const int src = hit ? __builtin_ctzll(hit) : 0;
      prefix = (uint32_t)__builtin_amdgcn_readlane((int)mine, src);
      need -= __builtin_amdgcn_readlane(gt, src);
    } else {
      while (sh > 0) {
        const int shift = sh > kLowBits ? sh - kLowBits : 0;
        const int nbins = 1 << (sh - shift);
        for (int b = tid; b < nbins; b += kThreads) l.hist[b] = 0;
        __syncthreads();
        each_staged(column, cnt, [&](int, uint32_t k) {
          const uint32_t d = k - smin;
          if (k > kNegInfKey && (d & mask) == prefix) atomicAdd(&l.hist[(d >> shift) & (nbins - 1)], 1);
        });
        __syncthreads();
        const Pick q = find_bin(l.hist, nbins, need, l.scan, &l.pick[0]);
        prefix |= q.bin << shift;
        mask |= ((uint32_t)nbins - 1u) << shift;
        need = q.need;
        sh = shift;
      }
    }
    tk = smin + prefix;
  }
  T = key_score(tk);
  // ---- the counts before the workgroup's share, and the ties
  int gt = 0, eq = 0, ties = 0;
  if (TIES || from > 0) {
    each_staged(column, TIES ? cnt : cnt0, [&](int j, uint32_t k) {
      if constexpr (TIES) {
        ties += k == tk ? 1 : 0;
        eq += k == tk && j < cnt0 ? 1 : 0;
      } else {
        gt += k > tk ? 1 : 0;
        eq += k == tk ? 1 : 0;
      }
    });
    if constexpr (TIES) ties = wave_reduce(ties, 0, OpAdd());
    else gt = wave_reduce(gt + up0, 0, OpAdd());
    eq = wave_reduce(eq, 0, OpAdd());
  }
  if (lane == 0) {
    l.wgt[wave] = gt;
    l.weq[wave] = eq;
    if constexpr (TIES) l.ties[wave] = ties;
  }
  return kFound;
}

// ---- whole-head path: the key of T (and `need`, the rank of T among the keys
// equal to it) from order keys alone, which rank NaN too.  Also leaves the
// per-wave counts of the keys before `from` in wgt and weq.
__device__ __forceinline__ uint32_t whole_threshold(const float* s, int n_cand, int ms, bool use_band, const Band& band,
                                                    int from, SelectLds& l, int& need) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = (1ull << lane) - 1ull;

  int* hist = l.hist;
  uint32_t* cand = l.buf;   // staged key offsets
  int *scan_lds = l.scan, *wgt = l.wgt, *weq = l.weq;
  uint32_t* red = l.red[0];
  Pick& sh_pick = l.pick[0];
  int& sh_pos = l.pos;

  __syncthreads();   // the LDS may hold another path's values until here
  uint32_t T = 0u;
  bool found = false;
  if (use_band) {
    const uint32_t lo = band.lo;
    const uint64_t hi = band.hi;
    // ---- one pass: count the keys above the band, stage those inside it
    if (tid == 0) sh_pos = 0;
    __syncthreads();
    // wave w walks candidates [w * seg, (w + 1) * seg)
    const int seg = (n_cand + kWaves * kIter - 1) / (kWaves * kIter) * kIter;
    const int wb = min(wave * seg, n_cand), we = min(wb + seg, n_cand);
    int up_count = 0;
    walk_segment(s, wb, we, [&](int t, const float (&v)[4]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int pos = wb + t * kIter + e * 64 + lane;
        const uint32_t key = order_key(v[e]);
        const bool ok = pos < we;
        const bool up = ok && (uint64_t)key >= hi;
        const bool in = ok && !up && key >= lo;
        up_count += up ? 1 : 0;
        const uint64_t bal = __ballot(in);
        if (bal) {                              // wave-uniform
          int base = 0;
          if (lane == 0) base = atomicAdd(&sh_pos, __popcll(bal));
          base = __shfl(base, 0, 64);
          const int at = base + __popcll(bal & below);
          if (in && at < kCandCap) cand[at] = key - lo;
        }
      }
    });
    for (int o = 32; o >= 1; o >>= 1) up_count += __shfl_xor(up_count, o, 64);
    if (lane == 0) wgt[wave] = up_count;
    __syncthreads();
    int above = 0;
    for (int w = 0; w < kWaves; ++w) above += wgt[w];
    const int banded = sh_pos;
    __syncthreads();
    if (above < ms && above + banded >= ms && banded <= kCandCap) {   // T is the (ms - above)-th largest staged key
      need = ms - above;
      T = lo + resolve_staged(cand, banded, (uint32_t)min<uint64_t>(hi - lo - 1u, 0xffffffffull), need, hist, scan_lds,
                              &sh_pick);
      found = true;
    }
  }
  if (!found) {
    // ---- no band, or it missed T or overflowed LDS: radix select on d = key - (smallest key)
    uint32_t kmin, kmax, prefix, mask;
    int kabove;
    need = ms;
    key_range(s, n_cand, red, kmin, kmax, kabove);
    // With at least ms keys above -inf the threshold is one of them: those
    // keys alone are binned (-inf marks what must not be chosen, e.g. the
    // non-members of the GQA union, and would stretch the range over the
    // whole key space).  Otherwise every key and the whole range are used.
    uint32_t kfloor = kNegInfKey + 1u;
    if (kabove < ms) {
      kfloor = 0u;
      kmin = 0u;
      kmax = 0xffffffffu;
    }
    int hi_bit = top_shift(kmin, kmax);
    histogram<false>(s, nullptr, n_cand, kfloor, kmin, hi_bit, kTopBins, 0u, 0u, hist);
    Pick pk = find_bin(hist, kTopBins, need, scan_lds, &sh_pick);
    prefix = pk.bin << hi_bit;
    mask = ~0u << hi_bit;
    need = pk.need;
    const bool staged = pk.count <= kCandCap;
    if (staged && hi_bit > 0) {
      // copy the bin's offsets into LDS (order is irrelevant to the threshold)
      if (tid == 0) sh_pos = 0;
      __syncthreads();
      for (int j0 = tid; j0 < n_cand; j0 += kThreads * kHistBatch) {
        float v[kHistBatch];
#pragma unroll
        for (int u = 0; u < kHistBatch; ++u) v[u] = s[min(j0 + u * kThreads, n_cand - 1)];
#pragma unroll
        for (int u = 0; u < kHistBatch; ++u) {
          const uint32_t key = order_key(v[u]), d = key - kmin;
          const bool hit = j0 + u * kThreads < n_cand && key >= kfloor && (d & mask) == prefix;
          const uint64_t bal = __ballot(hit);
          if (bal) {                              // wave-uniform
            int base = 0;
            if (lane == 0) base = atomicAdd(&sh_pos, __popcll(bal));
            base = __shfl(base, 0, 64);
            const int at = base + __popcll(bal & below);
            if (hit && at < kCandCap) cand[at] = d;
          }
        }
      }
      __syncthreads();
    }
    // the hi_bit low bits of d, at most kLowBits per pass
    while (hi_bit > 0) {
      const int shift = hi_bit > kLowBits ? hi_bit - kLowBits : 0;
      const int nbins = 1 << (hi_bit - shift);
      if (staged) histogram<true>(nullptr, cand, pk.count, 0u, 0u, shift, nbins, mask, prefix, hist);
      else histogram<false>(s, nullptr, n_cand, kfloor, kmin, shift, nbins, mask, prefix, hist);
      const Pick q = find_bin(hist, nbins, need, scan_lds, &sh_pick);
      prefix |= q.bin << shift;
      mask |= ((uint32_t)nbins - 1u) << shift;
      need = q.need;
      hi_bit = shift;
    }
    T = prefix + kmin;
  }
  // ---- the keys before the workgroup's share
  int gt = 0, eq = 0;
  for (int j0 = tid; j0 < from; j0 += kThreads * kHistBatch) {
    float v[kHistBatch];
#pragma unroll
    for (int u = 0; u < kHistBatch; ++u) v[u] = s[min(j0 + u * kThreads, from - 1)];
#pragma unroll
    for (int u = 0; u < kHistBatch; ++u) {
      const uint32_t key = order_key(v[u]);
      const bool ok = j0 + u * kThreads < from;
      gt += (ok && key > T) ? 1 : 0;
      eq += (ok && key == T) ? 1 : 0;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    gt += __shfl_xor(gt, o, 64);
    eq += __shfl_xor(eq, o, 64);
  }
  if (lane == 0) {
    wgt[wave] = gt;
    weq[wave] = eq;
    l.ties[wave] = -1;
  }
  return T;
}

// A workgroup's share of the candidates: [from, to), in rounds of one block of
// `block` consecutive candidates (at most kLoads steps) per wave.
struct Share {
  int from, to, rounds, block;
};

__device__ __forceinline__ Share share_of(int n_cand, int split, int part) {
  const int parts = split * kWaves;
  const int len = ((n_cand + parts - 1) / parts + 63) / 64 * 64;   // candidates per wave
  Share h;
  h.from = min(part * kWaves * len, n_cand);
  h.to = min(h.from + kWaves * len, n_cand);
  h.rounds = (len + kLoads * 64 - 1) / (kLoads * 64);
  h.block = ((len + h.rounds - 1) / h.rounds + 63) / 64 * 64;
  return h;
}

// Ranks the share and writes it out.  A candidate's kept index is (scores
// above T before it) + min(scores equal to T before it, need); its evicted
// index is its position minus that.  A round's blocks are counted from the
// registers that hold them, the waves' counts meet in LDS, and the blocks are
// ranked from the same registers.  above(v), equal(v): whether a score ranks
// above T or equal to it.  `own` holds the first block.
template <Sink SINK, class Above, class Equal>
__device__ __forceinline__ void compact(const float* s, int n_cand, const Share& h, int need, const Output<SINK>& out,
                                        SelectLds& l, float (&own)[kLoads], Above&& above, Equal&& equal) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // The lists of a block are put together in LDS (the staged scores are no
  // longer needed) and copied out by 16-byte stores: two stores of single
  // entries per step took 20 us of a 32768-candidate head, these take 3 us.
  int* klist = reinterpret_cast<int*>(l.buf) + wave * (2 * kLoads * 64);
  int* elist = klist + kLoads * 64;
  const int steps = h.block / 64;
  if constexpr (SINK == kFlags) {
    // The usual case, every score equal to T is kept: a score's bit depends on
    // no other score.
    __syncthreads();
    if (wave_reduce(lane < kWaves ? l.ties[lane] : 0, 0, OpAdd()) == need) {
      for (int t = 0; t < h.rounds; ++t) {
        const int at = h.from + (t * kWaves + wave) * h.block, end = min(at + h.block, h.to);
        const int nat = at + kWaves * h.block;
        float nxt[kLoads];
        if (t + 1 < h.rounds && nat < h.to) load_steps<64>(s, nat, n_cand, lane, nxt);
        each_step<64>(at, steps, end, lane, [&](int r, int pos0, bool inside) {
          const uint64_t keep = __ballot(inside && (above(own[r]) || equal(own[r])));
          if (keep && lane == 0) atomicOr(reinterpret_cast<unsigned long long*>(out.flag) + pos0 / 64, keep);
        });
#pragma unroll
        for (int r = 0; r < kLoads; ++r) own[r] = nxt[r];
      }
      return;
    }
  }
  int gt0 = 0, eq0 = 0;   // scores above and equal to T before the round
  for (int t = 0; t < h.rounds; ++t) {
    const int at = h.from + (t * kWaves + wave) * h.block, end = min(at + h.block, h.to);
    const int nat = at + kWaves * h.block;
    float nxt[kLoads];
    if (t + 1 < h.rounds && nat < h.to) load_steps<64>(s, nat, n_cand, lane, nxt);
    int gt = 0, eq = 0;   // wave-uniform
    each_step<64>(at, steps, end, lane, [&](int r, int, bool inside) {
      if constexpr (SINK != kFlags) gt += __popcll(__ballot(inside && above(own[r])));   // bits have no place in a list
      eq += __popcll(__ballot(inside && equal(own[r])));
    });
    if (lane == 0) l.cnt[t & 1][wave] = (uint32_t)gt | (uint32_t)eq << 16;
    __syncthreads();   // before the first round also: the staged scores are no longer read, wgt and weq are there
    if (t == 0 && h.from > 0) {
      gt0 = wave_reduce(lane < kWaves ? l.wgt[lane] : 0, 0, OpAdd());
      eq0 = wave_reduce(lane < kWaves ? l.weq[lane] : 0, 0, OpAdd());
    }
    const int c = (int)l.cnt[t & 1][lane & (kWaves - 1)];
    const uint32_t before = (uint32_t)wave_reduce(lane < wave ? c : 0, 0, OpAdd());
    int eqb = eq0 + (int)(before >> 16);
    int kb0 = gt0 + (int)(before & 0xffffu) + min(eqb, need);   // kept before the block, then before the step
    const int kg = kb0, eg = at - kb0;
    each_step<64>(at, steps, end, lane, [&](int r, int pos0, bool inside) {
      bool kept = inside && above(own[r]);
      const uint64_t ties = __ballot(inside && equal(own[r]));
      if (ties) {   // wave-uniform: the first need - eqb of them are kept
        kept |= ((ties >> lane) & 1ull) && eqb + __popcll(ties & ((1ull << lane) - 1ull)) < need;
        eqb += __popcll(ties);
      }
      const uint64_t keep = __ballot(kept);
      if constexpr (SINK == kFlags) {
        if (keep && lane == 0) atomicOr(reinterpret_cast<unsigned long long*>(out.flag) + pos0 / 64, keep);
      } else {
        const int kb = __builtin_amdgcn_mbcnt_hi((uint32_t)(keep >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)keep, kb0));
        const int pos = pos0 + lane;
        if (inside) (kept ? klist : elist)[kept ? kb - kg : pos - kb - eg] = pos;
      }
      kb0 += __popcll(keep);
    });
    if constexpr (SINK != kFlags) {
      if (at < end) {
        const int nk = min(kb0, out.ms) - kg, ne = min(end - kb0, out.ne) - eg;
        for (int c2 = 0; c2 < out.copies; ++c2) {
          if (nk > 0) copy_list(klist, out.kh + (size_t)c2 * out.m + kg, nk, lane);
          if (ne > 0) copy_list(elist, out.eh + (size_t)c2 * out.ne + eg, ne, lane);
        }
      }
    }
    if (t + 1 < h.rounds) {
      const uint32_t round = (uint32_t)wave_reduce(lane < kWaves ? c : 0, 0, OpAdd());
      gt0 += (int)(round & 0xffffu);
      eq0 += (int)(round >> 16);
#pragma unroll
      for (int r = 0; r < kLoads; ++r) own[r] = nxt[r];
    }
  }
}

template <Sink SINK>
__global__ __launch_bounds__(kThreads) void select_kernel(SelectArgs a) {
  __shared__ SelectLds l;
  // heads along x: consecutive workgroups go to the XCDs in turn, so a head's
  // workgroups share an L2 when the head count is a multiple of eight
  const int64_t head = blockIdx.x;
  const int part = blockIdx.y;
  const int n_cand = a.n_cand, ms = a.ms;
  const float* s = a.score + (size_t)head * n_cand;
  const Output<SINK> out(a, head);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (SINK != kFlags && part == 0)
    for (int c = 0; c < (SINK == kShared ? a.copies : 1); ++c)
      for (int r = tid; r < a.mr; r += kThreads) out.kh[(size_t)c * a.m + ms + r] = n_cand + r;
  if (n_cand == 0) return;
  const Share h = share_of(n_cand, a.split, part);
  if (h.from >= h.to) return;   // the whole workgroup

  // the first block loads while T is found
  const int at = h.from + wave * h.block;
  float own[kLoads];
  if (at < h.to) load_steps<64>(s, at, n_cand, lane, own);

  float T = __uint_as_float(0x7fc00000u);   // ms == 0: nothing is greater than or equal to it
  int need = 0;
  Band band{0u, 1ull << 32, n_cand};   // of a short head: every key
  Found found = kFound;
  if (ms == 0) {
    if (tid < kWaves) l.wgt[tid] = l.weq[tid] = l.ties[tid] = 0;   // compact reads them after a barrier
  } else {
    const bool all = n_cand <= kAllSteps * kSpan;
    float cur[kLoads];
    auto load_first = [&] {
      if (wave * 64 < n_cand) load_steps<kSpan>(s, wave * 64, n_cand, lane, cur);
    };
    if (all) {
      *reinterpret_cast<int4*>(l.hist + 4 * tid) = make_int4(0, 0, 0, 0);
      load_first();
    } else if (sample_band(s, n_cand, ms, l, band, load_first) == 0) {
      found = kNotInBand;
    } else if (band.holds > kCandCap) {
      found = kNotInBand;   // scores equal to T in masses
    } else if (n_cand > kColumnsMax || band.holds > kColumnFull * kThreads) {
      found = kInBand;
    }
    if (found == kFound) found = column_threshold<SINK == kFlags>(s, n_cand, ms, all, band, h.from, l, cur, T, need);
  }
  if (found == kFound) {
    compact<SINK>(s, n_cand, h, need, out, l, own, [=](float v) { return v > T; }, [=](float v) { return v == T; });
  } else {
    const uint32_t tk = whole_threshold(s, n_cand, ms, found == kInBand, band, h.from, l, need);
    if (at < h.to) load_steps<64>(s, at, n_cand, lane, own);
    compact<SINK>(s, n_cand, h, need, out, l, own, [=](float v) { return order_key(v) > tk; },
                  [=](float v) { return order_key(v) == tk; });
  }
}

template <Sink SINK>
hipError_t launch(const Shape& s, const float* score, int32_t* kept, int32_t* evicted, uint64_t* flag, int copies,
                  hipStream_t st) {
  SelectArgs a{};
  a.score = score;
  a.kept = kept;
  a.evicted = evicted;
  a.flag = flag;
  a.copies = copies;
  a.n = s.n;
  a.n_cand = s.n_cand;
  a.m = s.m;
  a.mr = s.mr;
  a.ms = s.ms;
  // Workgroups per head: as many as fill the 256 CUs once (a workgroup's LDS
  // takes a CU), while a wave still compacts 64 candidates or more.
  a.split = 1;
  while (a.split < kMaxSplit && 2 * a.split * s.heads <= 256 && s.n_cand >= 2 * a.split * kWaves * 64) a.split *= 2;
  hipLaunchKernelGGL(select_kernel<SINK>, dim3((unsigned)s.heads, a.split), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select(const Shape& s, const float* score, int32_t* kept, int32_t* evicted, hipStream_t st) {
  return launch<kLists>(s, score, kept, evicted, nullptr, 1, st);
}

hipError_t launch_select_flags(const Shape& s, const float* score, uint64_t* flag, hipStream_t st) {
  return launch<kFlags>(s, score, nullptr, nullptr, flag, s.hkv, st);
}

hipError_t launch_select_shared(const Shape& s, const float* score, int32_t* kept, int32_t* evicted, int copies,
                                hipStream_t st) {
  return launch<kShared>(s, score, kept, evicted, nullptr, copies, st);
}

}  // namespace selkv
