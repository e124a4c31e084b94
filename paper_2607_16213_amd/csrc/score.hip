// selkv_score: contribution scores of Sec. 3.2 (Eq. 1) from the
// observation-window attention of Sec. 3.1, recomputed on the fly.
//
// For one KV head the window rows are the G*W query rows of its G query
// heads (row r = h*W + i is position n-W+i, causal).  The logits
// scale * Q K^T are produced on MFMA (16x16x32 bf16, or 16x16x4 fp32) with
// Q fragments in registers and K streamed from HBM:
//   pass 1  per (key chunk, row group): online row max / sum of exp  -> ws
//   combine per KV head: merge the chunk partials in chunk order into
//           (-M, 1/L) per row                                        -> ws
//   pass 2  per key chunk: recompute the logits, normalise
//           (2^(x - M) * 1/L), sum the G*W rows of every key column
//           (a_j, divided by G), value norms from V, write attn, vnorm
//   pool    centred K-wide moving average of c = a * ||v|| over
//           [0, n - m_r'), in fp64
// The attention matrix itself is never stored.
//
// At most 256 window rows (the shapes of the paper's workloads)
// take the shared-tile passes further down: K tiles go through a ring of LDS
// stages shared by the workgroup's waves, which split the window rows (and,
// with few rows, the keys of a tile), and pass 1 keeps a per-row exponent
// reference that only moves when a logit exceeds it by 2^16, so a logit costs
// one fma, one exp2, one add and a share of a max.  Unless the call is large,
// pass 2 merges the chunk partials itself and the combine kernel is not
// launched.  More rows take the general passes below, which read K once per
// group of 32 to 128 rows (fp32, 8192 tokens x 8 heads x 128 rows: 109 us
// there, 65 us by shared tiles; 102400 tokens 805 and 504 us).
//
// General passes, work split inside a 4-wave workgroup: RW waves share each K tile, each
// holding NRB 16-row blocks of Q (RW * NRB * 16 rows per row group); the
// 4 / RW pairs walk interleaved 16-key tiles of the chunk.  Every K load is
// issued unconditionally (rows past the chunk end re-read its last row and
// are masked) and the next tile is loaded before the current one is used.
// Tiles that every row sees in full skip all masking.
//
// Fragment layout (both MFMA operands, all dtypes): lane l handles matrix
// index l % 16 (a window row for Q, a key for K) and lane group g = l / 16
// owns the 16-byte chunks c*4 + g of that row, so one load instruction reads
// 64 contiguous bytes from each of 16 rows.  MFMA output lane l holds rows
// 4g .. 4g+3 of the 16-row block for key l % 16.
#include <algorithm>

#include "common.hpp"
#include "internal.hpp"

namespace selkv {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kThreads = 256;          // 4 waves
constexpr int kWaves = kThreads / 64;
constexpr int kMaxChunkKeys = 4096;   // LDS column accumulator bound
constexpr int kColsumStages = 2;       // K/V tiles in registers in pass 2 (loads in flight + 1)
// Pass 1 keeps each row's exponent reference fixed until a logit exceeds it
// by more than this (log2 units); sums of up to 2^kRefSlack stay exact in fp32
// range, and a logit costs one fma, one exp2, one add and one compare.
constexpr float kRefSlack = 16.f;
constexpr int kMinChunkKeys = 128;
constexpr int kTargetBlocks = 2048;
constexpr int kTiledRows = 256;        // window rows the shared-tile passes take

template <typename T, int D>
struct Row {
  static constexpr int kBytes = D * (int)sizeof(T);
  static constexpr int kNch = kBytes / 64;   // 16-byte chunks per lane per row
};

struct ScoreArgs {
  const char* K;
  const char* V;
  const char* Q;
  float* attn;
  float* vnorm;
  float2* part;
  float2* stats;
  int n, W, R, G;
  int chunk_keys, nchunks, rpad, nrg;
  int chunk_keys2;   // shared-tile pass 2
  int merged;        // shared-tile pass 2: the row statistics are in stats (else the partials are merged there)
  float c2;  // scale * log2(e): logits are kept in the log2 domain
};

__device__ __forceinline__ void lse_merge(float& m, float& s, float m2, float s2) {
  const float M = fmaxf(m, m2);
  if (M == kNegInf) {
    s = 0.f;
  } else {
    s = s * fast_exp2(m - M) + s2 * fast_exp2(m2 - M);
  }
  m = M;
}

template <typename T, int D, int NRB>
__device__ __forceinline__ void load_q(const char* Qh, int R, int row0, int col, int grp,
                                       Chunk16 (&q)[NRB][Row<T, D>::kNch]) {
  constexpr int NCH = Row<T, D>::kNch;
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb) {
    const int row = row0 + rb * 16 + col;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
      q[rb][c] = row < R ? load16(Qh + (size_t)row * Row<T, D>::kBytes + (c * 4 + grp) * 16) : zero16();
  }
}

// K (or V) fragments of the 16-key tile starting at t; keys past `last` re-read row `last`.
template <typename T, int D>
__device__ __forceinline__ void load_tile(const char* Xh, int t, int last, int col, int grp,
                                          Chunk16 (&f)[Row<T, D>::kNch]) {
  constexpr int NCH = Row<T, D>::kNch;
  const int key = min(t + col, last);
#pragma unroll
  for (int c = 0; c < NCH; ++c) f[c] = load16(Xh + (size_t)key * Row<T, D>::kBytes + (c * 4 + grp) * 16);
}

// Runs body(tile, t) over the 16-key tiles t = t0, t0 + step, ... < ke,
// with load(tile, t) issued STAGES - 1 tiles ahead of use.
template <int STAGES, typename Tile, typename Load, typename Body>
__device__ __forceinline__ void pipeline(int t0, int ke, int step, Load&& load, Body&& body) {
  static_assert(STAGES == 2 || STAGES == 3, "two or three register buffers");
  int t = t0;
  if (t >= ke) return;
  if constexpr (STAGES == 2) {
    Tile ta, tb;
    load(ta, t);
    while (true) {
      load(tb, t + step);
      body(ta, t);
      t += step;
      if (t >= ke) break;
      load(ta, t + step);
      body(tb, t);
      t += step;
      if (t >= ke) break;
    }
  } else {
    Tile ta, tb, tc;
    load(ta, t);
    load(tb, t + step);
    while (true) {
      load(tc, t + 2 * step);
      body(ta, t);
      t += step;
      if (t >= ke) break;
      load(ta, t + 2 * step);
      body(tb, t);
      t += step;
      if (t >= ke) break;
      load(tb, t + 2 * step);
      body(tc, t);
      t += step;
      if (t >= ke) break;
    }
  }
}

template <typename T, int D>
struct KTile {
  Chunk16 k[Row<T, D>::kNch];
};

// K fragments plus this wave's share of the V rows (for the norms).
template <typename T, int D, int NV>
struct KVTile {
  Chunk16 k[Row<T, D>::kNch];
  Chunk16 v[NV];
};

// Whether window row `row` (of R, window W) sees key `key` of an n-key cache.
__device__ __forceinline__ bool row_sees(int row, int key, int R, int W, int n, int ke) {
  return key < ke && row < R && key <= n - W + row % W;
}

// Pass 1: per-row (max, sum of exp2) over this block's key chunk.
template <typename T, int D, int NRB, int RW>
__global__ __launch_bounds__(kThreads) void score_rowstats_kernel(ScoreArgs a) {
  constexpr int NCH = Row<T, D>::kNch;
  constexpr int TS = 4 / RW;
  constexpr int ROWS = RW * NRB * 16;
  const int chunk = blockIdx.x;
  const int64_t head = blockIdx.y;
  const int rg = blockIdx.z;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int half = wave % RW, stream = wave / RW;
  const int n = a.n, W = a.W;
  const char* Kh = a.K + (size_t)head * n * Row<T, D>::kBytes;
  const char* Qh = a.Q + (size_t)head * a.R * Row<T, D>::kBytes;
  const int row0 = rg * ROWS + half * NRB * 16;

  Chunk16 q[NRB][NCH];
  load_q<T, D, NRB>(Qh, a.R, row0, col, grp, q);

  float m[NRB][4], s[NRB][4];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[rb][i] = kNegInf;
      s[rb][i] = 0.f;
    }

  const int kb = chunk * a.chunk_keys;
  const int ke = min(n, kb + a.chunk_keys);
  const int full_end = min(ke, n - W + 1);     // keys below this are seen by every row
  const int R = a.R;
  using Tile = KTile<T, D>;
  auto load = [&](Tile& tl, int t) { load_tile<T, D>(Kh, t, ke - 1, col, grp, tl.k); };
  pipeline<2, Tile>(kb + stream * 16, ke, TS * 16, load, [&](const Tile& tl, int t) {
    const bool fast = t + 16 <= full_end;
    f32x4 acc[NRB];
    auto logits = [&]() {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c) acc[rb] = Mma<T>::step(q[rb][c], tl.k[c], acc[rb]);
      }
    };
    logits();
    if (fast) {
      // common case: every key visible and no logit in the wave more than
      // kRefSlack above its row's reference (acc becomes the exponent)
      bool up = false;
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[rb][i] = fmaf(acc[rb][i], a.c2, -m[rb][i]);
          up |= acc[rb][i] > kRefSlack;
        }
      if (!__any(up)) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[rb][i] += fast_exp2(acc[rb][i]);
        return;
      }
      logits();   // rare: recompute the tile for the general update
    }
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool valid = fast || row_sees(row0 + rb * 16 + grp * 4 + i, t + col, R, W, n, ke);
        if (valid) {
          const float x = acc[rb][i] * a.c2;
          const float dlt = x - m[rb][i];
          const float e = fast_exp2(-fabsf(dlt));
          if (dlt > 0.f) {
            s[rb][i] = fmaf(s[rb][i], e, 1.f);
            m[rb][i] = x;
          } else {
            s[rb][i] += e;
          }
        }
      }
    }
  });

  // merge the 16 lanes (keys) that share each row
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) {
        const float m2 = xor_shfl(m[rb][i], off);
        const float s2 = xor_shfl(s[rb][i], off);
        lse_merge(m[rb][i], s[rb][i], m2, s2);
      }

  __shared__ float2 red[TS][ROWS];
  if (col == 0) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        red[stream][half * NRB * 16 + rb * 16 + grp * 4 + i] = make_float2(m[rb][i], s[rb][i]);
  }
  __syncthreads();
  for (int r = threadIdx.x; r < ROWS; r += kThreads) {
    float mm = red[0][r].x, ss = red[0][r].y;
#pragma unroll
    for (int w = 1; w < TS; ++w) lse_merge(mm, ss, red[w][r].x, red[w][r].y);
    a.part[((size_t)head * a.nchunks + chunk) * a.rpad + rg * ROWS + r] = make_float2(mm, ss);
  }
}

// Combine the chunk partials of every row, in chunk order: (max, 1/sum).
__global__ __launch_bounds__(kThreads) void score_combine_kernel(ScoreArgs a) {
  constexpr int kBatch = 8;   // partial loads in flight per thread
  const int64_t head = blockIdx.x;
  for (int row = threadIdx.x; row < a.rpad; row += blockDim.x) {
    const float2* p = a.part + (size_t)head * a.nchunks * a.rpad + row;
    float M = kNegInf, L = 0.f;
    for (int c0 = 0; c0 < a.nchunks; c0 += kBatch) {
      float2 v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) v[u] = p[(size_t)min(c0 + u, a.nchunks - 1) * a.rpad];
#pragma unroll
      for (int u = 0; u < kBatch; ++u)
        if (c0 + u < a.nchunks) lse_merge(M, L, v[u].x, v[u].y);
    }
    // pass 2 takes p = 2^(x - M) * (1/L): the exponent stays near 0 and 1/L
    // is one correctly rounded division, so no per-row rounding of log2 L
    // (about 1e-6 absolute at L ~ 1e5) enters every probability of the row.
    // Padding rows get (-inf, 0), whose p is then 0.
    const bool live = row < a.R && L > 0.f;
    a.stats[(size_t)head * a.rpad + row] = make_float2(live ? -M : kNegInf, live ? 1.f / L : 0.f);
  }
}

// Pass 2: column sums of the normalised window attention, value norms, c.
template <typename T, int D, int NRB, int RW>
__global__ __launch_bounds__(kThreads) void score_colsum_kernel(ScoreArgs a) {
  constexpr int NCH = Row<T, D>::kNch;
  constexpr int EPC = Elem<T>::kPerChunk;
  constexpr int TS = 4 / RW;
  constexpr int ROWS = RW * NRB * 16;
  const int chunk = blockIdx.x;
  const int64_t head = blockIdx.y;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int half = wave % RW, stream = wave / RW;
  const int n = a.n, W = a.W;
  const char* Kh = a.K + (size_t)head * n * Row<T, D>::kBytes;
  const char* Vh = a.V + (size_t)head * n * Row<T, D>::kBytes;
  const char* Qh = a.Q + (size_t)head * a.R * Row<T, D>::kBytes;
  const float2* st = a.stats + (size_t)head * a.rpad;
  const int kb = chunk * a.chunk_keys;
  const int ke = min(n, kb + a.chunk_keys);
  const int full_end = min(ke, n - W + 1);

  __shared__ float colacc[RW][kMaxChunkKeys];
  __shared__ float vn_l[RW][kMaxChunkKeys];   // squared-norm partials, one per row half

  for (int rg = 0; rg < a.nrg; ++rg) {
    const int row0 = rg * ROWS + half * NRB * 16;
    Chunk16 q[NRB][NCH];
    load_q<T, D, NRB>(Qh, a.R, row0, col, grp, q);
    float off[NRB][4], inv[NRB][4];   // -M and 1/L of each row
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float2 sv = st[row0 + rb * 16 + grp * 4 + i];
        off[rb][i] = sv.x;
        inv[rb][i] = sv.y;
      }
    // each row half reads its share of every V row once: chunks c with c % RW == half
    const bool norms = rg == 0;
    const int R = a.R;

    constexpr int NV = NCH / RW > 0 ? NCH / RW : 1;
    using Tile = KVTile<T, D, NV>;
    auto load = [&](Tile& tl, int t) {
      load_tile<T, D>(Kh, t, ke - 1, col, grp, tl.k);
      if (norms) {
        const int vkey = min(t + col, ke - 1);
#pragma unroll
        for (int c = 0; c < NV; ++c)
          tl.v[c] = load16(Vh + (size_t)vkey * Row<T, D>::kBytes + ((c * RW + half) * 4 + grp) * 16);
      }
    };
    pipeline<kColsumStages, Tile>(kb + stream * 16, ke, TS * 16, load, [&](const Tile& tl, int t) {
      const bool fast = t + 16 <= full_end;
      const int key = t + col;
      float cs = 0.f;
      f32x4 acc[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) {
        acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c) acc[rb] = Mma<T>::step(q[rb][c], tl.k[c], acc[rb]);
      }
      if (fast) {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) cs = fmaf(fast_exp2(fmaf(acc[rb][i], a.c2, off[rb][i])), inv[rb][i], cs);
      } else {
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float p = fast_exp2(fmaf(acc[rb][i], a.c2, off[rb][i]));
            const bool vis = row_sees(row0 + rb * 16 + grp * 4 + i, key, R, W, n, ke);
            cs = fmaf(vis ? p : 0.f, inv[rb][i], cs);
          }
      }
      cs = add_xor16(cs);
      cs = add_xor32(cs);
      const int local = key - kb;
      if (grp == 0 && key < ke) colacc[half][local] = (rg == 0 ? 0.f : colacc[half][local]) + cs;
      if (norms) {
        float ss = 0.f;
#pragma unroll
        for (int c = 0; c < NV; ++c)
#pragma unroll
          for (int e = 0; e < EPC; ++e) {
            const float x = Elem<T>::get(tl.v[c], e);
            ss = fmaf(x, x, ss);
          }
        ss = add_xor16(ss);
        ss = add_xor32(ss);
        if (grp == 0 && key < ke) vn_l[half][local] = ss;
      }
    });
  }
  __syncthreads();
  for (int k = kb + (int)threadIdx.x; k < ke; k += kThreads) {
    const int local = k - kb;
    float total = colacc[0][local];
#pragma unroll
    for (int h = 1; h < RW; ++h) total += colacc[h][local];
    const float av = total / (float)a.G;
    float ss = vn_l[0][local];
#pragma unroll
    for (int h = 1; h < RW; ++h) ss += vn_l[h][local];
    const size_t o = (size_t)head * n + k;
    a.attn[o] = av;
    a.vnorm[o] = sqrtf(ss);
  }
}

// Centred moving average of width K over the candidate range, zero outside,
// of c = a * ||v|| (Eq. 1).  The product of the two fp32 outputs is exact in
// fp64 and the K-term sum and the division are taken there too, so the score
// carries one rounding to fp32 beyond the errors of a and ||v||.  Each
// workgroup stages its kPoolOut outputs' products plus the K - 1 halo values
// in LDS (zeros outside [0, n_cand)), then each output sums its K
// neighbours from LDS in ascending position.
constexpr int kPoolOut = 1024;
constexpr int kPoolMaxK = 1025;

__global__ __launch_bounds__(kThreads) void score_pool_kernel(const float* attn, const float* vnorm, float* score,
                                                             int n, int n_cand, int K) {
  __shared__ double tile[kPoolOut + kPoolMaxK - 1];
  const int64_t head = blockIdx.y;
  const int j0 = blockIdx.x * kPoolOut;
  const int h = K / 2;
  const float* av = attn + (size_t)head * n;
  const float* vn = vnorm + (size_t)head * n;
  if (2 * h < kThreads) {
    // the usual small K: every thread's loads are issued before any is
    // stored, so their latencies overlap (kPoolOut / kThreads + 1 each)
    constexpr int kL = kPoolOut / kThreads + 1;
    float x[kL], y[kL];
#pragma unroll
    for (int u = 0; u < kL; ++u) {
      const int jj = min(max(j0 - h + (int)threadIdx.x + u * kThreads, 0), n_cand - 1);   // clamped, masked below
      x[u] = av[jj];
      y[u] = vn[jj];
    }
#pragma unroll
    for (int u = 0; u < kL; ++u) {
      const int i = threadIdx.x + u * kThreads, jj = j0 - h + i;
      if (i < kPoolOut + 2 * h) tile[i] = (jj >= 0 && jj < n_cand) ? (double)x[u] * (double)y[u] : 0.0;
    }
  } else {
    for (int i = threadIdx.x; i < kPoolOut + 2 * h; i += kThreads) {
      const int jj = j0 - h + i;
      const int jc = min(max(jj, 0), n_cand - 1);   // clamped load, masked below
      const double c = (double)av[jc] * (double)vn[jc];
      tile[i] = (jj >= 0 && jj < n_cand) ? c : 0.0;
    }
  }
  __syncthreads();
  for (int q = threadIdx.x; q < kPoolOut; q += kThreads) {
    const int j = j0 + q;
    if (j < n_cand) {
      double sum = 0.0;
      for (int t = 0; t < K; ++t) sum += tile[q + t];
      score[(size_t)head * n_cand + j] = (float)(sum / (double)K);
    }
  }
}

// ---------------------------------------------------------------------------
// Shared-tile passes (at most 256 window rows).  The workgroup streams
// its key chunk in TK-key tiles that every wave reads from LDS; each thread
// loads an equal share of a tile with fully contiguous 16-byte loads and keeps
// kDepth tiles of loads in flight (registers).  LDS rows are stored
// with their 16-byte chunks XOR-swizzled by the row index, so the 16 lanes
// that read one chunk of 16 different rows hit distinct banks.  (A ring of LDS
// stages filled by LDS-DMA loads needs no registers for them, but reads of
// some stages wait for every load in flight: pass 2 was 5% slower.)
//
// A configuration <D, NW, NRB, RW>: NW waves, of which RW share the window
// rows (NRB 16-row MFMA blocks each: RW * NRB * 16 rows) and KS = NW / RW
// share the 16-key subtiles of a tile.
// Tiles of loads in flight per thread.  Two suffice beside two or three
// workgroups per CU, and more only hold registers: with 4 / 3 / 2 tiles one
// 8192-token layer takes 30.4 / 30.0 / 28.0 us, a 102400-token layer
// 146 / 140 / 136 us and 32 of them 3.91 / 3.74 / 3.74 ms.
constexpr int kDepth = 2;
// Pass 2 keeps its per-key outputs in LDS and writes them kOutKeys at a time:
// a global store on every trip would sit among the tile loads and make every
// wait for the oldest tile also wait for it.
constexpr int kOutKeys = 1024;

template <typename T_, int D_, int NW_, int NRB_, int RW_>
struct Tiled {
  using T = T_;
  static constexpr int D = D_, NW = NW_, NRB = NRB_, RW = RW_;
  static constexpr int NT = NW * 64;                     // threads
  static constexpr int TK = 8 * NW;                      // keys per tile
  static constexpr int KS = NW / RW;                     // waves sharing a tile's keys
  static constexpr int SUB = TK / 16 / KS;               // 16-key subtiles of a wave
  static constexpr int ROWS = RW * NRB * 16;
  static constexpr int RB = D * (int)sizeof(T);          // bytes per row
  static constexpr int NCHUNK = RB / 16;                 // 16-byte chunks per row
  static constexpr int NCH = RB / 64;                    // MFMA k-steps per row
  static constexpr int TILE = TK * RB;                   // bytes per tile
  static constexpr int LPT = TILE / (NT * 16);           // 16-byte loads per thread per tile
  static_assert(LPT >= 1 && TILE % (NT * 16) == 0, "tile must split evenly over the workgroup");
  static_assert(SUB >= 1 && RW * KS == NW, "waves must split rows and keys evenly");
};

// Thread tid's j-th piece of a tile: row and chunk inside the tile.
template <class C>
__device__ __forceinline__ void piece(int j, int tid, int& row, int& ch) {
  const int off = (j * C::NT + tid) * 16;
  row = off / C::RB;
  ch = (off % C::RB) / 16;
}

template <class C>
__device__ __forceinline__ void issue_tile(const char* Xh, int t0, int ke, int tid, Chunk16 (&r)[C::LPT]) {
#pragma unroll
  for (int j = 0; j < C::LPT; ++j) {
    int row, ch;
    piece<C>(j, tid, row, ch);
    r[j] = load16(Xh + (size_t)min(t0 + row, ke - 1) * C::RB + ch * 16);
  }
}

template <class C>
__device__ __forceinline__ int swz(int row, int ch) {
  return row * C::RB + ((ch ^ (row & (C::NCHUNK - 1))) * 16);
}

template <class C>
__device__ __forceinline__ void commit_tile(char* stage, int tid, const Chunk16 (&r)[C::LPT]) {
#pragma unroll
  for (int j = 0; j < C::LPT; ++j) {
    int row, ch;
    piece<C>(j, tid, row, ch);
    store16(stage + swz<C>(row, ch), r[j]);
  }
}

// Logits of this wave's rows against the 16 keys kk*16 .. kk*16+15 of the staged tile.
template <class C>
__device__ __forceinline__ void tile_logits(const char* stage, int kk, int col, int grp,
                                            const Chunk16 (&q)[C::NRB][C::NCH], f32x4 (&acc)[C::NRB]) {
  Chunk16 bf[C::NCH];
  const int row = kk * 16 + col;
#pragma unroll
  for (int c = 0; c < C::NCH; ++c) bf[c] = *reinterpret_cast<const Chunk16*>(stage + swz<C>(row, c * 4 + grp));
#pragma unroll
  for (int rb = 0; rb < C::NRB; ++rb) {
    acc[rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C::NCH; ++c) acc[rb] = Mma<typename C::T>::step(q[rb][c], bf[c], acc[rb]);
  }
}

// Drives the tile pipeline: body(stage, tile) for tile = 0 .. ntiles-1 on
// the staged K tile, with after(tile) called once the tile's body has run
// on every wave.  WITH_V: the same rows of V travel alongside in registers
// (never staged) and vhook(tile, pieces) sees them when the K tile is stored.
// pre() runs behind the first loads (work that overlaps their latency).
// Register slots are indexed statically (the loop is unrolled by kDepth) so
// the compiler waits only for the oldest tile's loads.
template <class C, bool WITH_V, typename Pre, typename VHook, typename Body, typename After>
__device__ __forceinline__ void tiled_stream(const char* Kh, const char* Vh, int kb, int ke, int tid,
                                             char (*lds)[C::TILE], Pre&& pre, VHook&& vhook, Body&& body,
                                             After&& after) {
  constexpr int LPT = C::LPT, TK = C::TK;
  const int ntiles = (ke - kb + TK - 1) / TK;
  Chunk16 rk[kDepth][LPT];
  Chunk16 rv[WITH_V ? kDepth : 1][LPT];
#pragma unroll
  for (int p = 0; p < kDepth; ++p) {
    issue_tile<C>(Kh, kb + p * TK, ke, tid, rk[p]);
    if constexpr (WITH_V) issue_tile<C>(Vh, kb + p * TK, ke, tid, rv[p]);
  }
  pre();
  commit_tile<C>(lds[0], tid, rk[0]);
  if constexpr (WITH_V) vhook(0, rv[0]);
  issue_tile<C>(Kh, kb + kDepth * TK, ke, tid, rk[0]);
  if constexpr (WITH_V) issue_tile<C>(Vh, kb + kDepth * TK, ke, tid, rv[0]);
  __syncthreads();
  // Loads and LDS stores run unconditionally (past the chunk they re-read
  // its last key and fill stages nobody reads), so the register slots look
  // the same on every trip and the compiler waits only for the oldest slot.
  static_assert(kDepth % 2 == 0, "a pass of the loop covers a whole number of stage pairs");
  for (int i = 0; i < ntiles; i += kDepth) {
#pragma unroll
    for (int u = 0; u < kDepth; ++u) {
      const int tile = i + u;
      if (tile > 0 && tile <= ntiles) after(tile - 1);
      const int nu = (u + 1) % kDepth;     // a constant once the loop is unrolled
      // consume the slot (K to LDS, V to norms), then refill it
      commit_tile<C>(lds[(u + 1) & 1], tid, rk[nu]);
      if constexpr (WITH_V) vhook(tile + 1, rv[nu]);
      issue_tile<C>(Kh, kb + (tile + 1 + kDepth) * TK, ke, tid, rk[nu]);
      if constexpr (WITH_V) issue_tile<C>(Vh, kb + (tile + 1 + kDepth) * TK, ke, tid, rv[nu]);
      if (tile < ntiles) body(lds[u & 1], tile);
      __syncthreads();
    }
  }
  if (ntiles % kDepth == 0) after(ntiles - 1);   // the loop ran exactly the chunk's tiles
}

template <class C>
__global__ __launch_bounds__(C::NT, C::NW == 4 && sizeof(typename C::T) == 2 ? 3 : 2) void score_rowstats_tiled(ScoreArgs a) {
  constexpr int NRB = C::NRB;
  __shared__ __align__(16) char lds[2][C::TILE];
  const int chunk = blockIdx.x;
  const int64_t head = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int n = a.n, W = a.W, R = a.R;
  const char* Kh = a.K + (size_t)head * n * C::RB;
  const char* Qh = a.Q + (size_t)head * R * C::RB;
  const int ks = wave / C::RW;                       // this wave's share of a tile's subtiles
  const int row0 = (wave % C::RW) * NRB * 16;
  const bool active = row0 < R;

  Chunk16 q[NRB][C::NCH];
  load_q<typename C::T, C::D, NRB>(Qh, R, row0, col, grp, q);
  float m[NRB][4], s[NRB][4];
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      m[rb][i] = kNegInf;
      s[rb][i] = 0.f;
    }
  const int kb = chunk * a.chunk_keys;
  const int ke = min(n, kb + a.chunk_keys);
  const int full_end = min(ke, n - W + 1);

  auto no_pre = [] {};
  auto no_vhook = [](int, const Chunk16 (&)[C::LPT]) {};
  auto no_after = [](int) {};
  tiled_stream<C, false>(Kh, nullptr, kb, ke, tid, lds, no_pre, no_vhook, [&](const char* stage, int tile) {
    f32x4 acc[C::SUB][NRB];
#pragma unroll
    for (int k2 = 0; k2 < C::SUB; ++k2) tile_logits<C>(stage, ks * C::SUB + k2, col, grp, q, acc[k2]);
    if (!active) return;
#pragma unroll
    for (int k2 = 0; k2 < C::SUB; ++k2) {
      const int t = kb + tile * C::TK + (ks * C::SUB + k2) * 16;
      if (t >= ke) break;
      const bool fast = t + 16 <= full_end;
      if (fast) {
        f32x4 x[NRB];
        float top = kNegInf;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
#pragma unroll
          for (int i = 0; i < 4; ++i) x[rb][i] = fmaf(acc[k2][rb][i], a.c2, -m[rb][i]);
          top = fmaxf(fmaxf(top, x[rb][0]), fmaxf(fmaxf(x[rb][1], x[rb][2]), x[rb][3]));
        }
        if (!__any(top > kRefSlack)) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) s[rb][i] += fast_exp2(x[rb][i]);
          continue;
        }
      }
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const bool valid = fast || row_sees(row0 + rb * 16 + grp * 4 + i, t + col, R, W, n, ke);
          const float x = acc[k2][rb][i] * a.c2;
          const float dlt = x - m[rb][i];
          const float e = fast_exp2(-fabsf(dlt));
          const bool up = valid && dlt > 0.f;
          s[rb][i] = up ? fmaf(s[rb][i], e, 1.f) : s[rb][i] + (valid ? e : 0.f);
          m[rb][i] = up ? x : m[rb][i];
        }
    }
  }, no_after);

#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) {
        const float m2 = xor_shfl(m[rb][i], off);
        const float s2 = xor_shfl(s[rb][i], off);
        lse_merge(m[rb][i], s[rb][i], m2, s2);
      }
  // the KS waves that hold the same rows merge in key order (through the
  // tile stages, free since the stream's last barrier)
  float2* red = reinterpret_cast<float2*>(lds[0]);   // [KS - 1][ROWS]
  static_assert((C::KS - 1) * C::ROWS * (int)sizeof(float2) <= C::TILE, "row statistics fit one stage");
  if constexpr (C::KS > 1) {
    if (ks > 0 && col == 0) {
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          red[(ks - 1) * C::ROWS + row0 + rb * 16 + grp * 4 + i] = make_float2(m[rb][i], s[rb][i]);
    }
    __syncthreads();
  }
  if (ks == 0 && col == 0) {
#pragma unroll
    for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = row0 + rb * 16 + grp * 4 + i;
        float mm = m[rb][i], ss = s[rb][i];
#pragma unroll
        for (int k = 1; k < C::KS; ++k) lse_merge(mm, ss, red[(k - 1) * C::ROWS + r].x, red[(k - 1) * C::ROWS + r].y);
        a.part[((size_t)head * a.nchunks + chunk) * a.rpad + r] = make_float2(mm, ss);
      }
  }
}

// A workgroup barrier for LDS data that leaves loads in flight.
__device__ __forceinline__ void lds_sync() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Merges the chunk partials of the head's rows for this workgroup: every
// thread takes two rows (one 16-byte load per chunk) of every GROUPS-th
// chunk, the groups then combine in order through `red` (LDS,
// GROUPS * ROWS float2).  Leaves -M in s_off and 1/L in s_inv (padding rows:
// -inf and 0, whose probabilities are then 0).  Every workgroup of a head
// forms the same values in the same order.
template <class C>
__device__ __forceinline__ void merge_partials(const ScoreArgs& a, int64_t head, int tid, float2* red, float* s_off,
                                               float* s_inv) {
  constexpr int PAIRS = C::ROWS / 2;
  constexpr int GROUPS = C::NT / PAIRS;
  constexpr int kBatch = 8;   // partial loads in flight per thread
  if (a.merged) {             // the whole workgroup
    if (tid < C::ROWS) {
      const float2 v = a.stats[(size_t)head * C::ROWS + tid];
      s_off[tid] = v.x;
      s_inv[tid] = v.y;
    }
    lds_sync();
    return;
  }
  const int pair = tid % PAIRS, g = tid / PAIRS;
  const float2* p = a.part + (size_t)head * a.nchunks * C::ROWS + pair * 2;
  float M0 = kNegInf, L0 = 0.f, M1 = kNegInf, L1 = 0.f;
  for (int c0 = g; c0 < a.nchunks; c0 += GROUPS * kBatch) {
    float4 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      v[u] = *reinterpret_cast<const float4*>(p + (size_t)min(c0 + u * GROUPS, a.nchunks - 1) * C::ROWS);
#pragma unroll
    for (int u = 0; u < kBatch; ++u)
      if (c0 + u * GROUPS < a.nchunks) {
        lse_merge(M0, L0, v[u].x, v[u].y);
        lse_merge(M1, L1, v[u].z, v[u].w);
      }
  }
  *reinterpret_cast<float4*>(&red[g * C::ROWS + pair * 2]) = make_float4(M0, L0, M1, L1);
  lds_sync();
  if (tid < C::ROWS) {
    float M = kNegInf, L = 0.f;
#pragma unroll
    for (int k = 0; k < GROUPS; ++k) {
      const float2 v = red[k * C::ROWS + tid];
      lse_merge(M, L, v.x, v.y);
    }
    const bool live = tid < a.R && L > 0.f;
    s_off[tid] = live ? -M : kNegInf;
    s_inv[tid] = live ? 1.f / L : 0.f;
  }
  lds_sync();
}

template <class C>
__global__ __launch_bounds__(C::NT, C::NW == 4 ? (sizeof(typename C::T) == 2 ? 3 : 2) : 1) void score_colsum_tiled(ScoreArgs a) {
  constexpr int NRB = C::NRB;
  __shared__ __align__(16) char lds[2][C::TILE];
  __shared__ float s_cs[2][C::RW][C::TK];   // per-row-wave column sums of a tile
  __shared__ float s_vn[3][C::TK];          // squared value norms of a tile
  // a and ||v|| of the keys not yet written; before the first tile, the merge of the partials
  __shared__ __align__(16) float s_out[2][kOutKeys];
  // -M and 1/L of the rows, read from LDS where they are used (four
  // consecutive rows per 16-byte read) to stay within the register budget
  __shared__ __align__(16) float s_off[C::ROWS], s_inv[C::ROWS];
  const int chunk = blockIdx.x;
  const int64_t head = blockIdx.y;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int col = lane & 15, grp = lane >> 4;
  const int n = a.n, W = a.W, R = a.R;
  const char* Kh = a.K + (size_t)head * n * C::RB;
  const char* Vh = a.V + (size_t)head * n * C::RB;
  const char* Qh = a.Q + (size_t)head * R * C::RB;
  const int ks = wave / C::RW, rw = wave % C::RW;
  const int row0 = rw * NRB * 16;
  const bool active = row0 < R;

  Chunk16 q[NRB][C::NCH];
  load_q<typename C::T, C::D, NRB>(Qh, R, row0, col, grp, q);
  static_assert(C::NT / (C::ROWS / 2) * C::ROWS * (int)sizeof(float2) <= (int)sizeof(s_out), "merge fits the outputs' LDS");
  const int kb = chunk * a.chunk_keys2;
  const int ke = min(n, kb + a.chunk_keys2);
  const int full_end = min(ke, n - W + 1);
  const float G = (float)a.G;

  // squared value norms: each thread's pieces of a V tile (bf16: four pairs,
  // each squared and summed by one fp32-accumulating dot2), summed over the
  // NCHUNK consecutive threads that hold one row (fixed order)
  auto vnorms = [&](int tile, const Chunk16 (&v)[C::LPT]) {
#pragma unroll
    for (int j = 0; j < C::LPT; ++j) {
      float ss = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (sizeof(typename C::T) == 2) {
          const bf16x2 x = __builtin_bit_cast(bf16x2, v[j].w[e]);
          ss = __builtin_amdgcn_fdot2_f32_bf16(x, x, ss, false);
        } else {
          const float x = __uint_as_float(v[j].w[e]);
          ss = fmaf(x, x, ss);
        }
      }
#pragma unroll
      for (int o = C::NCHUNK / 2; o >= 1; o >>= 1) ss += xor_shfl(ss, o);
      int row, ch;
      piece<C>(j, tid, row, ch);
      if (ch == 0) s_vn[tile % 3][row] = ss;
    }
  };
  auto merge = [&] { merge_partials<C>(a, head, tid, reinterpret_cast<float2*>(s_out), s_off, s_inv); };
  float* attn = a.attn + (size_t)head * n;
  float* vnorm = a.vnorm + (size_t)head * n;

  tiled_stream<C, true>(Kh, Vh, kb, ke, tid, lds, merge, vnorms, [&](const char* stage, int tile) {
    f32x4 acc[C::SUB][NRB];
#pragma unroll
    for (int k2 = 0; k2 < C::SUB; ++k2) tile_logits<C>(stage, ks * C::SUB + k2, col, grp, q, acc[k2]);
#pragma unroll
    for (int k2 = 0; k2 < C::SUB; ++k2) {
      const int kk = ks * C::SUB + k2;
      const int t = kb + tile * C::TK + kk * 16;
      float cs = 0.f;
      if (active && t < ke) {
        f32x4 off[NRB], inv[NRB];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb) {
          off[rb] = *reinterpret_cast<const f32x4*>(&s_off[row0 + rb * 16 + grp * 4]);
          inv[rb] = *reinterpret_cast<const f32x4*>(&s_inv[row0 + rb * 16 + grp * 4]);
        }
        if (t + 16 <= full_end) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) cs = fmaf(fast_exp2(fmaf(acc[k2][rb][i], a.c2, off[rb][i])), inv[rb][i], cs);
        } else {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float p = fast_exp2(fmaf(acc[k2][rb][i], a.c2, off[rb][i]));
              const bool vis = row_sees(row0 + rb * 16 + grp * 4 + i, t + col, R, W, n, ke);
              cs = fmaf(vis ? p : 0.f, inv[rb][i], cs);
            }
        }
        cs = add_xor16(cs);
        cs = add_xor32(cs);
      }
      if (grp == 0) s_cs[tile & 1][rw][kk * 16 + col] = cs;
    }
  }, [&](int tile) {
    // wave 0 alone fills and empties s_out (its LDS accesses stay in order)
    static_assert(C::TK <= 64, "one wave finishes a tile's keys");
    if (tid < 64) {
      const int at = (tile * C::TK) % kOutKeys;
      if (tid < C::TK) {
        float part[C::RW];   // the row waves' sums, added pairwise
#pragma unroll
        for (int w = 0; w < C::RW; ++w) part[w] = s_cs[tile & 1][w][tid];
#pragma unroll
        for (int step = 1; step < C::RW; step *= 2)
#pragma unroll
          for (int w = 0; w + step < C::RW; w += 2 * step) part[w] += part[w + step];
        s_out[0][at + tid] = part[0] / G;
        s_out[1][at + tid] = sqrtf(s_vn[tile % 3][tid]);
      }
      const int done = tile * C::TK + C::TK;             // keys finished
      if (at + C::TK == kOutKeys || kb + done >= ke) {   // wave-uniform: the buffer is full, or the chunk ends
        const int first = kb + tile * C::TK - at;
        for (int k = tid; first + k < min(ke, kb + done); k += 64) {
          attn[first + k] = s_out[0][k];
          vnorm[first + k] = s_out[1][k];
        }
      }
    }
  });
}

template <typename T, int D, int NRB, int RW>
hipError_t launch_t(const Shape& s, const ScorePlan& p, ScoreArgs& a, float* score, int pool_kernel,
                    hipStream_t st) {
  const dim3 blk(kThreads);
  hipLaunchKernelGGL((score_rowstats_kernel<T, D, NRB, RW>), dim3(p.nchunks, (unsigned)s.heads, p.nrg), blk, 0, st,
                     a);
  hipLaunchKernelGGL(score_combine_kernel, dim3((unsigned)s.heads), blk, 0, st, a);
  hipLaunchKernelGGL((score_colsum_kernel<T, D, NRB, RW>), dim3(p.nchunks, (unsigned)s.heads), blk, 0, st, a);
  if (s.n_cand > 0)
    hipLaunchKernelGGL(score_pool_kernel, dim3((s.n_cand + kPoolOut - 1) / kPoolOut, (unsigned)s.heads), blk, 0,
                       st, a.attn, a.vnorm, score, s.n, s.n_cand, pool_kernel);
  return hipGetLastError();
}

// General passes: row blocks per wave and waves sharing a tile.  128 rows per
// row group; fp32 at d = 128 keeps 32, so Q stays within 64 VGPRs per wave.
template <typename T, int D>
struct General {
  static constexpr bool kWide = sizeof(T) == 4 && D == 128;
  static constexpr int NRB = kWide ? 2 : 4, RW = kWide ? 1 : 2;
};

template <typename T, int D>
hipError_t launch_d(const Shape& s, const ScorePlan& p, ScoreArgs& a, float* score, int pool_kernel,
                    hipStream_t st) {
  return launch_t<T, D, General<T, D>::NRB, General<T, D>::RW>(s, p, a, score, pool_kernel, st);
}

// Calls f with the shared-tile configuration that holds `rows` window rows.
template <typename T, int D, typename F>
void with_tiled(int rows, F&& f) {
  switch (rows) {
    case 32: f(Tiled<T, D, 4, 1, 2>{}); break;
    case 64: f(Tiled<T, D, 4, 2, 2>{}); break;
    case 128: f(Tiled<T, D, 4, 2, 4>{}); break;
    default: f(Tiled<T, D, 8, 2, 8>{}); break;
  }
}

template <typename T, int D>
hipError_t launch_tiled(const Shape& s, const ScorePlan& p, ScoreArgs& a, float* score, int pool_kernel,
                        hipStream_t st) {
  with_tiled<T, D>(p.rpad, [&](auto c) {
    using C = decltype(c);
    hipLaunchKernelGGL(score_rowstats_tiled<C>, dim3(p.nchunks, (unsigned)s.heads), dim3(C::NT), 0, st, a);
    if (p.combine) hipLaunchKernelGGL(score_combine_kernel, dim3((unsigned)s.heads), dim3(kThreads), 0, st, a);
    hipLaunchKernelGGL(score_colsum_tiled<C>, dim3(p.nchunks2, (unsigned)s.heads), dim3(C::NT), 0, st, a);
  });
  if (s.n_cand > 0)
    hipLaunchKernelGGL(score_pool_kernel, dim3((s.n_cand + kPoolOut - 1) / kPoolOut, (unsigned)s.heads),
                       dim3(kThreads), 0, st, a.attn, a.vnorm, score, s.n, s.n_cand, pool_kernel);
  return hipGetLastError();
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

ScorePlan plan_score(const Shape& s, int dtype) {
  ScorePlan p{};
  if (s.R <= kTiledRows) {
    // shared-tile passes: the smallest configuration that holds the rows
    p.tiled = 1;
    int rows = 32;
    while (rows < s.R) rows *= 2;
    p.nrg = 1;
    p.rpad = rows;
    // Keys per workgroup.  A workgroup pays for its queries, the merge of the
    // partials and the first tiles before it streams, so a call that two
    // workgroups per CU can hold gets just those: one 8192-token layer (8
    // heads) takes 28 us and one 102400-token layer 136 us with 512 workgroups
    // per pass (165 and 231 us when pass 2 had one per 4096 keys); 158 us with
    // 2048 + 768 workgroups, 466 us with 6400 each; with fewer the reads in
    // flight run short (173 us at 512 + 256).  The 8-wave configuration fills
    // a CU with one (a 32768-token layer with a window of 64: 80 us against
    // 98 at two).  Calls beyond that get short chunks, so that the last round
    // of workgroups is small beside the call: 32 layers of 102400 tokens take
    // 3.74 ms with 2048 + 1024 keys per workgroup, 3.80 ms with 12800 + 4096,
    // 4.2 - 4.3 ms with 512 workgroups.  Their many workgroups would repeat
    // the merge of the partials, so one kernel does it first (6 - 12 us of the
    // call).  fp32 at d = 64 keeps the matrix cores busy longest and fits
    // three workgroups on a CU, which pays once their chunks are long (16
    // layers of 16384 tokens: 659 us with 768 workgroups, 695 with 512; one
    // layer of 32768: 108 against 105); the others lose by it (d = 128, one
    // layer of 102400: 648 against 507 us).
    const int tk = rows > 128 ? 64 : 32;   // keys per tile
    const int64_t tiles = (s.n + tk - 1) / tk, total = tiles * s.heads;
    const int64_t few = rows > 128 ? 256 : dtype == SELKV_F32 && s.d == 64 && total >= 32768 ? 768 : 512;
    auto chunk_tiles = [&](int64_t least) { return std::min(std::max((total + few - 1) / few, least), tiles); };
    // The fewest tiles of a chunk, in calls that leave CUs idle.  An fp32 tile
    // of the eight waves of 129 to 256 rows is long work: two and one are
    // enough (8 heads x 600 tokens, d = 128: 48.5 us; 75 us with four and two,
    // 57.5 by the general passes).  One in pass 1 too would take 40 us, but its
    // partials are so many that attn is 3% further from its 64-bit value
    // (3.45e-8 against 3.35e-8; 4.8e-8 by the general passes).
    const bool slow = rows > 128 && dtype == SELKV_F32;
    int64_t t1 = chunk_tiles(slow ? 2 : 4), t2 = chunk_tiles(slow ? 1 : 2);
    if (t1 > 8192 / tk) t1 = std::max<int64_t>(2048 / tk, (tiles + 511) / 512);   // at most 512 partials to merge per row
    if (t2 > 4096 / tk) {
      t2 = 1024 / tk;
      p.combine = 1;
    }
    p.chunk_keys = (int)(t1 * tk);
    p.nchunks = (int)((tiles + t1 - 1) / t1);
    p.chunk_keys2 = (int)(t2 * tk);
    p.nchunks2 = (int)((tiles + t2 - 1) / t2);
    p.part_off = 0;
    p.stats_off = align256((size_t)s.heads * p.nchunks * p.rpad * sizeof(float2));
    p.bytes = p.stats_off + align256((size_t)s.heads * p.rpad * sizeof(float2));
    return p;
  }
  const int rows = (dtype == SELKV_F32 && s.d == 128) ? 32 : 128;   // as General
  p.nrg = (s.R + rows - 1) / rows;
  p.rpad = p.nrg * rows;

  const int64_t tiles = (s.n + 63) / 64;
  int64_t nchunks = (kTargetBlocks + s.heads - 1) / s.heads;
  if (nchunks > tiles) nchunks = tiles;
  if (nchunks < 1) nchunks = 1;
  int64_t ck = ((s.n + nchunks - 1) / nchunks + 63) / 64 * 64;
  const int64_t n64 = ((int64_t)s.n + 63) / 64 * 64;
  const int64_t min_ck = n64 < kMinChunkKeys ? n64 : kMinChunkKeys;
  if (ck < min_ck) ck = min_ck;
  if (ck > kMaxChunkKeys) ck = kMaxChunkKeys;
  p.chunk_keys = (int)ck;
  p.nchunks = (int)((s.n + ck - 1) / ck);

  p.part_off = 0;
  p.stats_off = align256((size_t)s.heads * p.nchunks * p.rpad * sizeof(float2));
  p.bytes = p.stats_off + align256((size_t)s.heads * p.rpad * sizeof(float2));
  return p;
}

namespace {

ScoreArgs make_args(const Shape& s, const ScorePlan& p, float scale, const void* K, const void* V, const void* Qwin,
                    float* attn, float* vnorm, void* ws) {
  ScoreArgs a{};
  a.K = static_cast<const char*>(K);
  a.V = static_cast<const char*>(V);
  a.Q = static_cast<const char*>(Qwin);
  a.attn = attn;
  a.vnorm = vnorm;
  char* w = static_cast<char*>(ws);
  a.part = reinterpret_cast<float2*>(w + p.part_off);
  a.stats = reinterpret_cast<float2*>(w + p.stats_off);
  a.n = s.n;
  a.W = s.W;
  a.R = s.R;
  a.G = s.G;
  a.chunk_keys = p.chunk_keys;
  a.nchunks = p.nchunks;
  a.chunk_keys2 = p.chunk_keys2;
  a.merged = p.combine;
  a.rpad = p.rpad;
  a.nrg = p.nrg;
  a.c2 = scale * kLog2e;
  return a;
}

template <typename T, int D>
void launch_rowstats_general(const Shape& s, const ScorePlan& p, const ScoreArgs& a, hipStream_t st) {
  hipLaunchKernelGGL((score_rowstats_kernel<T, D, General<T, D>::NRB, General<T, D>::RW>),
                     dim3(p.nchunks, (unsigned)s.heads, p.nrg), dim3(kThreads), 0, st, a);
}

}  // namespace

hipError_t launch_row_stats(const Shape& s, const ScorePlan& p, int dtype, float scale, const void* K,
                            const void* Qwin, void* ws, hipStream_t st) {
  const ScoreArgs a = make_args(s, p, scale, K, nullptr, Qwin, nullptr, nullptr, ws);
  if (p.tiled) {
    auto go = [&](auto c) {
      using C = decltype(c);
      hipLaunchKernelGGL(score_rowstats_tiled<C>, dim3(p.nchunks, (unsigned)s.heads), dim3(C::NT), 0, st, a);
    };
    if (dtype == SELKV_BF16 && s.d == 128) with_tiled<bf16_t, 128>(p.rpad, go);
    else if (dtype == SELKV_BF16) with_tiled<bf16_t, 64>(p.rpad, go);
    else if (s.d == 128) with_tiled<float, 128>(p.rpad, go);
    else with_tiled<float, 64>(p.rpad, go);
  } else if (dtype == SELKV_BF16) {
    if (s.d == 128) launch_rowstats_general<bf16_t, 128>(s, p, a, st);
    else launch_rowstats_general<bf16_t, 64>(s, p, a, st);
  } else {
    if (s.d == 128) launch_rowstats_general<float, 128>(s, p, a, st);
    else launch_rowstats_general<float, 64>(s, p, a, st);
  }
  hipLaunchKernelGGL(score_combine_kernel, dim3((unsigned)s.heads), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_score(const Shape& s, const ScorePlan& p, int dtype, float scale, const void* K, const void* V,
                        const void* Qwin, float* score, float* attn, float* vnorm, int pool_kernel, void* ws,
                        hipStream_t st) {
  ScoreArgs a = make_args(s, p, scale, K, V, Qwin, attn, vnorm, ws);
  if (p.tiled) {
    if (dtype == SELKV_BF16 && s.d == 128) return launch_tiled<bf16_t, 128>(s, p, a, score, pool_kernel, st);
    if (dtype == SELKV_BF16) return launch_tiled<bf16_t, 64>(s, p, a, score, pool_kernel, st);
    if (s.d == 128) return launch_tiled<float, 128>(s, p, a, score, pool_kernel, st);
    return launch_tiled<float, 64>(s, p, a, score, pool_kernel, st);
  }
  if (dtype == SELKV_BF16) {
    if (s.d == 128) return launch_d<bf16_t, 128>(s, p, a, score, pool_kernel, st);
    return launch_d<bf16_t, 64>(s, p, a, score, pool_kernel, st);
  }
  if (s.d == 128) return launch_d<float, 128>(s, p, a, score, pool_kernel, st);
  return launch_d<float, 64>(s, p, a, score, pool_kernel, st);
}

}  // namespace selkv
