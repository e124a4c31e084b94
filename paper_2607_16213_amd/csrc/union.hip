// GQA union mode (Sec. 3.3 union selection, Sec. 3.6 GQA rule) for
// selkv_select / selkv_bias with SELKV_SELECT_UNION.
//
//   select  the selection kernel runs over the heads and sets their picks'
//           bits in one row per cache, the flagged candidates get their mean score across the heads
//           (fp32, head order) and the rest -inf, and the same selection
//           kernel picks the m_s best means (lower position on ties) plus the
//           recent window and writes them for every head of the cache.
//   bias    the bias kernels write each head's R - 1 (absorbed / a); one pass
//           averages it over the heads of the cache in head order and writes
//           alpha * log1p(mean) for every head.
// The bits are set by integer atomics (or), so the outcome does not depend on
// scheduling.
#include "common.hpp"
#include "internal.hpp"

namespace selkv {
namespace {

constexpr int kThreads = 256;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

__global__ __launch_bounds__(kThreads) void clear_flags_kernel(uint64_t* p, int64_t words) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i < words) p[i] = 0ull;
}

// key[b][j] = mean over the cache's heads of score[b, h, j] if flagged, else -inf.
__global__ __launch_bounds__(kThreads) void union_key_kernel(const float* score, const uint64_t* flag, float* key,
                                                             int hkv, int n_cand) {
  const int64_t b = blockIdx.y;
  const int j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= n_cand) return;
  const size_t o = (size_t)b * n_cand + j;
  float v = kNegInf;
  if ((flag[b * ((n_cand + 63) / 64) + j / 64] >> (j % 64)) & 1ull) {
    float acc = 0.f;
    for (int h = 0; h < hkv; ++h) acc += score[((size_t)b * hkv + h) * n_cand + j];
    v = acc / (float)hkv;
  }
  key[o] = v;
}

// bias[b, h, s] = alpha * log1p(mean over h' of r1[b, h', s]) for every h.
__global__ __launch_bounds__(kThreads) void union_bias_kernel(const float* r1, float* bias, int hkv, int m,
                                                              float alpha) {
  const int64_t b = blockIdx.y;
  const int s = blockIdx.x * kThreads + threadIdx.x;
  if (s >= m) return;
  float acc = 0.f;
  for (int h = 0; h < hkv; ++h) acc += r1[((size_t)b * hkv + h) * m + s];
  const float mean = acc / (float)hkv;
  const float v = mean > 0.f ? alpha * log1pf(mean) : 0.f;
  for (int h = 0; h < hkv; ++h) bias[((size_t)b * hkv + h) * m + s] = v;
}

}  // namespace

UnionPlan plan_union(const Shape& s) {
  UnionPlan p{};
  const size_t batch = (size_t)(s.heads / s.hkv);
  const size_t nc = s.n_cand > 0 ? (size_t)s.n_cand : 1;
  p.key_off = 0;
  p.flag_off = p.key_off + align256(batch * nc * sizeof(float));
  // one bit per candidate in 64-bit words; the reported size keeps the four
  // bytes per candidate it has always had where the words take less
  const size_t words = batch * ((nc + 63) / 64) * sizeof(uint64_t), ints = batch * nc * sizeof(int32_t);
  p.select_bytes = p.flag_off + align256(words > ints ? words : ints);
  p.ratio_bytes = align256((size_t)s.heads * s.m * sizeof(float));
  return p;
}

hipError_t launch_union_select(const Shape& s, const UnionPlan& p, const float* score, int32_t* kept,
                               int32_t* evicted, void* ws, hipStream_t st) {
  // only the recent window is kept: every head's own lists are the shared ones
  if (s.ms == 0 || s.n_cand == 0) return launch_select(s, score, kept, evicted, st);
  const int64_t batch = s.heads / s.hkv;
  char* w = static_cast<char*>(ws);
  uint64_t* flag = reinterpret_cast<uint64_t*>(w + p.flag_off);
  float* key = reinterpret_cast<float*>(w + p.key_off);
  const int64_t words = batch * ((s.n_cand + 63) / 64);
  hipLaunchKernelGGL(clear_flags_kernel, dim3((unsigned)((words + kThreads - 1) / kThreads)), dim3(kThreads), 0, st,
                     flag, words);
  hipError_t e = launch_select_flags(s, score, flag, st);         // every head's own picks
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(union_key_kernel, dim3((s.n_cand + kThreads - 1) / kThreads, (unsigned)batch), dim3(kThreads),
                     0, st, score, flag, key, s.hkv, s.n_cand);
  Shape su = s;
  su.heads = batch;
  su.hkv = 1;
  return launch_select_shared(su, key, kept, evicted, s.hkv, st);
}

hipError_t launch_union_bias(const Shape& s, const float* r1, float* bias, float alpha, hipStream_t st) {
  const int64_t batch = s.heads / s.hkv;
  hipLaunchKernelGGL(union_bias_kernel, dim3((s.m + kThreads - 1) / kThreads, (unsigned)batch), dim3(kThreads), 0,
                     st, r1, bias, s.hkv, s.m, alpha);
  return hipGetLastError();
}

}  // namespace selkv
