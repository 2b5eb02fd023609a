// Router inference (paper, Sec. "Dependency-Closed Masks and Cache-Consistent Routing"; appendix
// paragraph "Router feature specification"): per prompt, a feature vector of hashed character
// trigrams (projected by a frozen random map), length, proxy-LM log-probability, character-class
// counts and five task descriptors; a three-layer MLP over it; temperature-scaled softmax; the
// dense plan when the top probability is below tau.
//
//   1. router_features_kernel, one workgroup of 1024 threads per prompt. The prompt is staged
//      through LDS in chunks with a small halo on both sides (bytes outside the prompt read as
//      zero, which no pattern byte equals; all byte loads of a chunk are in flight together).
//      A thread examines eight consecutive positions from 24 bytes in registers, case-folded eight
//      at a time: each position's trigram's 32-bit FNV-1a hash goes into an LDS histogram by an
//      LDS atomic increment (integer, so the histogram does not depend on the order of the
//      increments), its byte is classified through a table, and the descriptor patterns that can
//      start there are matched as words. Counts and descriptor bits are combined per wave and
//      then by LDS atomics; the workgroup writes the term frequencies [n_bins] and the 11 scalar
//      features. (A 7350-byte prompt: 26 us one byte at a time from LDS, mostly dependent LDS
//      reads of the patterns, byte classification and 5000 serialised atomics on five words.)
//   2. router_dense_kernel, launched three times (projection, hidden layer 1, hidden layer 2):
//      one wave per output row, lanes strided over the row, up to 8 prompts per workgroup
//      sharing each weight load, 512 weights of the row in flight at a time (the 2048-wide
//      projection of one prompt took 14 us with one load in flight); bias and ReLU in the epilogue;
//   3. router_head_kernel, one workgroup per prompt: the task logits, softmax of logits /
//      temperature (shifted by the maximum), the top probability (lowest task on ties) and the
//      decision.
// Everything is float32 except the text scan, which is integer and exact.
#include "device_common.hpp"
#include "kernels.hpp"

namespace tasp {
namespace {

constexpr int kFeatBlock = 1024;      // threads of the features kernel (one workgroup per prompt)
constexpr int kChunk = 8192;          // prompt bytes staged per round
constexpr int kHalo = 16;             // bytes kept on either side of a chunk (patterns need <= 9)
constexpr int kStaged = kChunk + 2 * kHalo;
constexpr int kStage = (kStaged + kFeatBlock - 1) / kFeatBlock;   // byte loads per thread
constexpr int kDenseRows = kBlock / kWave;   // output rows per workgroup
constexpr int kDensePrompts = 8;             // prompts per workgroup

enum : unsigned { kNumbered = 1u, kFence = 2u, kTranslate = 4u, kOptA = 8u, kOptB = 16u,
                  kRetrieval = 32u };

__device__ __forceinline__ unsigned fold(unsigned c) { return (c - 65u < 26u) ? c + 32u : c; }
__device__ __forceinline__ bool is_digit(unsigned c) { return c - 48u < 10u; }
__device__ __forceinline__ bool is_letter(unsigned c) { return (c | 32u) - 97u < 26u; }
__device__ __forceinline__ bool is_alnum(unsigned c) { return is_digit(c) || is_letter(c); }
__device__ __forceinline__ bool is_operator(unsigned c) {
  return c == '+' || c == '-' || c == '*' || c == '/' || c == '=' || c == '<' || c == '>' ||
         c == '%' || c == '^';
}
__device__ __forceinline__ bool is_code_punct(unsigned c) {
  return c == '{' || c == '}' || c == '[' || c == ']' || c == '(' || c == ')' || c == ';' ||
         c == '_' || c == '#' || c == '`' || c == '\\' || c == '|' || c == '&';
}

// FNV-1a (32-bit) of three bytes
__device__ __forceinline__ uint32_t fnv1a3(unsigned b0, unsigned b1, unsigned b2) {
  uint32_t h = 2166136261u;
  h = (h ^ b0) * 16777619u;
  h = (h ^ b1) * 16777619u;
  h = (h ^ b2) * 16777619u;
  return h;
}

// eight bytes with ASCII capitals folded to lower case
__device__ __forceinline__ uint64_t fold8(uint64_t x) {
  const uint64_t h = x & 0x7f7f7f7f7f7f7f7full;
  const uint64_t ge_a = h + 0x3f3f3f3f3f3f3f3full, gt_z = h + 0x2525252525252525ull;   // bit 7 of each byte
  return x | (((ge_a ^ gt_z) & ~x & 0x8080808080808080ull) >> 2);
}
constexpr uint64_t word_of(const char* s, int n) {
  uint64_t v = 0;
  for (int i = 0; i < n; ++i) v |= uint64_t(uint8_t(s[i])) << (8 * i);
  return v;
}
__device__ __forceinline__ unsigned byte_of(uint64_t w, int i) { return unsigned(w >> (8 * i)) & 0xffu; }

// descriptor patterns that start at the first byte of w (the eight bytes at a position; f: folded)
__device__ __forceinline__ unsigned patterns_at(uint64_t w, uint64_t f, bool line_start, bool word_start) {
  unsigned fl = 0;
  if (line_start) {
    int k = 0;
    while (k < 3 && is_digit(byte_of(w, k))) ++k;
    const unsigned e = byte_of(w, k);
    if (k > 0 && (e == '.' || e == ')') && byte_of(w, k + 1) == ' ') fl |= kNumbered;
    unsigned lab = 0xffu;
    const unsigned c0 = byte_of(w, 0), c1 = byte_of(w, 1), c2 = byte_of(w, 2);
    if (c0 == '(' && c1 - 65u < 4u && c2 == ')' && byte_of(w, 3) == ' ') lab = c1 - 65u;
    else if (c0 - 65u < 4u && (c1 == '.' || c1 == ')') && c2 == ' ') lab = c0 - 65u;
    if (lab == 0) fl |= kOptA;
    if (lab == 1) fl |= kOptB;
  }
  if ((w & 0xffffffu) == word_of("```", 3)) fl |= kFence;
  if (f == word_of("translat", 8)) fl |= kTranslate;
  if (word_start && (f & 0xffffu) == word_of("wh", 2)) {
    if (((f & 0xffffffu) == word_of("who", 3) && !is_letter(byte_of(f, 3))) ||
        ((f & 0xffffffffull) == word_of("when", 4) && !is_letter(byte_of(f, 4))) ||
        (((f & 0xffffffffffull) == word_of("where", 5) || (f & 0xffffffffffull) == word_of("which", 5)) &&
         !is_letter(byte_of(f, 5))))
      fl |= kRetrieval;
  }
  return fl;
}

// sum over the wave
__device__ __forceinline__ int wave_sum_int(int v) {
  v += __builtin_amdgcn_mov_dpp(v, kQuadXor1, 0xF, 0xF, true);
  v += __builtin_amdgcn_mov_dpp(v, kQuadXor2, 0xF, 0xF, true);
  v += __builtin_amdgcn_mov_dpp(v, kRowHalfMirror, 0xF, 0xF, true);
  v += __builtin_amdgcn_mov_dpp(v, kRowMirror, 0xF, 0xF, true);
  return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) + __builtin_amdgcn_readlane(v, 32) +
         __builtin_amdgcn_readlane(v, 48);
}

__global__ __launch_bounds__(kFeatBlock) void router_features_kernel(RouterFeatArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint32_t hist[];     // [n_bins]
  __shared__ __attribute__((aligned(16))) uint8_t tb[kStaged];
  __shared__ uint32_t cls[256];        // byte class as four 8-bit counters: digit, operator, code, '?'
  __shared__ int cnt[4];
  __shared__ unsigned flags;
  const int b = blockIdx.x, tid = threadIdx.x;
  long start = 0, end = a.n_text;
  if (a.offsets) {
    start = min(max(long(a.offsets[b]), 0L), long(a.n_text));
    end = min(max(long(a.offsets[b + 1]), start), long(a.n_text));
  }
  const int n = int(end - start);
  // this prompt's bytes; loads at an offset past them return zero without touching memory
  const __amdgpu_buffer_rsrc_t rt = make_rsrc(a.text + start, uint32_t(n));
  for (int i = tid; i < a.n_bins; i += kFeatBlock) hist[i] = 0u;
  if (tid < 4) cnt[tid] = 0;
  if (tid == 0) flags = 0u;
  if (tid < 256)
    cls[tid] = (is_digit(tid) ? 1u : 0u) | (is_operator(tid) ? 1u << 8 : 0u) |
               (is_code_punct(tid) ? 1u << 16 : 0u) | (tid == '?' ? 1u << 24 : 0u);
  __syncthreads();
  int cd = 0, co = 0, cc = 0, cq = 0;
  unsigned fl = 0;
  const uint32_t nb = uint32_t(a.n_bins);
  const bool pow2 = (nb & (nb - 1)) == 0;
  for (int c0 = 0; c0 < n; c0 += kChunk) {
    uint8_t v[kStage];
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const int i = u * kFeatBlock + tid;
      const long q = long(c0) - kHalo + i;
      v[u] = __builtin_amdgcn_raw_buffer_load_b8(
          rt, (i < kStaged && q >= 0 && q < n) ? int(q) : int(kOOB), 0, 0);
    }
    __syncthreads();                                   // the previous chunk is consumed
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      const int i = u * kFeatBlock + tid;
      if (i < kStaged) tb[i] = v[u];
    }
    __syncthreads();
    // eight positions from 24 staged bytes: the eight before, the eight, the eight after
    const int p0 = c0 + 8 * tid;
    if (p0 < n) {
      const uint64_t* t8 = reinterpret_cast<const uint64_t*>(tb + kHalo - 8) + tid;
      const uint64_t before = t8[0], cur = t8[1], next = t8[2];
      const uint64_t fcur = fold8(cur), fnext = fold8(next);
      uint32_t packed = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint64_t w = j ? (cur >> (8 * j)) | (next << (64 - 8 * j)) : cur;
        const uint64_t f = j ? (fcur >> (8 * j)) | (fnext << (64 - 8 * j)) : fcur;
        const unsigned prev = j ? byte_of(cur, j - 1) : byte_of(before, 7);
        const int p = p0 + j;
        if (p + 3 <= n) {
          const uint32_t h = fnv1a3(byte_of(f, 0), byte_of(f, 1), byte_of(f, 2));
          atomicAdd(&hist[pow2 ? h & (nb - 1) : h % nb], 1u);
        }
        packed += cls[byte_of(w, 0)];                  // (bytes past the prompt are zero: no class)
        fl |= patterns_at(w, f, p == 0 || prev == '\n', p == 0 || !is_alnum(prev));
      }
      cd += packed & 0xffu;
      co += (packed >> 8) & 0xffu;
      cc += (packed >> 16) & 0xffu;
      cq += packed >> 24;
    }
  }
  cd = wave_sum_int(cd);
  co = wave_sum_int(co);
  cc = wave_sum_int(cc);
  cq = wave_sum_int(cq);
  unsigned any = 0;
#pragma unroll
  for (unsigned bit = kNumbered; bit <= kRetrieval; bit <<= 1) any |= __ballot(fl & bit) ? bit : 0u;
  if ((tid & 63) == 0) {
    atomicAdd(&cnt[0], cd);
    atomicAdd(&cnt[1], co);
    atomicAdd(&cnt[2], cc);
    atomicAdd(&cnt[3], cq);
    atomicOr(&flags, any);
  }
  __syncthreads();
  const float inv_n = float(max(1, n - 2));
  float* tf = a.tf + size_t(b) * a.n_bins;
  for (int i = tid; i < a.n_bins; i += kFeatBlock) tf[i] = float(hist[i]) / inv_n;
  if (tid < kRouterScalars) {
    const unsigned g = flags;
    float v = 0.0f;
    if (tid == 0) v = log1pf(float(n));
    else if (tid == 1) v = a.logprob[b];
    else if (tid < 6) v = log1pf(float(cnt[tid - 2]));
    else if (tid == 6) v = (g & kNumbered) ? 1.0f : 0.0f;
    else if (tid == 7) v = (g & kFence) ? 1.0f : 0.0f;
    else if (tid == 8) v = (g & kTranslate) ? 1.0f : 0.0f;
    else if (tid == 9) v = ((g & kOptA) && (g & kOptB)) ? 1.0f : 0.0f;
    else v = (g & kRetrieval) ? 1.0f : 0.0f;
    a.feats[size_t(b) * a.ld_feats + a.proj_dim + tid] = v;
  }
}

// NB: prompts of the workgroup (at most). The order of a row's sums does not depend on NB, so a
// prompt's result does not depend on the prompts beside it.
template <int NB>
__global__ __launch_bounds__(kBlock) void router_dense_kernel(RouterDenseArgs a) {
  constexpr int U = NB <= 2 ? 8 : 4;                   // row elements in flight per lane
  const int lane = threadIdx.x & 63;
  const int j = blockIdx.x * kDenseRows + (threadIdx.x >> 6);
  const int b0 = blockIdx.y * kDensePrompts;
  if (j >= a.N) return;                               // whole waves leave together
  const int nb = min(NB, a.B - b0);
  // (a row of w and the prompts' inputs; offsets past them read zero)
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.w + size_t(j) * a.K, uint32_t(a.K) * 4u);
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(a.x + size_t(b0) * a.ldx, (uint32_t(nb - 1) * uint32_t(a.ldx) + uint32_t(a.K)) * 4u);
  float acc[NB];
#pragma unroll
  for (int u = 0; u < NB; ++u) acc[u] = 0.0f;
  for (int k0 = lane; k0 - lane < a.K; k0 += U * kWave) {
    float w[U], x[NB][U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int k = k0 + i * kWave;
      w[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rw, k < a.K ? 4 * k : int(kOOB), 0, 0));
#pragma unroll
      for (int u = 0; u < NB; ++u)
        x[u][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                                rx, (k < a.K && u < nb) ? int(uint32_t(u) * uint32_t(a.ldx) + uint32_t(k)) * 4 : int(kOOB), 0, 0));
    }
#pragma unroll
    for (int i = 0; i < U; ++i)
#pragma unroll
      for (int u = 0; u < NB; ++u) acc[u] = fmaf(w[i], x[u][i], acc[u]);
  }
  const float bias = a.bias ? a.bias[j] : 0.0f;
#pragma unroll
  for (int u = 0; u < NB; ++u) {
    const float v = wave_sum(acc[u]) + bias;
    if (lane == 0 && u < nb) a.y[size_t(b0 + u) * a.ldy + j] = a.relu ? fmaxf(v, 0.0f) : v;
  }
}

__global__ __launch_bounds__(kBlock) void router_head_kernel(RouterHeadArgs a) {
  __shared__ float z[kMaxRouterTasks];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* h = a.h + size_t(b) * a.K;
  for (int t = wave; t < a.n_tasks; t += kBlock / kWave) {
    const float* w = a.w + size_t(t) * a.K;
    float acc = 0.0f;
    for (int k = lane; k < a.K; k += kWave) acc = fmaf(w[k], h[k], acc);
    acc = wave_sum(acc);
    if (lane == 0) z[t] = acc + a.bias[t];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  float u[kMaxRouterTasks];
  float m = -INFINITY;
  for (int t = 0; t < a.n_tasks; ++t) {
    u[t] = z[t] / a.temperature;
    m = fmaxf(m, u[t]);
  }
  float s = 0.0f;
  for (int t = 0; t < a.n_tasks; ++t) {
    u[t] = expf(u[t] - m);
    s += u[t];
  }
  float best = -1.0f;
  int task = 0;
  float* p = a.probs + size_t(b) * a.n_tasks;
  for (int t = 0; t < a.n_tasks; ++t) {
    const float v = u[t] / s;
    p[t] = v;
    if (v > best) {
      best = v;
      task = t;
    }
  }
  a.choice[b] = (best >= a.tau) ? task : -1;
}

}  // namespace

size_t router_features_lds_bytes(int n_bins) { return size_t(n_bins) * sizeof(uint32_t); }

hipError_t launch_router_features(const RouterFeatArgs& a, int n_prompts, hipStream_t s) {
  if (n_prompts < 1) return hipSuccess;
  const size_t lds = router_features_lds_bytes(a.n_bins);
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(&router_features_kernel),
      hipFuncAttributeMaxDynamicSharedMemorySize, int(router_features_lds_bytes(kMaxRouterBins)));
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(router_features_kernel, dim3(n_prompts), dim3(kFeatBlock), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_router_dense(const RouterDenseArgs& a, hipStream_t s) {
  if (a.B < 1 || a.N < 1) return hipSuccess;
  const dim3 grid((a.N + kDenseRows - 1) / kDenseRows, (a.B + kDensePrompts - 1) / kDensePrompts);
  if (a.B == 1) hipLaunchKernelGGL(router_dense_kernel<1>, grid, dim3(kBlock), 0, s, a);
  else if (a.B == 2) hipLaunchKernelGGL(router_dense_kernel<2>, grid, dim3(kBlock), 0, s, a);
  else if (a.B <= 4) hipLaunchKernelGGL(router_dense_kernel<4>, grid, dim3(kBlock), 0, s, a);
  else hipLaunchKernelGGL(router_dense_kernel<kDensePrompts>, grid, dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_router_head(const RouterHeadArgs& a, int n_prompts, hipStream_t s) {
  if (n_prompts < 1) return hipSuccess;
  if (a.n_tasks < 1 || a.n_tasks > kMaxRouterTasks) return hipErrorInvalidValue;
  hipLaunchKernelGGL(router_head_kernel, dim3(n_prompts), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace tasp
