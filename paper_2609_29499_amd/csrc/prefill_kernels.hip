// Prefill: the dense BF16 LM head over the prompt's tokens on the BF16 matrix cores, its operand,
// and RoPE with the cache append. (The layers' projections: prefill_i8.hip.)
//
// LM head. y[t][n] = sum_k A[t][k] W[n][k] with v_mfma_f32_16x16x32_bf16 and float32 accumulation.
// The activation A is carried as two BF16 planes, hi = bf16(v) and lo = bf16(v - hi), and every
// tile is multiplied twice (hi, then lo, into the same accumulator), so activations keep 16
// significant bits. The inverse RMS of the final norm is applied per token in the epilogue
// (W (c x) = c (W x)); the operand's producer writes x * gamma and per-64-element sums of squares
// of x, which are reduced once per workgroup.
//
// Tiling. A workgroup computes TM tokens x 128 rows; four waves in a 2 x 2 arrangement own TM / 2 x
// 64 each in 16 x 16 MFMA tiles. K advances in chunks of 32: the global loads of the next three
// chunks are in flight (in registers) while the current chunk's MFMAs run from LDS
// (double-buffered, one barrier per chunk). LDS rows hold one chunk (32 BF16) with their 16-byte
// quarters XOR-swizzled by row (bank-conflict free).
#include <algorithm>

#include "device_common.hpp"
#include "kernels.hpp"
#include "split_sums.hpp"

namespace tasp {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

constexpr int kTMax = 128;             // tokens per workgroup tile (largest)
constexpr int kTN = 128;               // rows per workgroup tile
constexpr int kKC = 32;                // k per chunk
constexpr int kLdsRow = 32;            // BF16 per LDS row (one chunk of k)
constexpr int kSsqBlk = 64;            // elements per sum-of-squares partial
constexpr long kPfMinTiles = 384;      // fewer 128-token tiles than this: use 64-token tiles
constexpr int kMaxKSplit = 8;          // K splits per tile of a layer projection at most
constexpr long kSplitRowCap = 2048;    // (tokens x splits) the partial buffer is sized for

template <int TM>
struct PfSmem {
  uint16_t a[2][2][TM * kLdsRow];      // [buffer][hi/lo][swizzled token row]
  uint16_t b[2][kTN * kLdsRow];        // [buffer][swizzled weight row]
  float rs[TM];                        // inverse RMS of the tile's tokens
};

// LDS offset (BF16 elements) of 16-byte quarter qu of LDS row `row`. Quarters are XOR-swizzled
// with bits 1-4 of the row: the 8 or 16 lanes served together by a 16-byte read (one fragment
// column: 16 consecutive rows, one quarter) or write (4 consecutive rows, all quarters) then
// touch distinct banks.
__device__ __forceinline__ int lds_q(int row, int qu) {
  return row * kLdsRow + 8 * (qu ^ (((row >> 1) ^ (row >> 3)) & 3));
}

template <int TM>
__global__ __launch_bounds__(kBlock) void pf_head_kernel(PfHeadArgs a) {
  constexpr int MT = TM / 32;                           // token tiles of 16 per wave
  constexpr int APT = TM / 32;                          // A pieces per thread and chunk
  __shared__ __attribute__((aligned(16))) PfSmem<TM> sm;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int r = lane & 15, q = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int T = a.T, N = a.N, K = a.K;
  const int m0 = blockIdx.y * TM, n0 = blockIdx.x * kTN;
  const int nk = (K + kKC - 1) / kKC;

  // ---- global -> register staging of one chunk
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.x, uint32_t(2 * a.plane) * 2u);
  const uint32_t row_bytes = uint32_t(K) * 2u;
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(a.w, uint32_t(N) * row_bytes);
  // A pieces: thread t loads pieces t + 256 i (i < APT): plane, token row, 16-byte quarter
  auto a_off = [&](int i, int k0) -> uint32_t {
    const int p = tid + kBlock * i;
    const int plane = p / (4 * TM), row = (p >> 2) & (TM - 1), qu = p & 3;
    const int t = m0 + row;
    const int k = k0 + 8 * qu;
    return (t < T && k < a.ldx) ? uint32_t(plane) * uint32_t(a.plane) * 2u + (uint32_t(t) * uint32_t(a.ldx) + uint32_t(k)) * 2u
                                : kOOB;
  };
  // weight pieces: row p / 4, quarter p % 4
  auto w_off = [&](int lr, int kbyte) -> uint32_t {
    const int row = n0 + lr;
    return row < N && kbyte < int(row_bytes) ? uint32_t(row) * row_bytes + uint32_t(kbyte) : kOOB;
  };
  struct Stage {
    int4 av[APT];
    int4 bv[2];
  };
  auto load = [&](int kc, Stage& st) {
    const int k0 = kc * kKC;
#pragma unroll
    for (int i = 0; i < APT; ++i) st.av[i] = buf_load16(ra, kc < nk ? a_off(i, k0) : kOOB);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int p = tid + kBlock * i;
      st.bv[i] = buf_load16(rw, kc < nk ? w_off(p >> 2, (k0 + 8 * (p & 3)) * 2) : kOOB);
    }
  };
  auto commit = [&](int buf, const Stage& st) {
#pragma unroll
    for (int i = 0; i < APT; ++i) {
      const int p = tid + kBlock * i;
      const int plane = p / (4 * TM), row = (p >> 2) & (TM - 1), qu = p & 3;
      *reinterpret_cast<int4*>(&sm.a[buf][plane][lds_q(row, qu)]) = st.av[i];
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int p = tid + kBlock * i;
      *reinterpret_cast<int4*>(&sm.b[buf][lds_q(p >> 2, p & 3)]) = st.bv[i];
    }
  };

  // three chunks in flight in registers: chunk c is loaded while chunk c - 3 is computed and
  // committed to LDS after chunk c - 1 has been computed
  Stage s0, s1, s2;
  load(0, s0);
  load(1, s1);
  load(2, s2);

  // ---- inverse RMS of the tile's tokens: thread t sums half of token t / 2
  {
    const int row = tid >> 1, half = tid & 1, t = m0 + row;
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(a.ssq, uint32_t(T) * uint32_t(a.n_ssq) * 4u);
    float v = 0.0f;
    for (int j0 = 0; j0 < a.n_ssq; j0 += 16) {
      float tv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int j = j0 + 2 * u + half;
        tv[u] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                              rq, int((t < T && j < a.n_ssq) ? (uint32_t(t) * uint32_t(a.n_ssq) + uint32_t(j)) * 4u : kOOB), 0, 0));
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) v += tv[u];
    }
    v += __shfl_xor(v, 1, kWave);
    if (half == 0 && row < TM) sm.rs[row] = rsqrtf(v * a.inv_d + a.eps);
  }

  commit(0, s0);
  __syncthreads();

  f32x4 acc[MT][4];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  auto step = [&](int kc, Stage& mine, const Stage& next) {
    const int buf = kc & 1;
    load(kc + 3, mine);                                 // chunk kc was committed already
    bf16x8 bw[4];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
      bw[nt] = *reinterpret_cast<const bf16x8*>(&sm.b[buf][lds_q(wn * 64 + nt * 16 + r, q)]);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
      const int ar = lds_q(wm * (TM / 2) + mt * 16 + r, q);
      const bf16x8 ahi = *reinterpret_cast<const bf16x8*>(&sm.a[buf][0][ar]);
      const bf16x8 alo = *reinterpret_cast<const bf16x8*>(&sm.a[buf][1][ar]);
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bw[nt], acc[mt][nt], 0, 0, 0);
        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bw[nt], acc[mt][nt], 0, 0, 0);
      }
    }
    if (kc + 1 < nk) commit(buf ^ 1, next);
    __syncthreads();
  };
  for (int kc = 0; kc < nk; kc += 3) {
    step(kc, s0, s1);
    if (kc + 1 < nk) step(kc + 1, s1, s2);
    if (kc + 2 < nk) step(kc + 2, s2, s0);
  }

  // epilogue: lane (r, q) holds tokens 4 q + i of each token tile for row r of each row tile
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tl = wm * (TM / 2) + mt * 16 + 4 * q + i;
      const int t = m0 + tl;
      if (t >= T) continue;
      const float rb = sm.rs[tl];
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) {
        const int n = n0 + wn * 64 + nt * 16 + r;
        if (n < N) a.y[size_t(t) * a.ldy + n] = acc[mt][nt][i] * rb;
      }
    }
}

// Operand of the LM head: x * gamma as hi/lo planes and per-64-element sums of squares of x.
// Thread = four consecutive elements of token blockIdx.y; 16 lanes cover one 64-element block.
__global__ __launch_bounds__(kBlock) void pf_prep_kernel(const float* __restrict__ x, int D,
                                                         const uint16_t* __restrict__ gamma,
                                                         uint16_t* xo, size_t plane, int ldxo,
                                                         float* ssq, int n_ssq) {
  const int t = blockIdx.y, i0 = (blockIdx.x * kBlock + threadIdx.x) * 4;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(x + size_t(t) * D, uint32_t(D) * 4u);
  const float4 v = __builtin_bit_cast(float4, buf_load16(rx, i0 < D ? uint32_t(i0) * 4u : kOOB));
  float ss = fmaf(v.x, v.x, fmaf(v.y, v.y, fmaf(v.z, v.z, v.w * v.w)));
  if (i0 < D) {
    const float e[4] = {v.x * bf16_to_f32(gamma[i0]), v.y * bf16_to_f32(gamma[i0 + 1]),
                        v.z * bf16_to_f32(gamma[i0 + 2]), v.w * bf16_to_f32(gamma[i0 + 3])};
    uint32_t hi[2], lo[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const uint16_t h0 = f32_to_bf16(e[2 * k]), h1 = f32_to_bf16(e[2 * k + 1]);
      hi[k] = uint32_t(h0) | (uint32_t(h1) << 16);
      lo[k] = uint32_t(f32_to_bf16(e[2 * k] - bf16_to_f32(h0))) |
              (uint32_t(f32_to_bf16(e[2 * k + 1] - bf16_to_f32(h1))) << 16);
    }
    uint16_t* row = xo + size_t(t) * ldxo + i0;          // 8-byte aligned: ldxo % 64 == 0
    *reinterpret_cast<uint2*>(row) = make_uint2(hi[0], hi[1]);
    *reinterpret_cast<uint2*>(row + plane) = make_uint2(lo[0], lo[1]);
  } else if (i0 < (D + kKC - 1) / kKC * kKC) {           // the last chunk's padding (finite)
    uint16_t* row = xo + size_t(t) * ldxo + i0;
    *reinterpret_cast<uint2*>(row) = make_uint2(0, 0);
    *reinterpret_cast<uint2*>(row + plane) = make_uint2(0, 0);
  }
  ss = row16_sum(ss);
  if ((threadIdx.x & 15) == 0 && i0 < D) ssq[size_t(t) * n_ssq + i0 / kSsqBlk] = ss;
}

// RoPE of the T tokens' q and k at positions pos0 + t. q (scaled by log2(e) / sqrt(d_h)) goes to
// the attention operand as hi/lo planes [2][m_q][T][d_h]; k and v are rounded to BF16 and
// written to the cache rows pos0 + t of their retained groups. An item is four consecutive
// rotation pairs (q, k) or four consecutive v elements.
__device__ __forceinline__ void store_bf16x4(uint16_t* dst, const float (&v)[4]) {
  const uint32_t a = uint32_t(f32_to_bf16(v[0])) | (uint32_t(f32_to_bf16(v[1])) << 16);
  const uint32_t b = uint32_t(f32_to_bf16(v[2])) | (uint32_t(f32_to_bf16(v[3])) << 16);
  *reinterpret_cast<uint2*>(dst) = make_uint2(a, b);
}

// One item per thread, a token's items over blockIdx.y (a workgroup per token walked all of them, with
// one wait per K split: 14.1 us at 16 tokens of the 8B layer, 4.2 now).
__global__ __launch_bounds__(kBlock) void pf_rope_kernel(PfRopeArgs a) {
  const int t = blockIdx.x;
  const int dh = a.dh, half = dh / 2, h4 = half / 4;
  const uint32_t row = uint32_t(t) * uint32_t(a.ld_qkv), stride = uint32_t(a.split_stride) * 4u;
  const __amdgpu_buffer_rsrc_t rq =
      make_rsrc(a.qkv, uint32_t(a.ks - 1) * stride + uint32_t(a.T) * uint32_t(a.ld_qkv) * 4u);
  const int pos = a.pos0 + t;
  const float* cs = a.rope_cos + size_t(pos) * half;
  const float* sn = a.rope_sin + size_t(pos) * half;
  const float qscale = kLog2e * rsqrtf(float(dh));
  const int nq = a.m_q * h4, nk = a.m_kv * h4, nv = a.m_kv * (dh / 4);
  const int it = blockIdx.y * kBlock + threadIdx.x;
  if (it < nq + nk + nv) {
    if (it < nq + nk) {
      const bool is_q = it < nq;
      const int u = is_q ? it : it - nq;
      const int h = u / h4, i = 4 * (u % h4);
      const uint32_t at = row + uint32_t((is_q ? h : a.m_q + h) * dh + i);
      const uint32_t off[2] = {at * 4u, (at + uint32_t(half)) * 4u};
      const float4 c = *reinterpret_cast<const float4*>(cs + i);
      const float4 sv = *reinterpret_cast<const float4*>(sn + i);
      float4 x[2] = {__builtin_bit_cast(float4, buf_load16(rq, off[0])), __builtin_bit_cast(float4, buf_load16(rq, off[1]))};
      add_splits(rq, off, stride, 1, a.ks, x);
      const float4 x1 = x[0], x2 = x[1];
      const float sc = is_q ? qscale : 1.0f;
      const float y1[4] = {(x1.x * c.x - x2.x * sv.x) * sc, (x1.y * c.y - x2.y * sv.y) * sc,
                           (x1.z * c.z - x2.z * sv.z) * sc, (x1.w * c.w - x2.w * sv.w) * sc};
      const float y2[4] = {(x2.x * c.x + x1.x * sv.x) * sc, (x2.y * c.y + x1.y * sv.y) * sc,
                           (x2.z * c.z + x1.z * sv.z) * sc, (x2.w * c.w + x1.w * sv.w) * sc};
      if (is_q) {
        uint16_t* qo = a.q_out + (size_t(h) * a.T_ld + t) * dh;
        float l1[4], l2[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          l1[e] = y1[e] - bf16_to_f32(f32_to_bf16(y1[e]));
          l2[e] = y2[e] - bf16_to_f32(f32_to_bf16(y2[e]));
        }
        store_bf16x4(qo + i, y1);
        store_bf16x4(qo + i + half, y2);
        store_bf16x4(qo + a.q_plane + i, l1);
        store_bf16x4(qo + a.q_plane + i + half, l2);
      } else {
        uint16_t* kc = a.kc + (size_t(a.kv_idx[h]) * a.S + pos) * dh;
        store_bf16x4(kc + i, y1);
        store_bf16x4(kc + i + half, y2);
      }
    } else {
      const int u = it - nq - nk;
      const int j = u / (dh / 4), e = 4 * (u % (dh / 4));
      const uint32_t off[1] = {(row + uint32_t((a.m_q + a.m_kv + j) * dh + e)) * 4u};
      float4 v[1] = {__builtin_bit_cast(float4, buf_load16(rq, off[0]))};
      add_splits(rq, off, stride, 1, a.ks, v);
      const float w[4] = {v[0].x, v[0].y, v[0].z, v[0].w};
      store_bf16x4(a.vc + (size_t(a.kv_idx[j]) * a.S + pos) * dh + e, w);
    }
  }
}

}  // namespace

hipError_t launch_pf_head(const PfHeadArgs& a, hipStream_t s) {
  if (a.T < 1 || a.N < 1 || a.K < 1 || a.K % 8 != 0 || a.ldx % 64 != 0 || a.ldx < a.K) return hipErrorInvalidValue;
  // 128-token tiles halve the weight re-reads; smaller ones when that leaves CUs idle
  const int gx = (a.N + kTN - 1) / kTN;
  if (long(gx) * ((a.T + kTMax - 1) / kTMax) >= kPfMinTiles)
    hipLaunchKernelGGL((pf_head_kernel<kTMax>), dim3(gx, (a.T + kTMax - 1) / kTMax), dim3(kBlock), 0, s, a);
  else
    hipLaunchKernelGGL((pf_head_kernel<kTMax / 2>), dim3(gx, (a.T + kTMax / 2 - 1) / (kTMax / 2)), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_pf_prep(const float* x, int D, int T, const uint16_t* gamma, uint16_t* xo,
                          size_t plane, int ldxo, float* ssq, hipStream_t s) {
  if (D % 16 != 0 || T < 1 || ldxo % 4 != 0 || plane % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pf_prep_kernel, dim3((D + 4 * kBlock - 1) / (4 * kBlock), T), dim3(kBlock), 0, s, x, D,
                     gamma, xo, plane, ldxo, ssq, (D + kSsqBlk - 1) / kSsqBlk);
  return hipGetLastError();
}

hipError_t launch_pf_rope(const PfRopeArgs& a, hipStream_t s) {
  if (a.T < 1 || a.m_kv < 1) return hipSuccess;
  // the sources are addressed by 31-bit byte offsets
  if (a.ks < 1 || (size_t(a.ks - 1) * (a.ks > 1 ? a.split_stride : 0) + size_t(a.T) * a.ld_qkv) * 4 >= size_t(kOOB))
    return hipErrorInvalidValue;
  const int items = a.m_q * (a.dh / 8) + a.m_kv * (a.dh / 8 + a.dh / 4);
  hipLaunchKernelGGL(pf_rope_kernel, dim3(a.T, (items + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

int pf_ssq_block() { return kSsqBlk; }

size_t pf_split_buffer_floats(int max_prefill, int n_max) {
  // splits pay while the tiles leave CUs idle, i.e. up to a few hundred tokens; past the cap the
  // launch takes fewer splits
  const long rows = std::min<long>(long(kMaxKSplit) * std::max(max_prefill, 0), kSplitRowCap);
  return size_t(rows) * size_t(std::max(n_max, 0));
}

}  // namespace tasp
