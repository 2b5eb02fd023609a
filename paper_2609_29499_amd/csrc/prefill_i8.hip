// Prefill projections over INT8 panels and over the groupwise store on the INT8 matrix cores:
// C[t][n] = sum_k A[t][k] P[n][k] with v_mfma_i32_32x32x32_i8 and exact int32 accumulation.
//
// Operands. A token's activations are carried as 24-bit fixed point under one power-of-two scale
// per token, in three signed base-256 digits (q = 65536 d2 + 256 d1 + d0, each digit in -128..127),
// written by pf_quant_kernel; the INT8 panel bytes are multiplied as they are, without widening.
// Per (token, row) the three digit sums are exact integers and are joined in float32 in the
// epilogue, so the only rounding before it is the digit grid: half a step of 2^-22 to 2^-23 of
// the token's largest activation. Against an operand pair of hi and lo BF16 (about 2^-19 of each
// activation, on the BF16 matrix cores) the error of a random token is lower (rms 2^-22
// of the token's rms for a largest value of 4 to 5 rms), and the issued matrix work is three
// INT8 passes instead of two BF16 passes at half the rate.
//
// Rows with outliers. Beside a value far above the rest one scale leaves the rest fewer bits than a
// hi/lo pair does (with one value 1000 times the rms of 4096 others, an output that does not use that
// column is off by 7e-5 of itself, with a pair by 2.4e-6). pf_quant_kernel compares the two errors of
// every row (its comment has the rule) and carries a row for which digits are the worse form as a
// pair. A tile with such rows multiplies its digit rows as always and then goes over K again with the
// pairs, up to 64 of them gathered at a time, on the BF16 matrix cores with the panel bytes widened; a
// tile of pairs alone skips the digits. The waves share the panel rows of that pass, not the tokens, so
// that each widens its own only.
//
// Row layout of an operand: 4 ld bytes. Digits: ld bytes of d2, ld of d1, ld of d0. A pair: ld BF16 of
// hi, ld of lo. ld is a multiple of the 128-byte chunk and either form is zero from K to the end of its
// last chunk, so panel bytes past the end of a row multiply zeros. A row takes the 4 ld bytes of the
// float32 row it came from: the O and down inputs are written in float32 and turned into their form in
// place. The tokens' scales (float32, times the inverse RMS for a normed input) are an array of their
// own, the sign bit telling a pair from digits.
//
// Tiling. Workgroups of TM tokens x TN rows (gate/up: TN / 2 channels, gate and up rows of a
// channel in one wave); each wave holds its outputs, times three digits, in registers. K advances
// in chunks of 128, one memory line per row: digit rows and panel rows go from memory straight
// into two LDS stages (buffer loads with an LDS destination, 16-byte pieces XOR-swizzled by row on
// the memory side), the next chunk in flight while one is multiplied, one barrier per chunk. Where few
// tiles leave a CU one workgroup, its waves deal the chunks among groups (KW below).
//
// Groupwise store (shared-store plans). A chunk of 128 columns is one scale group, so the three digit
// sums of a chunk are exact integers that meet one BF16 scale: 256 d2 + d1 is formed in one int32
// accumulator (shifted between the two passes), converted and added to a float32 sum with the
// scale, then d0 (five vector operations per output and chunk next to 48 matrix operations per 64
// outputs and lane). Rows come through the plan's row map; a column-mapped operand is laid out in
// the store's own chunks, those with any retained column (listed by the operand's writer), dropped
// columns zero. It replaced four passes of hi/lo weights times hi/lo activations on the BF16 matrix
// cores: one 8B layer at 1000 tokens 1005 -> 586 us.
//
// What bounds it. Large calls: the matrix cores at the clock they leave. The 2 x 16384 x 8192 gate/up
// projection at 2048 tokens (1.29 ms; hi/lo operands on the BF16 matrix cores took 2.24) keeps them busy
// 64 % of its cycles at a clock of 1.80 GHz, of 2.4 nominal; one round of 128 x 256 tiles (8B gate/up
// at 512 tokens) 53 % at 2.01 GHz. The LDS serves reads for 41 % of the cycles, half of that in conflicts
// that the swizzle leaves. Chunks are whole 128-byte lines, and a wave's tile is 32 x 128 rather than
// 64 x 64, which needs fewer fragment reads per product. Short prompts: the latency of a chunk (KW below).
#include <algorithm>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "split_sums.hpp"

namespace tasp {
namespace {

typedef int __attribute__((ext_vector_type(4))) i32x4;
typedef int __attribute__((ext_vector_type(16))) i32x16;
typedef float __attribute__((ext_vector_type(16))) f32x16;
// four floats of a caller's array, which is only 4-byte aligned
typedef float __attribute__((ext_vector_type(4), aligned(4))) f32x4u;

constexpr int kKC = 128;                // k per chunk: one 128-byte line of a digit or panel row
constexpr int kXcds = 8;
constexpr int kNumCu = 256;
constexpr int kGroupM = 4;              // token tiles walked together by one XCD's workgroups

// No vector memory or LDS operation of this wave outstanding, and none moved across by the compiler:
// its loads into a stage have landed and its reads of one are done. The builtin wait and barrier alone
// order neither: the compiler may sink the last reads' wait, with the products that need it, past them.
__device__ __forceinline__ void stage_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(7 << 4);                   // vmcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");
}

// LDS slot of 16-byte piece p of row `row` (rows of kKC bytes): any 8 consecutive rows read at one
// piece meet distinct 16-byte columns
__device__ __forceinline__ int slot(int row, int p) { return p ^ (row & 7); }

// eight INT8 values (exact in BF16) as a matrix operand, and an operand of the LDS
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
__device__ __forceinline__ uint32_t widen2(uint32_t w, int i) {
  return __builtin_amdgcn_perm(__float_as_uint(float(int8_t(w >> (8 * i + 8)))), __float_as_uint(float(int8_t(w >> (8 * i)))),
                               0x07060302u);
}
__device__ __forceinline__ bf16x8 widen8(const uint2& w) {
  return __builtin_bit_cast(bf16x8, make_int4(int(widen2(w.x, 0)), int(widen2(w.x, 2)), int(widen2(w.y, 0)), int(widen2(w.y, 2))));
}

// the three digit sums of one output, joined in float32
__device__ __forceinline__ float join(int s2, int s1, int s0) {
  return fmaf(float(s2), 65536.0f, fmaf(float(s1), 256.0f, float(s0)));
}

// Workgroup id -> (n tile, m tile, split). Ids go round-robin over the XCDs; each XCD takes a
// contiguous run of an order that walks kGroupM token tiles together, so that the workgroups an
// XCD holds at one time share digit and panel rows in its L2. The token tile moves on by one in every
// n tile: an XCD's shader engines take its workgroups in turn, and without the shift all tiles of the
// same tokens, the slow ones if these have outlier rows, fell to one engine.
__device__ __forceinline__ void tile_of(int id, int total, int gx, int gy, int& bx, int& by, int& bz) {
  const int x = id % kXcds, j = id / kXcds;
  const int o = x * (total / kXcds) + min(x, total % kXcds) + j;
  bz = o / (gx * gy);
  const int rem = o - bz * (gx * gy);
  const int grp = rem / (kGroupM * gx);
  const int gm = min(kGroupM, gy - grp * kGroupM);
  const int in = rem - grp * (kGroupM * gx);
  bx = in / gm;
  by = grp * kGroupM + (in + bx) % gm;
}

// NT tiles of 32 tokens x 32 rows per wave; WGM x WGN waves; WAVES: per SIMD; SH: groupwise store.
// KW > 1: KW groups of WGM x WGN waves share the tile, group kw multiplying chunks kw, kw + KW, .. from
// stages of its own (without a barrier where a group is one wave), and their digit sums meet in LDS.
// With one workgroup per CU a chunk costs its latency and not its products; KW chunks are in flight
// instead of one (8B layer: gate/up at 16 tokens 26.5 us on 32 x 128 tiles, 15 on 32 x 64 with four
// groups; at 128 tokens 33 us on 64 x 128 tiles, 29 with two groups; down at 512 tokens 61 and 54).
template <int MODE, int NT, int WGM, int WGN, int KW, int WAVES, bool SH>
__global__ __launch_bounds__(64 * WGM * WGN * KW, WAVES) void pf_i8_kernel(PfI8Args a, int gx, int gy) {
  constexpr bool GU = (MODE == MM_GATEUP);
  constexpr int HN = 16 * NT;                           // gate/up: channels per wave
  constexpr int TM = 32 * WGM, TN = 32 * NT * WGN, NW = WGM * WGN;
  constexpr int EC = 16 / KW;                           // outputs per row tile and lane
  constexpr int kUnrollK = KW > 1 ? 4 : 2;              // steps of 32 columns
  constexpr int RPL = 1024 / kKC, LPR = kKC / 16;       // rows per 1 KiB load, lanes per row
  constexpr int APER = 3 * TM / RPL / NW, BPER = TN / RPL / NW;
  static_assert(APER * RPL * NW == 3 * TM && BPER * RPL * NW == TN, "even share of the loads");
  static_assert(HN % (RPL * NW) == 0, "a panel load of a wave lies in gate or in up rows, the same for every wave");
  static_assert(TM <= 64 * NW, "one token scale per thread");
  static_assert(KW == 1 || KW == 2 || KW == 4, "the groups share a lane's 16 outputs of a row tile by fours");
  // A group's stage: the digit planes' token rows of kKC bytes, then the panel rows. Each stage is one
  // flat array indexed by one sum, so that the compiler tells the two apart (through members of nested
  // objects it loses track and makes a read of one wait for the loads into the other).
  constexpr int SA = 3 * TM * kKC, SB = TN * kKC, SBYTES = SA + SB;
  typedef uint8_t Stage[KW * SBYTES];
  __shared__ __attribute__((aligned(16))) Stage st0;
  __shared__ __attribute__((aligned(16))) Stage st1;

  const int tid = threadIdx.x, lane = tid & 63, wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kw = KW > 1 ? wave_id / NW : 0, wave = wave_id - kw * NW;   // group, wave of it
  const int r = lane & 31, hi = lane >> 5;
  const int wm = wave / WGN, wn = wave % WGN;
  const int T = a.T, N = a.N;
  int bx, by, bz;
  tile_of(blockIdx.x, gridDim.x, gx, gy, bx, by, bz);
  const int m0 = by * TM, n0 = bx * (GU ? TN / 2 : TN);
  const int nk_all = (a.K + kKC - 1) / kKC;
  const int kc0 = int((long(bz) * nk_all) / a.ks);
  const int nk = int((long(bz + 1) * nk_all) / a.ks) - kc0;

  const uint32_t xrow = 4u * uint32_t(a.ldx);           // bytes of an operand row
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.x, uint32_t(T) * xrow);
  // the tile's token scales: one per thread for the epilogue, and all of them in every wave for their
  // signs (first of all loads, so that waiting for them does not wait for the chunks)
  const __amdgpu_buffer_rsrc_t rt = make_rsrc(a.tok, uint32_t(T) * 4u);
  auto token_scale = [&](int t) {                       // (zero past the tile and past the last token)
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rt, int(t < TM && m0 + t < T ? 4u * uint32_t(m0 + t) : kOOB), 0, 0));
  };
  const float tscale = token_scale(tid);
  const float tsign[2] = {token_scale(lane), TM > 64 ? token_scale(lane + 64) : 0.0f};
  const uint32_t ldw = SH ? uint32_t(a.sv.ld) : uint32_t(a.ld);
  const uint32_t w_bytes = (SH ? uint32_t(a.sv.store_rows) : uint32_t(N)) * ldw;
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(SH ? a.sv.w : a.w, !SH && GU ? a.w2_off + w_bytes : w_bytes);
  const __amdgpu_buffer_rsrc_t rw2 = make_rsrc(SH && GU ? a.sv.w2 : nullptr, SH && GU ? w_bytes : 0u);
  // store row of panel row `row` (-1 past the panel)
  auto panel_row = [&](int row) { return row >= N ? -1 : (SH && a.sv.rows ? a.sv.rows[row] : row); };

  // this lane's share of a chunk: a load covers RPL rows, LPR lanes each; the wave's loads are
  // digit rows RPL (wave + NW j) .. (plane-major), then panel rows RPL (wave + NW j) ..
  uint32_t abase[APER], bbase[BPER];
  // panel load j: gate or up rows
  auto up_load = [](int j) { return GU && (RPL * NW * j) % (2 * HN) >= HN; };
#pragma unroll
  for (int j = 0; j < APER; ++j) {
    const int i = wave + NW * j, plane = i / (TM / RPL);
    const int lr = (i % (TM / RPL)) * RPL + lane / LPR, t = m0 + lr;
    abase[j] = t < T ? uint32_t(t) * xrow + uint32_t(plane) * uint32_t(a.ldx) + 16u * slot(lr, lane % LPR) : kOOB;
  }
#pragma unroll
  for (int j = 0; j < BPER; ++j) {
    const int lr = (wave + NW * j) * RPL + lane / LPR;
    const int row = panel_row(GU ? n0 + HN * (lr / (2 * HN)) + lr % HN : n0 + lr);
    bbase[j] = row >= 0 ? (!SH && up_load(j) ? a.w2_off : 0u) + uint32_t(row) * ldw + 16u * slot(lr, lane % LPR) : kOOB;
  }
  // Chunks past the last reload it (into a stage that is not read again), so that every step
  // issues alike. A row of a per-row panel may end inside its last chunk: the bytes loaded past it
  // are the next row's, or of the sections behind the panels, and meet zero digits. Store rows are
  // whole chunks; with a column map the operand's chunk kc is store chunk a.chunks[kc].
  const bool mapped = SH && a.sv.cols != nullptr;
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(a.chunks, mapped ? uint32_t(nk_all) * 4u : 0u);
  auto clamp_chunk = [&](int kc) { return kc0 + max(min(kw + KW * kc, nk - 1), 0); };
  auto list_entry = [&](int kc) {                       // loaded one step before it is used
    return mapped ? __builtin_amdgcn_raw_buffer_load_b32(rl, 4 * clamp_chunk(kc), 0, 0) : 0u;
  };
  auto store_chunk = [&](int kc, uint32_t entry) {
    return mapped ? int(__builtin_amdgcn_readfirstlane(int(entry))) : clamp_chunk(kc);
  };
  auto issue_panel = [&](int wk, Stage& S) {
#pragma unroll
    for (int j = 0; j < BPER; ++j) {
      const __amdgpu_buffer_rsrc_t rj = SH && up_load(j) ? rw2 : rw;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rj, static_cast<void*>(&S[kw * SBYTES + SA + (wave + NW * j) * 1024]), 16, int(bbase[j]), wk, 0, 0);
    }
  };
  auto issue = [&](int kc, int wc, Stage& S) {
    const int k0 = clamp_chunk(kc) * kKC;
#pragma unroll
    for (int j = 0; j < APER; ++j)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, static_cast<void*>(&S[kw * SBYTES + (wave + NW * j) * 1024]), 16, int(abase[j]), k0, 0, 0);
    issue_panel(SH ? wc * kKC : k0, S);
  };

  // panel rows of the lane's outputs, and (groupwise store) the byte offsets of their scales
  int col[NT];
  uint32_t gbase[SH ? NT : 1];
  const uint32_t sgroups = ldw / 128u;
  const __amdgpu_buffer_rsrc_t rg = make_rsrc(SH ? a.sv.gs : nullptr, SH ? uint32_t(a.sv.store_rows) * sgroups * 2u : 0u);
  const __amdgpu_buffer_rsrc_t rg2 = make_rsrc(SH && GU ? a.sv.gs2 : nullptr,
                                               SH && GU ? uint32_t(a.sv.store_rows) * sgroups * 2u : 0u);
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    col[nt] = GU ? n0 + HN * wn + 32 * (nt % (NT / 2)) + r : n0 + (wn * NT + nt) * 32 + r;
    if constexpr (SH) {
      const int row = panel_row(col[nt]);
      gbase[nt] = row >= 0 ? uint32_t(row) * sgroups * 2u : kOOB;
    }
  }
  struct Scales {
    uint32_t s[SH ? NT : 1];
  };
  auto load_scales = [&](int wc) {
    Scales v{};
    if constexpr (SH) {
      const int off = 2 * wc;
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const __amdgpu_buffer_rsrc_t rn = GU && nt >= NT / 2 ? rg2 : rg;
        v.s[nt] = __builtin_amdgcn_raw_buffer_load_b16(rn, int(gbase[nt]), off, 0);
      }
    }
    return v;
  };

  const int first = store_chunk(0, list_entry(0));
  uint32_t entry = list_entry(1);
  Scales sc0 = load_scales(first), sc1{};
  issue(0, first, st0);

  // per-row panels: the digit sums over all of K; groupwise store: the scaled float32 sum, and the
  // digit sums of one chunk (one scale group) at a time
  i32x16 acc[SH ? 1 : 3][SH ? 1 : NT];
  f32x16 facc[NT];
#pragma unroll
  for (int d = 0; d < (SH ? 1 : 3); ++d)
#pragma unroll
    for (int j = 0; j < (SH ? 1 : NT); ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[d][j][e] = 0;
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int e = 0; e < 16; ++e) facc[j][e] = 0.0f;

  auto frag_a = [&](const Stage& S, int d, int ks) {   // (tile rows differ from r by multiples of 32)
    return *reinterpret_cast<const i32x4*>(&S[kw * SBYTES + d * TM * kKC + (wm * 32 + r) * kKC + 16 * slot(r, 2 * ks + hi)]);
  };
  auto frag_b = [&](const Stage& S, int nt, int ks) {
    return *reinterpret_cast<const i32x4*>(&S[kw * SBYTES + SA + ((wn * NT + nt) * 32 + r) * kKC + 16 * slot(r, 2 * ks + hi)]);
  };
  auto compute = [&](const Stage& S, const Scales& sv) {
    if constexpr (!SH) {
#pragma unroll kUnrollK
      for (int ks = 0; ks < kKC / 32; ++ks) {
        i32x4 bf[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) bf[nt] = frag_b(S, nt, ks);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
          const i32x4 af = frag_a(S, d, ks);
#pragma unroll
          for (int nt = 0; nt < NT; ++nt)
            acc[d][nt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af, bf[nt], acc[d][nt], 0, 0, 0);
        }
      }
    } else {
      // |256 d2 + d1 sums| <= 128 * 127 * 32768 < 2^29.0 and |d0 sum| <= 2^21: both exact in int32
      // two row tiles at a time, so that their fragments and sums fit the registers
#pragma unroll
      for (int h = 0; h < NT; h += 2) {
        __builtin_amdgcn_sched_barrier(0);              // (overlapping the pairs spills)
        i32x4 bf[kKC / 32][2];
#pragma unroll
        for (int ks = 0; ks < kKC / 32; ++ks)
#pragma unroll
          for (int j = 0; j < 2; ++j) bf[ks][j] = frag_b(S, h + j, ks);
        i32x16 u[2];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) u[j][e] = d == 1 ? u[j][e] << 8 : 0;
#pragma unroll
          for (int ks = 0; ks < kKC / 32; ++ks) {
            const i32x4 af = frag_a(S, d, ks);
#pragma unroll
            for (int j = 0; j < 2; ++j) u[j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af, bf[ks][j], u[j], 0, 0, 0);
          }
          if (d == 0) continue;
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float s = bf16_to_f32(uint16_t(sv.s[h + j])) * (d == 1 ? 256.0f : 1.0f);
#pragma unroll
            for (int e = 0; e < 16; ++e) facc[h + j][e] = fmaf(float(u[j][e]), s, facc[h + j][e]);
          }
        }
      }
    }
  };
  // chunk kc sits in stage kc % 2: wait for this wave's loads of it and its reads of the other stage,
  // meet the other waves that share the stages (one wave's group has none), load the next chunk into
  // the other stage, multiply
  auto stage_ready = [&] {
    stage_done();
    if constexpr (NW > 1) {
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
  };
  auto step = [&](int kc, const Stage& cur, Stage& nxt, const Scales& sv, Scales& sn) {
    stage_ready();
    const int wc = store_chunk(kc + 1, entry);
    entry = list_entry(kc + 2);
    if constexpr (SH) sn = load_scales(wc);
    issue(kc + 1, wc, nxt);
    if (KW == 1 || kw + KW * kc < nk) compute(cur, sv);
  };
  const int nkw = (nk + KW - 1) / KW;                   // steps, the same for every group
  // the tile's tokens whose rows are pairs
  const unsigned long long pair_tok[2] = {__ballot(__float_as_int(tsign[0]) < 0), __ballot(__float_as_int(tsign[1]) < 0)};
  const int n_pair = __popcll(pair_tok[0]) + __popcll(pair_tok[1]);
  if (n_pair < min(TM, T - m0)) {
    for (int kc = 0; kc < nkw; kc += 2) {
      step(kc, st0, st1, sc0, sc1);
      if (kc + 1 < nkw) step(kc + 1, st1, st0, sc1, sc0);
    }
  }
  stage_done();
  __syncthreads();                                      // every wave is done with the stages
  // (KW > 1) the groups' sums: group kw adds up outputs EC kw .. + EC - 1 of every lane and row tile, the
  // others leave theirs in LDS (32 KiB per digit, two in st0, one in st1).
  constexpr int ND = SH ? 1 : 3, QG = 4 / KW;           // digits, groups of four outputs per wave group
  constexpr int QS = KW == 2 ? 2 : 4;                   // groups of four a wave leaves (KW 4: its own unused)
  constexpr size_t kSumBytes = KW > 1 ? size_t(KW) * NW * NT * QS * kWave * 16 : 0;   // of one digit
  static_assert((ND > 1 ? 2 : 1) * kSumBytes <= sizeof(st0) && kSumBytes <= sizeof(st1), "the sums fit the stages");
  auto sums = [&](int d, int k, int nt, int g) -> i32x4* {
    char* base = d < 2 ? reinterpret_cast<char*>(&st0) + size_t(d) * kSumBytes : reinterpret_cast<char*>(&st1);
    return reinterpret_cast<i32x4*>(base) + (((k * NW + wave) * NT + nt) * QS + g % QS) * kWave + lane;
  };
  auto bits = [&](int d, int nt, int e) {
    if constexpr (SH) return __float_as_int(facc[nt][e]);
    else return int(acc[d][nt][e]);
  };
  if constexpr (KW > 1) {
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          if (g / QG != kw) *sums(d, kw, nt, g) = i32x4{bits(d, nt, 4 * g), bits(d, nt, 4 * g + 1), bits(d, nt, 4 * g + 2), bits(d, nt, 4 * g + 3)};
    __syncthreads();
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int g = 0; g < QG; ++g) {
          i32x4 v[KW];
#pragma unroll
          for (int k = 0; k < KW; ++k) {
            v[k] = i32x4{bits(d, nt, EC * k + 4 * g), bits(d, nt, EC * k + 4 * g + 1), bits(d, nt, EC * k + 4 * g + 2), bits(d, nt, EC * k + 4 * g + 3)};
            if (k != kw) v[k] = *sums(d, k, nt, QG * kw + g);
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if constexpr (SH) {
              float f = __int_as_float(v[0][i]);
#pragma unroll
              for (int k = 1; k < KW; ++k) f += __int_as_float(v[k][i]);
              facc[nt][4 * g + i] = f;
            } else {
              int q = v[0][i];
#pragma unroll
              for (int k = 1; k < KW; ++k) q += v[k][i];
              acc[d][nt][4 * g + i] = q;
            }
          }
        }
  }
  if constexpr (!SH) {
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < EC; ++e) facc[nt][e] = join(acc[0][nt][e], acc[1][nt][e], acc[2][nt][e]);
  }
  auto token = [&](int e) { return wm * 32 + 8 * ((EC * kw + e) >> 2) + 4 * hi + (e & 3); };

  // ---- the pairs, MB of them at a time: MB x TN outputs of which a wave has MB x 32 PT (its group's
  // chunks), 64 columns of K a step. These are 128 bytes of hi and of lo of a token, where the digit planes
  // were, and one half of the panel rows' chunk.
  if (n_pair > 0) {
    // (the lane anew, so that nothing derived from it here is kept in registers through the loop above)
    int plane_id = lane;
    asm volatile("" : "+v"(plane_id));
    const int lane = plane_id, r = lane & 31, hi = lane >> 5;
    constexpr int MB = TM == 32 ? 32 : 64, MT = MB / 32, PT = NT / WGM, PPER = 2 * MB / RPL / NW;
    static_assert(PT * WGM == NT && PPER * RPL * NW == 2 * MB, "even share of the rows and loads");
    static_assert(MB * 256 + TM * 4 <= SA && KW * MB * TN * 4 <= int(sizeof(st0)), "list and sums fit the stages");
    int* const list = reinterpret_cast<int*>(reinterpret_cast<char*>(&st0) + MB * 256);   // tokens that are pairs
    float* const out = reinterpret_cast<float*>(&st0);                                    // [KW][MB][TN] sums
    // the wave's 32 tokens: which are pairs, and the pairs before them
    const uint32_t own = uint32_t(pair_tok[wm >> 1] >> (32 * (wm & 1)));
    const int before = (wm >> 1 ? __popcll(pair_tok[0]) : 0) + (wm & 1 ? __popc(uint32_t(pair_tok[wm >> 1])) : 0);
    // byte offset of the scales of the lane's rows in the wave's row tiles; gate or up of a row tile
    uint32_t pgroup[SH ? PT : 1];
    auto pair_row = [&](int j) { return (wave * PT + j) * 32; };       // its first row in the tile
    if constexpr (SH) {
#pragma unroll
      for (int j = 0; j < PT; ++j) {
        const int lr = pair_row(j) + r, row = panel_row(GU ? n0 + HN * (lr / (2 * HN)) + lr % HN : n0 + lr);
        pgroup[j] = row >= 0 ? uint32_t(row) * sgroups * 2u : kOOB;
      }
    }
    auto pair_scales = [&](int wc) {
      Scales v{};
      if constexpr (SH) {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
          const __amdgpu_buffer_rsrc_t rn = GU && pair_row(j) % (2 * HN) >= HN ? rg2 : rg;
          v.s[j] = __builtin_amdgcn_raw_buffer_load_b16(rn, int(pgroup[j]), 2 * wc, 0);
        }
      }
      return v;
    };
#pragma unroll 1
    for (int p0 = 0; p0 < n_pair; p0 += MB) {
      __syncthreads();                                  // what LDS held has been read
      if (tid < TM && __float_as_int(tscale) < 0)
        list[(tid >> 6 ? __popcll(pair_tok[0]) : 0) + __popcll(pair_tok[tid >> 6 ? 1 : 0] & ((1ull << lane) - 1))] = tid;
      __syncthreads();
      uint32_t pbase[PPER];
#pragma unroll
      for (int j = 0; j < PPER; ++j) {
        const int i = wave + NW * j, plane = i / (MB / RPL), lr = (i % (MB / RPL)) * RPL + lane / LPR;
        const int t = p0 + lr < n_pair ? m0 + list[p0 + lr] : 0;
        pbase[j] = p0 + lr < n_pair ? uint32_t(t) * xrow + uint32_t(plane) * 2u * uint32_t(a.ldx) + 16u * slot(lr, lane % LPR) : kOOB;
      }
      auto issue_pairs = [&](int kc, int half, int wc, Stage& S) {
        const int k0 = clamp_chunk(kc) * kKC;
#pragma unroll
        for (int j = 0; j < PPER; ++j)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, static_cast<void*>(&S[kw * SBYTES + (wave + NW * j) * 1024]), 16,
                                                   int(pbase[j]), 2 * k0 + kKC * half, 0, 0);
        issue_panel(SH ? wc * kKC : k0, S);
      };
      f32x16 sum[MT][PT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < PT; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e) sum[m][j][e] = 0.0f;
      // (lane (r, hi) of a product holds k = 8 hi .. + 7 of its 16 columns, on either side)
      auto multiply = [&](const Stage& S, int half, const Scales& sv) {
#pragma unroll
        for (int j = 0; j < PT; ++j) {
          f32x16 u[MT];
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int e = 0; e < 16; ++e) u[m][e] = SH ? 0.0f : sum[m][j][e];
#pragma unroll
          for (int ks = 0; ks < 4; ++ks) {
            const bf16x8 wf = widen8(*reinterpret_cast<const uint2*>(
                &S[kw * SBYTES + SA + (pair_row(j) + r) * kKC + 16 * slot(r, 4 * half + ks) + 8 * hi]));
#pragma unroll
            for (int m = 0; m < MT; ++m) {
              if (m > 0 && p0 + 32 * m >= n_pair) continue;
#pragma unroll
              for (int d = 0; d < 2; ++d) {
                const i32x4 x = *reinterpret_cast<const i32x4*>(
                    &S[kw * SBYTES + (d * MB + m * 32 + r) * kKC + 16 * slot(r, 2 * ks + hi)]);
                u[m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x), wf, u[m], 0, 0, 0);
              }
            }
          }
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            if constexpr (SH) {
              const float s = bf16_to_f32(uint16_t(sv.s[j]));
#pragma unroll
              for (int e = 0; e < 16; ++e) sum[m][j][e] = fmaf(u[m][e], s, sum[m][j][e]);
            } else {
              sum[m][j] = u[m];
            }
          }
        }
      };
      // a chunk's halves in st0 and st1, the next 64 columns in flight while one is multiplied
      int wc = store_chunk(0, list_entry(0));
      Scales sv = pair_scales(wc);
      issue_pairs(0, 0, wc, st0);
#pragma unroll 1
      for (int kc = 0; kc < nkw; ++kc) {
        const bool mine = KW == 1 || kw + KW * kc < nk;
        const int wn1 = store_chunk(kc + 1, list_entry(kc + 1));
        const Scales sn = pair_scales(wn1);
        stage_ready();
        issue_pairs(kc, 1, wc, st1);
        if (mine) multiply(st0, 0, sv);
        stage_ready();
        issue_pairs(kc + 1, 0, wn1, st0);
        if (mine) multiply(st1, 1, sv);
        wc = wn1;
        sv = sn;
      }
      stage_done();
      __syncthreads();                                  // every wave is done with the stages
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < PT; ++j)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            out[(kw * MB + 32 * m + 8 * (e >> 2) + 4 * hi + (e & 3)) * TN + pair_row(j) + r] = sum[m][j][e];
      __syncthreads();
      int first = 4 * hi;
      asm volatile("" : "+v"(first));                   // (or the masks of all outputs are kept over the loop)
#pragma unroll
      for (int e = 0; e < EC; ++e) {
        const uint32_t bit = 1u << (8 * ((EC * kw + e) >> 2) + first + (e & 3));
        const int i = before + __popc(own & (bit - 1)) - p0;
        if (!(own & bit) || i < 0 || i >= MB) continue;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          float f = out[i * TN + (wn * NT + nt) * 32 + r];
#pragma unroll
          for (int k = 1; k < KW; ++k) f += out[(k * MB + i) * TN + (wn * NT + nt) * 32 + r];
          facc[nt][e] = f;
        }
      }
    }
  }
  float* const ts = reinterpret_cast<float*>(&st1);
  if constexpr (KW > 1) __syncthreads();                // the sums have been read
  if (tid < TM) ts[tid] = fabsf(tscale);
  __syncthreads();

  // ---- epilogue: lane (r, hi) holds tokens 8 g + 4 hi + i of the token tile for row r
  // (KW > 1: outputs EC kw .. of each row tile)
  float sc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    sc[nt] = SH ? 1.0f : (col[nt] < N ? (GU && nt >= NT / 2 ? a.scale2 : a.scale)[col[nt]] : 0.0f);
  // the outputs through buffers (offsets past the end read zero and store nothing); the residuals of
  // the next row tile are loaded while one is stored (a load, a wait and a store per output chained
  // 64 memory latencies)
  const bool split = a.ks > 1;
  const uint32_t ldo = split ? uint32_t(N) : uint32_t(a.ldy);
  float* const dst = split ? a.part + size_t(bz) * T * N : a.y;
  const uint32_t out_bytes = (uint32_t(T - 1) * ldo + uint32_t(N)) * 4u;
  const __amdgpu_buffer_rsrc_t ry = make_rsrc(dst, out_bytes);
  const bool resid = MODE == MM_RESID && !split;
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(resid ? a.resid : nullptr, resid ? out_bytes : 0u);
  auto value = [&](int nt, int e, float tsc) {
    if constexpr (SH) return facc[nt][e] * tsc;
    else return facc[nt][e] * tsc * sc[nt];
  };
  auto offset = [&](int nt, int e) {
    const int t = m0 + token(e);
    return t < T && col[nt] < N ? (uint32_t(t) * ldo + uint32_t(col[nt])) * 4u : kOOB;
  };
  struct Resid {
    float v[MODE == MM_RESID ? EC : 1];
  };
  auto load_resid = [&](int nt) {
    Resid q{};
    if constexpr (MODE == MM_RESID) {
#pragma unroll
      for (int e = 0; e < EC; ++e)
        q.v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rr, int(offset(nt, e)), 0, 0));
    }
    return q;
  };
  Resid cur = load_resid(0), next{};
#pragma unroll
  for (int nt = 0; nt < (GU ? NT / 2 : NT); ++nt) {
    if (nt + 1 < NT) next = load_resid(nt + 1);
#pragma unroll
    for (int e = 0; e < EC; ++e) {
      const float tsc = ts[token(e)];
      float v = value(nt, e, tsc);
      if constexpr (GU) v = v / (1.0f + exp2f(-v * kLog2e)) * value(nt + NT / 2, e, tsc);
      else if constexpr (MODE == MM_RESID) v += cur.v[e];
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), ry, int(offset(nt, e)), 0, 0);
    }
    cur = next;
  }
}

// Float32 rows -> operand rows. One workgroup per token; thread i holds elements 4 (i + THREADS j).
// With a gain: the operand is x * gamma and the token's scale carries the inverse RMS of x. With
// K splits (part): x = resid + the splits' sum (in split order), which is also stored to y. The
// row is read in full before any of it is written, so source and destination may be one buffer.
// The scale is the largest power of two 2^-e that keeps q = rint(v 2^e) within three digits
// (|q| <= 0x7f7f7f); a row with a non-finite value gets a NaN scale, a zero row digits of zero.
//
// Digits or pair. In steps of the digit grid a digit's error has the variance 1 / 12, whatever the
// element; that of a pair, for a value f, is about f^2 2^-32 0.308 / 12 (the lo part's rounding, averaged
// over where lo falls in its binade and f in its own). Elements from an eighth of the row's largest up
// are held better by digits. Over the nonzero others the sums are compared: where the sum of f^2 -
// 2^32 / 0.308 is negative, digits would lose against a pair on outputs of these columns alone, and the
// row becomes a pair. Random rows stay digits (the rms of those elements is at least 1.6 times the
// threshold on 1000 Gaussian rows of 64, 2.4 times from 512 on, 1.13 times on 3200 rows of SwiGLU products of
// 150 to 28672); a row with one value of more than about 35 to 70 times the rms of the others does not. Nor
// does a row too small for a normal scale, whose digits would lack bits. (The comparison costs 0.5 to 1 us
// a launch: 8B layer at 512 tokens 243 -> 248 us. With one outlier token it takes 299 us, with one in nine
// tokens 305, in every token 306; the kernel on hi/lo operands throughout took 390.)
// MAPPED (groupwise store, no gain, no splits): x holds the retained columns in pieces of 16, piece p
// being store columns cols[p] .. + 15; the operand holds the store's chunks of 128 columns with any
// retained piece, in order, dropped pieces zero; the chunks' list is written to a.chunks.
// Bound by its 4 to 8 bytes read and 3 written per element.
constexpr float kPairSquare = 1.39e10f; // 2^32 / 0.308
constexpr int kMaxPieces = 2560;        // store pieces of the widest input (40960 columns)
template <int THREADS, int NV, bool MAPPED>
__global__ __launch_bounds__(THREADS) void pf_quant_kernel(PfQuantArgs a) {
  __shared__ float red[3][THREADS / kWave];
  const int tid = threadIdx.x, t = blockIdx.x, K = a.K, ld = a.ldo;
  int kz = (K + kKC - 1) / kKC * kKC;                    // digits written: K and its zero padding
  uint8_t* row = reinterpret_cast<uint8_t*>(a.o) + size_t(t) * 4 * ld;
  __shared__ short inv[MAPPED ? kMaxPieces : 1];         // store piece -> plan piece, -1 dropped
  __shared__ short chunk[MAPPED ? kMaxPieces / 8 : 1];   // operand chunk -> store chunk
  if constexpr (MAPPED) {
    const int np = a.store_cols / 16, nc = a.store_cols / kKC;
    __shared__ int n_chunks;
    for (int i = tid; i < np; i += THREADS) inv[i] = -1;
    __syncthreads();
    for (int p = tid; p < K / 16; p += THREADS) inv[a.cols[p] >> 4] = short(p);
    __syncthreads();
    if (tid < kWave) {
      int n = 0;
      for (int c0 = 0; c0 < nc; c0 += kWave) {
        const int c = c0 + tid;
        bool any = false;
        if (c < nc)
          for (int i = 0; i < 8; ++i) any |= inv[8 * c + i] >= 0;
        const unsigned long long m = __ballot(any);
        if (any) chunk[n + __popcll(m & ((1ull << tid) - 1))] = short(c);
        n += __popcll(m);
      }
      if (tid == 0) n_chunks = n;
    }
    __syncthreads();
    kz = n_chunks * kKC;
  }
  const __amdgpu_buffer_rsrc_t rp = make_rsrc(a.part, uint32_t(a.ks) * uint32_t(a.T) * uint32_t(K) * 4u);
  float4 v[NV];
  float amax = 0.0f, ss = 0.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int k = 4 * (tid + THREADS * j);
    v[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    int src = k;
    if constexpr (MAPPED) {
      if (k >= kz) continue;
      const int p = inv[8 * chunk[k / kKC] + (k % kKC) / 16];
      if (p < 0) continue;
      src = 16 * p + k % 16;
    } else if (k >= K) {
      continue;                                         // (K % 4 == 0 or the rest of the row is padding)
    }
    const f32x4u xv = *reinterpret_cast<const f32x4u*>(a.x + size_t(t) * a.ldx + src);
    v[j] = make_float4(xv.x, xv.y, xv.z, xv.w);
    if (a.ks) {
      const uint32_t off[1] = {(uint32_t(t) * uint32_t(K) + uint32_t(k)) * 4u};
      float4 sum[1] = {v[j]};
      add_splits(rp, off, uint32_t(a.T) * uint32_t(K) * 4u, 0, a.ks, sum);
      v[j] = sum[0];
    }
    if (a.ks) *reinterpret_cast<float4*>(a.y + size_t(t) * K + k) = v[j];
    if (a.gamma) {
      ss = fmaf(v[j].x, v[j].x, fmaf(v[j].y, v[j].y, fmaf(v[j].z, v[j].z, fmaf(v[j].w, v[j].w, ss))));
      const uint2 g = *reinterpret_cast<const uint2*>(a.gamma + k);
      v[j].x *= bf16_lo(g.x); v[j].y *= bf16_hi(g.x); v[j].z *= bf16_lo(g.y); v[j].w *= bf16_hi(g.y);
    } else if (!MAPPED) {
      // columns past K of the last four are padding, whatever the buffer holds
      if (k + 1 >= K) v[j].y = 0.0f;
      if (k + 2 >= K) v[j].z = 0.0f;
      if (k + 3 >= K) v[j].w = 0.0f;
    }
    // NaN-propagating maximum on the bits: |v| as an unsigned integer orders like the float, with
    // infinities and then NaNs above every finite value
    const uint32_t b = max(max(__float_as_uint(v[j].x) & 0x7fffffffu, __float_as_uint(v[j].y) & 0x7fffffffu),
                           max(__float_as_uint(v[j].z) & 0x7fffffffu, __float_as_uint(v[j].w) & 0x7fffffffu));
    amax = __uint_as_float(max(__float_as_uint(amax), b));
  }
  uint32_t mb = __float_as_uint(amax);
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    mb = max(mb, uint32_t(__shfl_xor(int(mb), o, kWave)));
    ss += __shfl_xor(ss, o, kWave);
  }
  const int w = tid >> 6;
  if ((tid & 63) == 0) {
    red[0][w] = __uint_as_float(mb);
    red[1][w] = ss;
  }
  __syncthreads();
  mb = 0;
  ss = 0.0f;
#pragma unroll
  for (int i = 0; i < THREADS / kWave; ++i) {
    mb = max(mb, __float_as_uint(red[0][i]));
    ss += red[1][i];
  }
  const bool finite = mb < 0x7f800000u;
  const float big = __uint_as_float(mb);
  // big 2^e in [2^22, 2^23), one less where the digits would not hold it; e <= 126 keeps the scale
  // a normal number
  int e = 22 - ((int(mb >> 23)) - 127);
  const bool tiny = mb < 0x00800000u || e > 126;
  if (tiny) e = 126;
  if (ldexpf(big, e) > 8355711.0f) --e;
  float up = ldexpf(1.0f, e > 127 ? 127 : e);
  // the comparison's sum, over the workgroup
  const float small = big * up * 0.125f;
  float more = 0.0f;
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const float f[4] = {v[j].x * up, v[j].y * up, v[j].z * up, v[j].w * up};
#pragma unroll
    for (int i = 0; i < 4; ++i)
      more += fabsf(f[i]) < small && f[i] != 0.0f ? fmaf(f[i], f[i], -kPairSquare) : 0.0f;
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) more += __shfl_xor(more, o, kWave);
  if ((tid & 63) == 0) red[2][w] = more;
  __syncthreads();
  more = 0.0f;
#pragma unroll
  for (int i = 0; i < THREADS / kWave; ++i) more += red[2][i];
  const bool pair = finite && (more < 0.0f || (tiny && mb != 0));
  asm volatile("" : "+v"(up));                          // (or the products above stay in registers)
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int k = 4 * (tid + THREADS * j);
    if (k >= kz) continue;
    const float f[4] = {v[j].x, v[j].y, v[j].z, v[j].w};
    if (pair) {
      uint32_t h[4], l[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        h[i] = f32_to_bf16(f[i]);
        l[i] = f32_to_bf16(f[i] - bf16_to_f32(uint16_t(h[i])));
      }
      *reinterpret_cast<uint2*>(row + 2 * k) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
      *reinterpret_cast<uint2*>(row + 2 * (size_t(ld) + k)) = make_uint2(l[0] | (l[1] << 16), l[2] | (l[3] << 16));
      continue;
    }
    uint32_t d2 = 0, d1 = 0, d0 = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int q = finite ? int(rintf(f[i] * up)) : 0;
      // balanced digits: adding 128 to the lower two makes the carries
      const int c = q + 0x8080;
      d0 |= ((uint32_t(c) & 0xffu) ^ 0x80u) << (8 * i);
      d1 |= (((uint32_t(c) >> 8) & 0xffu) ^ 0x80u) << (8 * i);
      d2 |= ((uint32_t(c >> 16)) & 0xffu) << (8 * i);
    }
    *reinterpret_cast<uint32_t*>(row + k) = d2;
    *reinterpret_cast<uint32_t*>(row + ld + k) = d1;
    *reinterpret_cast<uint32_t*>(row + 2 * size_t(ld) + k) = d0;
  }
  if (tid == 0) {
    float s = pair ? 1.0f : ldexpf(1.0f, -e);
    if (a.gamma) s *= rsqrtf(ss * a.inv_d + a.eps);
    a.tok[t] = !finite ? __uint_as_float(0x7fc00000u) : pair ? -s : s;
  }
  if constexpr (MAPPED) {
    if (t == 0)
      for (int i = tid; i < kz / kKC; i += THREADS) a.chunks[i] = chunk[i];
  }
}

// y = resid + the K splits' sum in split order (the last layer's output: no next operand)
__global__ __launch_bounds__(kBlock) void pf_i8_reduce_kernel(const float* __restrict__ part, int ks,
                                                              const float* __restrict__ resid, float* y,
                                                              int T, int N) {
  const int t = blockIdx.y, n = 4 * (blockIdx.x * kBlock + threadIdx.x);
  if (n >= N) return;
  const f32x4u r = *reinterpret_cast<const f32x4u*>(resid + size_t(t) * N + n);
  float4 v[1] = {make_float4(r.x, r.y, r.z, r.w)};
  const uint32_t stride = uint32_t(T) * uint32_t(N) * 4u, off[1] = {(uint32_t(t) * uint32_t(N) + uint32_t(n)) * 4u};
  add_splits(make_rsrc(part, uint32_t(ks) * stride), off, stride, 0, ks, v);
  *reinterpret_cast<f32x4u*>(y + size_t(t) * N + n) = f32x4u{v[0].x, v[0].y, v[0].z, v[0].w};
}

struct Shape {
  int tm, tn, kw, per_cu;
  float fixed;                          // us: launch, first chunk, epilogue
  float t_one, t_cu, t_full;            // us per step: few workgroups, one per CU, per_cu per CU
  float store;                          // factor of a groupwise store (vector work between the passes)
};
// 0: 128 x 256, eight waves of 32 x 128; 1: 64 x 128, four waves of 32 x 64; 2: 32 x 128, two waves
// of 32 x 64; 3: 32 x 64, four waves, each with every fourth chunk; 4: as 1, two groups of four waves,
// each with every other chunk. A step is a chunk per group. The times are measured (8B and 70B
// projections at 8 to 2048 tokens, each shape with 1 to 8 splits).
constexpr int kNumShapes = 5;
constexpr Shape kShapes[kNumShapes] = {{128, 256, 1, 1, 4.0f, 1.9f, 2.65f, 2.65f, 1.4f},
                                       {64, 128, 1, 2, 4.0f, 0.85f, 0.94f, 1.52f, 1.25f},
                                       {32, 128, 1, 2, 4.0f, 0.65f, 0.75f, 1.30f, 1.5f},
                                       {32, 64, 4, 1, 6.0f, 0.72f, 1.15f, 1.20f, 1.2f},
                                       {64, 128, 2, 1, 6.0f, 1.04f, 1.45f, 1.55f, 1.25f}};
constexpr int kMaxKSplit = 8;
constexpr int kMinSplitChunks = 2;

// expected time of a launch of w workgroups of n chunks each
float launch_us(const Shape& h, long w, int n, bool store) {
  const long slots = long(kNumCu) * h.per_cu;
  auto step = [&](long u) {             // step time with u workgroups on the chip
    return u <= kNumCu ? h.t_one + (h.t_cu - h.t_one) * float(u) / kNumCu
                       : h.t_cu + (h.t_full - h.t_cu) * float(u - kNumCu) / float(slots - kNumCu);
  };
  const long rounds = w / slots, rest = w % slots;
  const int steps = (n + h.kw - 1) / h.kw;
  return h.fixed + (store ? h.store : 1.0f) * float(steps) * (float(rounds) * h.t_full + (rest ? step(rest) : 0.0f));
}

template <int MODE, bool SH>
hipError_t launch_mode(const PfI8Args& a, int shape, hipStream_t s) {
  const Shape& h = kShapes[shape];
  const int rows = MODE == MM_GATEUP ? h.tn / 2 : h.tn;
  const int gx = (a.N + rows - 1) / rows, gy = (a.T + h.tm - 1) / h.tm;
  const dim3 grid(uint32_t(gx) * uint32_t(gy) * uint32_t(a.ks));
  if (shape == 0) hipLaunchKernelGGL((pf_i8_kernel<MODE, 4, 4, 2, 1, 2, SH>), grid, dim3(512), 0, s, a, gx, gy);
  else if (shape == 1) hipLaunchKernelGGL((pf_i8_kernel<MODE, 2, 2, 2, 1, 2, SH>), grid, dim3(256), 0, s, a, gx, gy);
  else if (shape == 2) hipLaunchKernelGGL((pf_i8_kernel<MODE, 2, 1, 2, 1, 1, SH>), grid, dim3(128), 0, s, a, gx, gy);
  else if (shape == 3) hipLaunchKernelGGL((pf_i8_kernel<MODE, 2, 1, 1, 4, 1, SH>), grid, dim3(256), 0, s, a, gx, gy);
  else hipLaunchKernelGGL((pf_i8_kernel<MODE, 2, 2, 2, 2, 2, SH>), grid, dim3(512), 0, s, a, gx, gy);
  return hipGetLastError();
}

template <int THREADS, bool MAPPED>
hipError_t launch_quant(const PfQuantArgs& a, int width, hipStream_t s) {
  const int nv = ((width + kKC - 1) / kKC * kKC + 4 * THREADS - 1) / (4 * THREADS);
  const dim3 g(a.T), b(THREADS);
  if (nv <= 1) hipLaunchKernelGGL((pf_quant_kernel<THREADS, 1, MAPPED>), g, b, 0, s, a);
  else if (nv <= 2) hipLaunchKernelGGL((pf_quant_kernel<THREADS, 2, MAPPED>), g, b, 0, s, a);
  else if (nv <= 4) hipLaunchKernelGGL((pf_quant_kernel<THREADS, 4, MAPPED>), g, b, 0, s, a);
  else if (nv <= 7) hipLaunchKernelGGL((pf_quant_kernel<THREADS, 7, MAPPED>), g, b, 0, s, a);
  else if (nv <= 11) hipLaunchKernelGGL((pf_quant_kernel<THREADS, 11, MAPPED>), g, b, 0, s, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

// The launch of least expected time (launch_us). A split adds its partial sums, written here and
// read by the consumer (about 4 TB/s). Large shapes move fewer bytes per product; small ones and
// splits fill the chip when there are few tokens: at 16 tokens the 8B down projection takes 44 us
// on 32 workgroups of shape 2 and 10.6 on 64 x 4 of shape 3, at 2048 tokens 184 us on shape 0
// and 242 on shape 1. Without splits the tokens may be cut in two launches, the first of whole
// rounds of shape 0, so that the last round is not mostly empty (8B gate/up at 700 tokens: 384
// tiles of shape 0 are one and a half rounds, 158 us, 144 us on shape 1; 512 tokens in one round of
// shape 0 and 188 on shape 1, 136 us). A cut has to promise 5 % of the projection, which is about what
// the model is off by: with any gain 8B layers of 780, 820, 1300 and 1800 tokens go from 384, 390, 648, 771 to
// 399, 408, 662, 792 us, 70B ones of 700, 900 and 1700 from 1139, 1355, 2439 to 1161, 1384, 2512, against
// 1700 tokens at 8B (751 -> 728) and 1300 and 1800 at 70B (1941 -> 1909, 2585 -> 2565); without cuts 1040
// tokens take 588 instead of 530 us, and 1728 instead of 1505.
PfI8Plan plan_pf_i8(MfmaMode mode, const PfI8Args& a) {
  const int chunks = (a.K + kKC - 1) / kKC;
  const bool store = a.sv.gs != nullptr;
  const bool can_split = mode != MM_GATEUP && a.part && a.N > 0;
  const long room = can_split ? long(a.part_floats / (size_t(a.T) * a.N)) : 1;
  const int max_ks = can_split ? int(std::max(1l, std::min({long(kMaxKSplit), long(chunks / kMinSplitChunks), room}))) : 1;
  auto tiles = [&](int i, int T) {
    const int rows = mode == MM_GATEUP ? kShapes[i].tn / 2 : kShapes[i].tn;
    return long((a.N + rows - 1) / rows) * ((T + kShapes[i].tm - 1) / kShapes[i].tm);
  };
  PfI8Plan best{0, 1, 0, 0};
  float best_us = 3e38f;
  for (int i = 0; i < kNumShapes; ++i)
    for (int k = 1; k <= max_ks; ++k) {
      const float us = launch_us(kShapes[i], tiles(i, a.T) * k, (chunks + k - 1) / k, store) +
                       (k > 1 ? float(k) * float(a.T) * float(a.N) * 4.0f * 2.0f / 4e6f : 0.0f);
      if (us < best_us) {
        best_us = us;
        best = PfI8Plan{i, k, 0, 0};
      }
    }
  for (int cut = kShapes[0].tm; cut < a.T; cut += kShapes[0].tm) {
    const float head = launch_us(kShapes[0], tiles(0, cut), chunks, store);
    for (int i = 1; i < kNumShapes; ++i) {
      const float us = head + launch_us(kShapes[i], tiles(i, a.T - cut), chunks, store);
      if (us < 0.95f * best_us) {
        best_us = us;
        best = PfI8Plan{0, 1, cut, i};
      }
    }
  }
  return best;
}

namespace {
hipError_t launch_part(MfmaMode mode, const PfI8Args& a, int shape, hipStream_t s) {
  if (a.sv.gs) {
    // store rows in whole chunks, one scale group each
    if (a.K % kKC != 0 || a.sv.ld % kKC != 0 || a.K > a.sv.ld || a.sv.store_rows < 1 ||
        (mode == MM_GATEUP && (!a.sv.w2 || !a.sv.gs2)))
      return hipErrorInvalidValue;
  } else if (a.K > a.ld || a.ld % 16 != 0) {
    return hipErrorInvalidValue;
  }
  if (a.T < 1 || a.K < 0 || a.ldx % kKC != 0 || a.ldx < a.K || a.ks < 1 || !a.tok || (a.sv.cols && !a.chunks) ||
      shape < 0 || shape >= kNumShapes || size_t(a.T) * 4 * a.ldx >= size_t(kOOB) ||
      size_t(a.T) * 4 * std::max(a.ldy, a.N) >= size_t(kOOB) ||
      (a.ks > 1 && (mode == MM_GATEUP || !a.part || size_t(a.ks) * a.T * a.N > a.part_floats)))
    return hipErrorInvalidValue;
  if (a.N == 0) return hipSuccess;
  const bool sh = a.sv.gs != nullptr;
  switch (mode) {
    case MM_QKV: return sh ? launch_mode<MM_QKV, true>(a, shape, s) : launch_mode<MM_QKV, false>(a, shape, s);
    case MM_RESID: return sh ? launch_mode<MM_RESID, true>(a, shape, s) : launch_mode<MM_RESID, false>(a, shape, s);
    case MM_GATEUP: return sh ? launch_mode<MM_GATEUP, true>(a, shape, s) : launch_mode<MM_GATEUP, false>(a, shape, s);
    default: return hipErrorInvalidValue;
  }
}
}  // namespace

hipError_t launch_pf_i8(MfmaMode mode, const PfI8Args& a0, const PfI8Plan& plan, hipStream_t s) {
  PfI8Args a = a0;
  a.ks = plan.ks;
  if (plan.cut <= 0) return launch_part(mode, a, plan.shape, s);
  if (plan.cut >= a.T || plan.ks != 1) return hipErrorInvalidValue;
  a.T = plan.cut;
  const hipError_t e = launch_part(mode, a, plan.shape, s);
  if (e != hipSuccess) return e;
  a.tok = a0.tok + plan.cut;
  a.x = a0.x + size_t(plan.cut) * 4 * a.ldx;
  if (a.resid) a.resid += size_t(plan.cut) * a.ldy;
  a.y += size_t(plan.cut) * a.ldy;
  a.T = a0.T - plan.cut;
  return launch_part(mode, a, plan.shape2, s);
}

hipError_t launch_pf_quant(const PfQuantArgs& a, hipStream_t s) {
  if (a.T < 1 || a.K < 0 || !a.tok || a.ldo % kKC != 0 || a.ldo < a.K || a.ldx % 4 != 0 || ((a.gamma || a.ks) && a.K % 4 != 0))
    return hipErrorInvalidValue;
  if (a.cols) {
    // the operand's width is at most the store's (one register array holds the row)
    if (!a.chunks || a.gamma || a.ks || a.K % 16 != 0 || a.store_cols % kKC != 0 || a.store_cols < a.K ||
        a.store_cols > 16 * kMaxPieces || a.ldo < a.store_cols)
      return hipErrorInvalidValue;
    return a.store_cols <= 4 * 256 * 7 ? launch_quant<256, true>(a, a.store_cols, s)
                                       : launch_quant<1024, true>(a, a.store_cols, s);
  }
  if (size_t(a.ks) * a.T * a.K * 4 >= size_t(kOOB)) return hipErrorInvalidValue;
  // wide rows, and short prompts (at most a workgroup per CU, each a chain of its own loads), on more
  // threads: 16 rows of 4096 and eight splits took 12 us on 256 threads with a wait per split, 4.6 now
  return a.K <= 4 * 256 * 7 && (a.T > kNumCu || a.K <= 1024) ? launch_quant<256, false>(a, a.K, s)
                                                            : launch_quant<1024, false>(a, a.K, s);
}

hipError_t launch_pf_i8_reduce(const float* part, int ks, const float* resid, float* y, int T, int N,
                               hipStream_t s) {
  if (N % 4 != 0 || T < 1 || ks < 0 || size_t(ks) * T * N * 4 >= size_t(kOOB)) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pf_i8_reduce_kernel, dim3((N / 4 + kBlock - 1) / kBlock, T), dim3(kBlock), 0, s, part, ks,
                     resid, y, T, N);
  return hipGetLastError();
}

}  // namespace tasp
