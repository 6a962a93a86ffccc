// GPU side of libsaki for gfx950 (CDNA4, wave64).
//
// Kernels (all on the caller's stream):
//   build_index_kernel   key codes c = B_k^T (k - mu) for every query head (Eq. 4)
//   append_index_kernel  the same for up to 16 keys
//   query_sketch_kernel  z = B_q^T q and b = q^T mu of many rows
//   score_batch_kernel   s = z . c + b on MFMA for blocks of 16 query rows,
//                        top-64 per row (two passes: block maxima and a
//                        threshold, then the candidates)
//   score_scan_kernel    z, b and s in one pass over the codes for long rows
//                        (batches of decode queries), running top-64 per row
//   score_decode_kernel  the same for few query rows per code set (decode):
//                        one key per lane, key range split into chunks
//   merge_kernel         reduces per-chunk partial top-64 lists of one row
//   keys_hi_kernel       bf16 hi/lo split of the keys and their norm bounds
//   exact_gate_kernel    exact top-64 and recall hits: float32 gate from the
//                        candidate list, bf16x3 MFMA scan, float64 decisions
//   exact_bf16_kernel, exact_mfma_kernel  fallback tiers of the same
//   exact_tau_kernel, exact_scan_kernel, exact_decide_kernel  the same where few
//                        query rows share many keys: a gate per row, one bf16x3
//                        scan of the keys, float64 decisions
//   exact_stream_kernel  exact float64 scores and top-64, one wave per 1 or 4
//                        rows: few keys, rows that the scan flags, workspaces
//                        or alignments that the scan does not take
//   moments_kernel       calibration moments in float64
//   attend_kernel        RoPE attention over the selected keys, a work-group
//                        per row
//   attend_rows_kernel   the same for many rows, a wave per row
//   export_kernel        debug read-back of the codes
// Top-k selection is in saki_topk.h.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "saki.h"
#include "saki_internal.h"
#include "saki_topk.h"

namespace {

using saki::kMaxK;
using saki::kTile;
using namespace saki_dev;

// MFMA operand and accumulator vectors
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8_t as_bf16x8(uint4 v) {
  bf16x8_t r;
  __builtin_memcpy(&r, &v, sizeof(r));
  return r;
}
__device__ __forceinline__ i16x4_t as_i16x4(uint2 v) {
  i16x4_t r;
  __builtin_memcpy(&r, &v, sizeof(r));
  return r;
}

constexpr int kStreamWaves = 4;  // waves per workgroup, streaming kernels
constexpr int kMfmaWaves = 2;    // waves per workgroup, MFMA kernels
constexpr int kMR = 16;          // query rows per wave on the MFMA kernels

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t bf16_bits(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ float bf16_round(float x) { return __uint_as_float(bf16_bits(x) << 16); }

// Storage types of the codes (template parameter ST of the index kernels).
constexpr int kStF32 = SAKI_F32, kStBf16 = SAKI_BF16, kStFp8 = SAKI_FP8;
template <int ST>
constexpr int code_bytes() { return ST == kStF32 ? 4 : ST == kStBf16 ? 2 : 1; }

// float32 -> fp8 E4M3 code: round to the nearest E4M3 value (ties to the even
// code), magnitudes of 448 and more saturate to 448 (finite inputs).
__device__ __forceinline__ uint32_t e4m3_bits(float x) {
  const uint32_t sign = (__float_as_uint(x) >> 24) & 0x80u;
  const float a = fabsf(x);
  if (!(a < 448.f)) return sign | 0x7Eu;
  if (a < 0x1p-6f) return sign | (uint32_t)rintf(a * 512.f);  // subnormal: multiples of 2^-9
  uint32_t u = __float_as_uint(a);
  u += 0x7FFFFu + ((u >> 20) & 1u);  // round the float32 significand to 3 bits, ties to even
  u &= 0xFFF00000u;
  const uint32_t code = (((u >> 23) - 120u) << 3) | ((u >> 20) & 7u);  // rebias 127 -> 7
  return sign | (code > 0x7Eu ? 0x7Eu : code);
}

// Four fp8 E4M3 codes (the bytes of w, lowest first) -> two words of bf16
// pairs, one instruction each (through float32 it took six, which bound the
// scoring of fp8 codes).  Exact: an E4M3 value has at most 4 significant bits.
__device__ __forceinline__ uint2 e4m3x4_to_bf16(uint32_t w) {
  const auto lo = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.f, false);  // bytes 0, 1
  const auto hi = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.f, true);   // bytes 2, 3
  uint2 r;
  __builtin_memcpy(&r.x, &lo, sizeof(r.x));
  __builtin_memcpy(&r.y, &hi, sizeof(r.y));
  return r;
}

template <bool BF>
__device__ __forceinline__ float load_key_elem(const void* p, size_t i) {
  if constexpr (BF) {
    const uint16_t v = reinterpret_cast<const uint16_t*>(p)[i];
    return __uint_as_float((uint32_t)v << 16);
  } else {
    return reinterpret_cast<const float*>(p)[i];
  }
}

// Key elements i .. i + 3 (i a multiple of 4) as floats.
template <bool BF>
__device__ __forceinline__ float4 load_key4(const void* p, size_t i) {
  if constexpr (BF) {
    const uint2 v = *reinterpret_cast<const uint2*>(reinterpret_cast<const uint16_t*>(p) + i);
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u),
                       __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
  } else {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(p) + i);
  }
}

// Unpack one 16-byte code piece into floats.
template <bool BF>
__device__ __forceinline__ void unpack_piece(uint4 v, float* out) {
  if constexpr (BF) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      out[2 * e] = __uint_as_float(w[e] << 16);
      out[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
    }
  } else {
    out[0] = __uint_as_float(v.x);
    out[1] = __uint_as_float(v.y);
    out[2] = __uint_as_float(v.z);
    out[3] = __uint_as_float(v.w);
  }
}

// Unpack one 16-byte piece of codes stored as ST into 16 / code_bytes<ST>() floats.
template <int ST>
__device__ __forceinline__ void unpack_codes(uint4 v, float* out) {
  if constexpr (ST == kStFp8) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint2 b = e4m3x4_to_bf16(w[e]);
      out[4 * e] = __uint_as_float(b.x << 16);
      out[4 * e + 1] = __uint_as_float(b.x & 0xffff0000u);
      out[4 * e + 2] = __uint_as_float(b.y << 16);
      out[4 * e + 3] = __uint_as_float(b.y & 0xffff0000u);
    }
  } else {
    unpack_piece<ST == kStBf16>(v, out);
  }
}

__device__ __forceinline__ int row_limit(int i, int Q, int N_valid, const int* q_pos) {
  if (i >= Q) return 0;
  if (!q_pos) return N_valid;
  const long long lim = (long long)q_pos[i] + 1;
  return lim < 0 ? 0 : (lim > N_valid ? N_valid : (int)lim);
}

// MI355X deals consecutive work-groups round-robin over its 8 XCDs, each with
// its own L2.  The MFMA kernels run on a 1-D grid of 8 * per_xcd work-groups
// and renumber them so that XCD x gets the contiguous logical range
// [x * per_xcd, (x + 1) * per_xcd): the row blocks of one head (which read the
// same codes / keys) then share one L2.  Returns -1 for padding work-groups.
constexpr int kXcds = 8;
__device__ __forceinline__ long long xcd_logical_block(long long total) {
  const long long hw = blockIdx.x;
  const long long per_xcd = (total + kXcds - 1) / kXcds;
  const long long logical = (hw % kXcds) * per_xcd + hw / kXcds;
  return logical < total ? logical : -1;
}

// Wave-wide max / min, returned in a scalar register (every lane holds the
// same value after the butterfly), so that what is derived from it stays on
// the scalar unit.
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int m = kWave / 2; m > 0; m >>= 1) v = max(v, __shfl_xor(v, m, kWave));
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ int wave_min_i(int v) {
#pragma unroll
  for (int m = kWave / 2; m > 0; m >>= 1) v = min(v, __shfl_xor(v, m, kWave));
  return __builtin_amdgcn_readfirstlane(v);
}

// max / min of floats as v_maximum3_f32 / v_minimum3_f32 (a NaN operand gives
// NaN; scores are never NaN), without the quieting moves fmaxf / fminf need.
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float vmin(float a, float b) { return __builtin_elementwise_minimum(a, b); }

// Final list entry of a row -> output index / score.
template <class KO>
__device__ __forceinline__ int out_index(typename KO::K e) {
  const int j = KO::index(e);
  return j == kPadIdx ? -1 : j;
}

// Hits of an exact list (one entry per lane, the first k lanes count) against
// approx_idx row `row` (length k; entries < 0 never match).
__device__ __forceinline__ int row_hits(int ej, const int* __restrict__ approx, size_t row, int k) {
  const int lane = lane_id();
  const int aj = lane < k ? approx[row * k + lane] : -1;
  bool found = false;
  for (int m = 0; m < k; ++m) {
    const int v = __shfl(aj, m, kWave);
    found |= (v >= 0 && v == ej);
  }
  const bool counts = lane < k && ej >= 0 && found;
  return __popcll(__ballot(counts));
}

// ---------------------------------------------------------------- build index

// Key codes c_j = B_k^T (k_j - mu) on the bf16 MFMA (16x16x32).  Each float32
// operand is split into three bf16 terms: x = x1 + x2 + x3 with x1 = bf16(x),
// x2 = bf16(x - x1), x3 = bf16(x - x1 - x2) (each term takes the next 8
// significant bits, so the three carry a float32's 24), and likewise
// w = w1 + w2 + w3 for B_k.  The six products x_a w_b with a + b <= 4 are
// formed, x1 w1 into one float32 accumulator and the five smaller ones into a
// second; what is left out (x2 w3, x3 w2, x3 w3 and the splits' remainders)
// is below 4 * 2^-24 |x| |w| per element, the size of float32 rounding, at
// 6 bf16 products where float32 operands would take 16 times the MFMA time of
// one.  A work-group takes a slice of the keys of one KV head (16-key groups,
// taken by its 8 waves in turn) and computes their codes for every query head of the group, so
// each key is read once (a short range, a decode append, takes one query head
// per work-group instead, so that the heads' factors load in parallel).  For
// a group of 16 keys and a block of 16 code dimensions the MFMA forms
// D[m][key] = sum_c B_k[c][m] (k - mu)[key][c] in 4 steps of 32 dimensions:
// lane (key qi, group g) loads dims 32 kk + 8 g .. + 7 of its key (the B
// operand) and of B_k's column m = 16 mc + qi (the A operand).  The three
// terms of B_k of up to build_heads_lds<r>() heads at a time sit in LDS,
// transposed (one row of 128 dims per code dimension, rows of 136 bf16 so
// that the 16 rows one read touches start 4 banks apart).  Lane (qi, g) ends
// with dims 16 mc + 4 g .. + 3 of key qi: one 16-byte float32 piece, half a
// bf16 piece or a quarter of an fp8 piece.  Centring is float32 (k - mu)
// before the product, as the paper writes it.
constexpr int kBuildKeys = 1024;         // keys per work-group, at least
constexpr int kBuildSplitKeys = 256;     // ranges up to this many keys: one query head per work-group
constexpr int kBuildRounds = 1;          // work-groups per slot the device holds
constexpr int kBuildRow = 136;           // bf16 per LDS row of B_k (128 dims + 8)
constexpr int kBuildLdsBytes = 104448;   // B_k of up to 4 heads at r = 32
template <int RK>
constexpr int build_heads_lds() { return kBuildLdsBytes / (3 * RK * kBuildRow * 2); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two floats rounded to bf16 (nearest even, v_cvt_pk_bf16_f32), packed low
// first.
__device__ __forceinline__ uint32_t bf16x2_bits(float a, float b) {
  const bf16x2_t v = __builtin_convertvector(f32x2_t{a, b}, bf16x2_t);
  uint32_t u;
  __builtin_memcpy(&u, &v, sizeof(u));
  return u;
}

// Splits a pair of floats into three packed bf16 pairs t[0] + t[1] + t[2].
__device__ __forceinline__ void split3_bf16x2(float a, float b, uint32_t t[3]) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    t[p] = bf16x2_bits(a, b);
    a -= __uint_as_float(t[p] << 16);
    b -= __uint_as_float(t[p] & 0xffff0000u);
  }
}

// grid (slices, H_kv or H_q (per_head), B), block 64 * kBuildWaves; the keys
// [n_begin rounded down to 16, n_end) are cut into gridDim.x contiguous
// slices, one per work-group, so that B_k is staged in LDS once per slice.
constexpr int kBuildWaves = 8;
template <int RK, bool KBF, int ST>
__global__ __launch_bounds__(kBuildWaves * kWave) void build_index_kernel(
    const void* __restrict__ keys, const float* __restrict__ Bk,
    const float* __restrict__ mu, int H_q, int H_kv, int N_cap, int n_tiles,
    uint8_t* __restrict__ index, int n_begin, int n_end, int per_head) {
  constexpr int D = saki::kHeadDim;
  constexpr int ES = code_bytes<ST>();
  constexpr int HB = build_heads_lds<RK>();
  static_assert(HB >= 1, "one head of B_k fits");
  constexpr size_t TB = (size_t)kTile * RK * ES;  // bytes of one 64-key tile
  constexpr int NM = RK / 16;
  constexpr int SG = 2;                // 16-key groups per wave step
  constexpr int MB = NM < 2 ? NM : 2;  // 16-dim code blocks per pass over a step's keys
  constexpr int PS = RK * kBuildRow;  // bf16 per term of one head
  __shared__ __align__(16) uint16_t bks[HB * 3 * PS];
  const int G = H_q / H_kv;
  const int gkv = per_head ? (int)blockIdx.y / G : (int)blockIdx.y, b = blockIdx.z;
  const int h_first = per_head ? (int)blockIdx.y : gkv * G;  // query heads [h_first, h_end)
  const int h_end = per_head ? h_first + 1 : h_first + G;
  const int tid = threadIdx.x, wave = tid / kWave, lane = tid % kWave;
  const int qi = lane % 16, g = lane / 16;
  // this work-group's keys [k0, k1): slices of the range from n_begin rounded
  // down to 16, a multiple of 16 keys each
  const int kb = (n_begin / 16) * 16;
  const int slice = ((n_end - kb + (int)gridDim.x - 1) / (int)gridDim.x + 15) / 16 * 16;
  const int k0 = kb + (int)blockIdx.x * slice;
  if (k0 >= n_end) return;  // the whole work-group
  const int k1 = min(n_end, k0 + slice);
  const size_t key_base = ((size_t)b * H_kv + gkv) * N_cap;
  __shared__ __align__(16) float mus[D];  // mu of the KV head (read after the first barrier below)
  if (tid < D / 4)
    reinterpret_cast<float4*>(mus)[tid] = reinterpret_cast<const float4*>(mu + (size_t)gkv * D)[tid];
  // raw key dims 32 kk + 8 g .. + 7 of key n (16 bytes of bf16 or 32 of float32 per kk)
  struct RawKey {
    uint4 v[KBF ? 4 : 8];
  };
  auto load_raw = [&](int n, bool ok, RawKey& r) {
#pragma unroll
    for (int i = 0; i < (KBF ? 4 : 8); ++i) {
      const size_t off = (key_base + n) * D + (KBF ? 32 * i + 8 * g : 32 * (i / 2) + 8 * g + 4 * (i % 2));
      r.v[i] = ok ? (KBF ? *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) + off)
                         : *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(keys) + off))
                  : uint4{0u, 0u, 0u, 0u};
    }
  };
  // (k - mu) split into three bf16 terms: xp[p][kk] holds dims 32 kk + 8 g .. + 7
  auto split_key = [&](const RawKey& r, bool ok, uint4 xp[3][4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      float f[8];
      if constexpr (KBF) {
        unpack_piece<true>(r.v[kk], f);
      } else {
        unpack_piece<false>(r.v[2 * kk], f);
        unpack_piece<false>(r.v[2 * kk + 1], f + 4);
      }
      float m[8];
      *reinterpret_cast<float4*>(m) = *reinterpret_cast<const float4*>(&mus[32 * kk + 8 * g]);
      *reinterpret_cast<float4*>(m + 4) = *reinterpret_cast<const float4*>(&mus[32 * kk + 8 * g + 4]);
      uint32_t t[4][3];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        split3_bf16x2(ok ? f[2 * e] - m[2 * e] : 0.f, ok ? f[2 * e + 1] - m[2 * e + 1] : 0.f, t[e]);
#pragma unroll
      for (int p = 0; p < 3; ++p) xp[p][kk] = uint4{t[0][p], t[1][p], t[2][p], t[3][p]};
    }
  };
  // code dims 16 (mc0 + mc) + 4 g .. + 3 of key n, mc < MB
  auto store = [&](int n, int h, int mc0, const f32x4_t* acc) {
    uint8_t* tb = index + (((size_t)b * H_q + h) * n_tiles + n / kTile) * TB;
#pragma unroll
    for (int mc = 0; mc < MB; ++mc) {
      const int m = 16 * (mc0 + mc) + 4 * g;  // first code dim of this lane
      uint8_t* dst = tb + (size_t)(m * ES / 16) * kTile * 16 + (size_t)(n % kTile) * 16 + (m * ES) % 16;
      const f32x4_t v = acc[mc];
      if constexpr (ST == kStFp8) {
        *reinterpret_cast<uint32_t*>(dst) = e4m3_bits(v[0]) | (e4m3_bits(v[1]) << 8) |
                                            (e4m3_bits(v[2]) << 16) | (e4m3_bits(v[3]) << 24);
      } else if constexpr (ST == kStBf16) {
        *reinterpret_cast<uint2*>(dst) =
            uint2{bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16)};
      } else {
        *reinterpret_cast<uint4*>(dst) = uint4{__float_as_uint(v[0]), __float_as_uint(v[1]),
                                               __float_as_uint(v[2]), __float_as_uint(v[3])};
      }
    }
  };
  // a wave takes SG groups of 16 keys per step, so that each B_k operand read
  // from LDS serves SG products
  const int n_steps = (k1 - k0 + 16 * SG - 1) / (16 * SG);
  auto key_at = [&](int st, int sg) { return k0 + 16 * (SG * st + sg) + qi; };
  auto key_ok = [&](int n) { return n >= n_begin && n < k1; };
  constexpr int NT = kBuildWaves * kWave;
  constexpr int FB = 4;  // B_k pairs per thread whose loads are issued together
  for (int h0 = h_first; h0 < h_end; h0 += HB) {
    const int nh = min(HB, h_end - h0);
    __syncthreads();  // the previous heads' reads are done
    // B_k[h][c][m] (row-major D x RK) -> term p at bks[((hh * 3 + p) * RK + m) * kBuildRow + c],
    // dims c = 2 c2, 2 c2 + 1 per pair
    for (int e0 = tid; e0 < nh * (D / 2) * RK; e0 += FB * NT) {
      float2 w[FB];
#pragma unroll
      for (int i = 0; i < FB; ++i) {
        const int e = e0 + i * NT;
        const int m = e % RK, c2 = (e / RK) % (D / 2), hh = e / (RK * (D / 2));
        const float* src = Bk + ((size_t)(h0 + hh) * D + 2 * c2) * RK + m;
        w[i] = e < nh * (D / 2) * RK ? make_float2(src[0], src[RK]) : make_float2(0.f, 0.f);
      }
#pragma unroll
      for (int i = 0; i < FB; ++i) {
        const int e = e0 + i * NT;
        const int m = e % RK, c2 = (e / RK) % (D / 2), hh = e / (RK * (D / 2));
        uint32_t t[3];
        split3_bf16x2(w[i].x, w[i].y, t);
        if (e < nh * (D / 2) * RK)
#pragma unroll
          for (int p = 0; p < 3; ++p)
            *reinterpret_cast<uint32_t*>(&bks[((hh * 3 + p) * RK + m) * kBuildRow + 2 * c2]) = t[p];
      }
    }
    __syncthreads();
    RawKey cur[SG];
    if (wave < n_steps)
#pragma unroll
      for (int sg = 0; sg < SG; ++sg) load_raw(key_at(wave, sg), key_ok(key_at(wave, sg)), cur[sg]);
    for (int st = wave; st < n_steps; st += kBuildWaves) {
      uint4 xp[SG][3][4];
#pragma unroll
      for (int sg = 0; sg < SG; ++sg) split_key(cur[sg], key_ok(key_at(st, sg)), xp[sg]);
      if (st + kBuildWaves < n_steps)  // the wave's next step, loaded under this one's products
#pragma unroll
        for (int sg = 0; sg < SG; ++sg)
          load_raw(key_at(st + kBuildWaves, sg), key_ok(key_at(st + kBuildWaves, sg)), cur[sg]);
#pragma unroll 1
      for (int hm = 0; hm < nh * (NM / MB); ++hm) {  // head hh, code dims from 16 mc0
        const int hh = hm / (NM / MB), mc0 = (hm % (NM / MB)) * MB;
        f32x4_t hi[SG][MB], lo[SG][MB];
#pragma unroll
        for (int sg = 0; sg < SG; ++sg)
#pragma unroll
          for (int mc = 0; mc < MB; ++mc) {
            hi[sg][mc] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            lo[sg][mc] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          }
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          // the operands of one 32-dim step at a time (register room)
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int mc = 0; mc < MB; ++mc) {
            const uint16_t* wr = &bks[(hh * 3 * RK + 16 * (mc0 + mc) + qi) * kBuildRow + 32 * kk + 8 * g];
            const bf16x8_t w1 = as_bf16x8(*reinterpret_cast<const uint4*>(wr));
            const bf16x8_t w2 = as_bf16x8(*reinterpret_cast<const uint4*>(wr + PS));
            const bf16x8_t w3 = as_bf16x8(*reinterpret_cast<const uint4*>(wr + 2 * PS));
#pragma unroll
            for (int sg = 0; sg < SG; ++sg) {
              const bf16x8_t x1 = as_bf16x8(xp[sg][0][kk]), x2 = as_bf16x8(xp[sg][1][kk]),
                             x3 = as_bf16x8(xp[sg][2][kk]);
              hi[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x1, hi[sg][mc], 0, 0, 0);
              lo[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w3, x1, lo[sg][mc], 0, 0, 0);
              lo[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, x2, lo[sg][mc], 0, 0, 0);
              lo[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x3, lo[sg][mc], 0, 0, 0);
              lo[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w2, x1, lo[sg][mc], 0, 0, 0);
              lo[sg][mc] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1, x2, lo[sg][mc], 0, 0, 0);
            }
          }
        }
#pragma unroll
        for (int sg = 0; sg < SG; ++sg) {
#pragma unroll
          for (int mc = 0; mc < MB; ++mc) hi[sg][mc] += lo[sg][mc];
          const int n = key_at(st, sg);
          if (key_ok(n)) store(n, h0 + hh, mc0, hi[sg]);
        }
      }
    }
  }
}

// Codes of a few appended keys (a decode step's newest one): one wave per 16
// code dimensions of a code set, the same products in the same order as
// build_index_kernel (so an index grown key by key equals one built at once),
// with B_k split in the registers that its loads fill.  Latency bounds it: one
// round of loads, 24 MFMAs, no LDS and no barrier.  One key of 32 heads took
// 6.8 us in build_index_kernel, which stages the terms of B_k in LDS for many
// keys; past one MFMA tile of keys it is the better one.
constexpr int kAppendKeys = 16;
template <int RK, bool KBF, int ST>
__global__ __launch_bounds__(kWave) void append_index_kernel(
    const void* __restrict__ keys, const float* __restrict__ Bk, const float* __restrict__ mu, int H_q,
    int H_kv, int N_cap, int n_tiles, uint8_t* __restrict__ index, int n_begin, int n_count) {
  constexpr int D = saki::kHeadDim;
  constexpr int ES = code_bytes<ST>();
  const int mc = blockIdx.x, h = blockIdx.y;
  const size_t b = blockIdx.z;
  const int gkv = h / (H_q / H_kv);
  const int lane = lane_id(), qi = lane % 16, g = lane / 16;
  const bool ok = qi < n_count;
  const int n = n_begin + (ok ? qi : 0);
  // lane (qi, g): dims 32 kk + 8 g + e of B_k's column 16 mc + qi and of key qi
  const float* wp = Bk + ((size_t)h * D + 8 * g) * RK + 16 * mc + qi;
  float w[4][8], x[4][8];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) w[kk][e] = wp[(size_t)(32 * kk + e) * RK];
  const size_t kr = ((b * H_kv + gkv) * N_cap + n) * D + 8 * g;
  const float* mr = mu + (size_t)gkv * D + 8 * g;
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
#pragma unroll
    for (int e = 0; e < 8; e += 4) {
      const float4 kv = load_key4<KBF>(keys, kr + 32 * kk + e);
      const float4 mv = *reinterpret_cast<const float4*>(mr + 32 * kk + e);
      x[kk][e] = ok ? kv.x - mv.x : 0.f;
      x[kk][e + 1] = ok ? kv.y - mv.y : 0.f;
      x[kk][e + 2] = ok ? kv.z - mv.z : 0.f;
      x[kk][e + 3] = ok ? kv.w - mv.w : 0.f;
    }
  f32x4_t hi = {0.f, 0.f, 0.f, 0.f}, lo = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    uint32_t wt[4][3], xt[4][3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      split3_bf16x2(w[kk][2 * e], w[kk][2 * e + 1], wt[e]);
      split3_bf16x2(x[kk][2 * e], x[kk][2 * e + 1], xt[e]);
    }
    bf16x8_t wv[3], xv[3];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      wv[p] = as_bf16x8(uint4{wt[0][p], wt[1][p], wt[2][p], wt[3][p]});
      xv[p] = as_bf16x8(uint4{xt[0][p], xt[1][p], xt[2][p], xt[3][p]});
    }
    hi = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[0], xv[0], hi, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[2], xv[0], lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[1], xv[1], lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[0], xv[2], lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[1], xv[0], lo, 0, 0, 0);
    lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv[0], xv[1], lo, 0, 0, 0);
  }
  hi += lo;
  if (!ok) return;
  const int m = 16 * mc + 4 * g;  // first code dim of this lane
  uint8_t* dst = index + ((b * H_q + h) * n_tiles + n / kTile) * ((size_t)kTile * RK * ES) +
                 (size_t)(m * ES / 16) * kTile * 16 + (size_t)(n % kTile) * 16 + (m * ES) % 16;
  if constexpr (ST == kStFp8)
    *reinterpret_cast<uint32_t*>(dst) =
        e4m3_bits(hi[0]) | (e4m3_bits(hi[1]) << 8) | (e4m3_bits(hi[2]) << 16) | (e4m3_bits(hi[3]) << 24);
  else if constexpr (ST == kStBf16)
    *reinterpret_cast<uint2*>(dst) =
        uint2{bf16_bits(hi[0]) | (bf16_bits(hi[1]) << 16), bf16_bits(hi[2]) | (bf16_bits(hi[3]) << 16)};
  else
    *reinterpret_cast<uint4*>(dst) = uint4{__float_as_uint(hi[0]), __float_as_uint(hi[1]), __float_as_uint(hi[2]),
                                           __float_as_uint(hi[3])};
}

// grid (tiles, B*H_q), block 64: codes -> float [B, H_q, N_cap, r].
template <int RK, int ST>
__global__ __launch_bounds__(64) void export_kernel(const uint8_t* __restrict__ index,
                                                    int n_tiles, int N_cap,
                                                    float* __restrict__ out) {
  constexpr int ES = code_bytes<ST>();
  constexpr int CPP = saki::kChunkBytes / ES;
  constexpr int NP = RK / CPP;
  const int tile = blockIdx.x;
  const size_t bh = blockIdx.y;
  const int t = threadIdx.x;
  const int n = tile * kTile + t;
  if (n >= N_cap) return;
  const uint8_t* tbase = index + (bh * n_tiles + tile) * ((size_t)kTile * RK * ES);
  for (int piece = 0; piece < NP; ++piece) {
    const uint4 v = *reinterpret_cast<const uint4*>(tbase + (size_t)piece * kTile * 16 + (size_t)t * 16);
    float f[CPP];
    unpack_codes<ST>(v, f);
    for (int e = 0; e < CPP; ++e) out[(bh * N_cap + n) * RK + piece * CPP + e] = f[e];
  }
}

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x2_t as_bf16x2(uint32_t v) {
  bf16x2_t r;
  __builtin_memcpy(&r, &v, sizeof(r));
  return r;
}

// ---------------------------------------------------------------- sketch scoring, decode

// Few query rows per code set.  The rows of a code set are its gq = H_q /
// index_heads query heads times the Q queries, numbered rho = i * gq + (h % gq),
// so that a work-group's R rows are the heads sharing the codes (for a
// GQA-shared index) before further queries.  A work-group of W = 4, 8 or 16 waves
// takes R rows and one chunk of keys, wave w the tiles w, w + W, ... of it, one
// key of a tile per lane, and leaves one sorted top-64 per row (W = 4 too for
// one row of a few keys; launch_decode has the rule).
//   sketch  z = B_q^T q (rounded to bf16 for bf16 and fp8 codes) and b = q^T mu
//           (Sec. 6), float32 sums of 128 / W dims per wave, added in wave
//           order; the wave's first tiles are requested before.
//   head    the scores of the wave's first 8 tiles stay in registers.  The 64th
//           largest of the work-group's 64 W lane maxima is a gate: 64 keys
//           score at least that, and of the 512 W keys about 67 do.  These go
//           to the row's candidates.
//   tail    every further key scoring above the gate is a candidate (the 64
//           head keys at the gate have lower indices, so ties lose nothing).
//           After every 16 tiles of a wave, candidates that fill more than half
//           of their room are cut to the best 64, whose last is the new gate.
// The candidates (at most decode_cap<R>()) are sorted 64 at a time and merged.  A
// work-group whose candidates do not fit (many equal scores, scores that rise
// along the keys) selects online instead, row by row (RowLists).
// An online top-64 per wave and row (a sort and a merge for every 64 keys
// that beat the threshold, about 5 in the first 2,048 keys) bound the short
// chunks: 21 us for 32 rows over 4,001 keys, and 85 us for 4 rows of each of 32
// fp8 code sets over 100,003 keys (1.2 TB/s).
constexpr int kDecodeWaves = 16;  // at most
constexpr int kDecodeTiles = 8;   // head tiles per wave
constexpr int kDecodeRound = 16;  // tail tiles per wave between checks
template <int R>
constexpr int decode_cap() { return R >= 4 ? 512 : 1024; }
// Bytes of LDS that W waves share besides the kernel's own arrays.
template <int RK, int R>
constexpr size_t decode_area(int W) {
  const size_t part = (size_t)W * R * (RK + 1) * 4, most = (size_t)R * W * kWave * 4, lists = (size_t)W * kWave * 16;
  return std::max(part, std::max(most, lists));
}

// Merges the n sorted lists of 64 at m[(r * stride + i) * 64], i < n, of each
// row r < R into list 0 of the row, by all waves of the work-group.
template <class KO, int R>
__device__ __forceinline__ void merge_tree(typename KO::K* m, int stride, int n, int wave, int waves,
                                           int lane) {
  for (int st = 1; st < n; st *= 2) {  // n is uniform over the work-group
    const int pairs = (n - st + 2 * st - 1) / (2 * st);
    for (int t = wave; t < R * pairs; t += waves) {
      typename KO::K* x = m + ((size_t)(t % R) * stride + (size_t)(t / R) * 2 * st) * kWave;
      typename KO::K a = x[lane];
      wave_merge<KO>(a, x[(size_t)st * kWave + lane]);
      x[lane] = a;
    }
    __syncthreads();
  }
}

// grid: 1-D, xcd_logical_block order over (code set of a sequence, chunk, row
// group), row groups fastest (they read the same codes), block 64 W.  The loops
// count tiles: steps past the last of up to 2^31 - 1 keys do not fit an int.
template <int RK, int ST, int R>
__global__ __launch_bounds__(kDecodeWaves * kWave) void score_decode_kernel(
    const uint8_t* __restrict__ index, int n_tiles, int N_valid, int Q,
    const int* __restrict__ q_pos, const float* __restrict__ q, const float* __restrict__ Bq,
    const float* __restrict__ mu, int H_q, int H_kv, int gq, int n_bi, int row_groups, int chunk_tiles,
    int n_chunks, int k, int* __restrict__ top_idx, float* __restrict__ top_score,
    uint64_t* __restrict__ part) {
  constexpr int ES = code_bytes<ST>();
  constexpr int CPP = saki::kChunkBytes / ES;
  constexpr int NP = RK / CPP;
  constexpr size_t TB = (size_t)kTile * RK * ES;
  using KO = KeysF32;
  using K = KO::K;
  constexpr int D = saki::kHeadDim;
  constexpr int WM = kDecodeWaves, T = kDecodeTiles, CAP = decode_cap<R>();
  constexpr int NO = R * (RK + 1);  // sketch outputs of R rows
  extern __shared__ __align__(16) uint8_t area[];  // decode_area<RK, R>(W): sketch parts, lane maxima, online lists
  __shared__ float zs[R][RK + 1];                // element RK: the mean term b
  __shared__ __align__(16) uint32_t zw[R][RK / 2];  // pairs of bf16 elements
  __shared__ K buf[R][CAP];
  __shared__ int cnt[R];
  const int tid = threadIdx.x, W = blockDim.x / kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave), lane = lane_id();
  const long long lb = xcd_logical_block((long long)row_groups * n_chunks * n_bi);
  if (lb < 0) return;  // the whole work-group
  const int rg = (int)(lb % row_groups), ch = (int)((lb / row_groups) % n_chunks);
  const size_t bi = (size_t)(lb / ((long long)row_groups * n_chunks));  // b * index_heads + code set
  const int index_heads = H_q / gq;
  const size_t b = bi / index_heads;
  const int ih = (int)(bi % index_heads);
  const int n_rho = gq * Q;
  const int row0 = rg * R;
  int lim[R];
  size_t flat[R];  // (b * H_q + h) * Q + i of each row
  int kmax = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int rho = row0 + r;
    const bool ok = rho < n_rho;
    const int i = ok ? rho / gq : 0;
    flat[r] = (b * H_q + ih * gq + (ok ? rho % gq : 0)) * Q + i;
    lim[r] = ok ? row_limit(i, Q, N_valid, q_pos) : 0;
    kmax = max(kmax, lim[r]);
  }
  const int tbeg = ch * chunk_tiles, tend = min(tbeg + chunk_tiles, (int)saki::n_tiles(kmax));
  const uint8_t* hbase = index + bi * n_tiles * TB;
  // a tile's pieces are loaded two tiles ahead of their use (up to 64 bytes per
  // key, 128 where the registers allow; wider codes are loaded as they are used)
  constexpr int ZW = ST == kStF32 ? RK : RK / 2;  // words of a row's z
  constexpr bool kScalarZ = R * ZW <= 64;
  constexpr int PF = kScalarZ && (NP <= 4 || (NP <= 8 && R == 1 && ST != kStFp8)) ? NP : 0;
  struct Raw {
    uint4 v[PF ? PF : 1];
  };
  auto tile_ptr = [&](int t) { return hbase + (size_t)t * TB + (size_t)lane * 16; };
  auto load = [&](int t, Raw& x) {
    if constexpr (PF > 0) {
      if (t >= tend) return;
      const uint8_t* tb = tile_ptr(t);
#pragma unroll
      for (int p = 0; p < PF; ++p) x.v[p] = *reinterpret_cast<const uint4*>(tb + (size_t)p * kTile * 16);
    }
  };
  const int t_first = tbeg + wave;
  Raw ra, rb;
  load(t_first, ra);
  load(t_first + W, rb);

  // ---- the query sketch
  {
    constexpr int DB = D / WM;  // dims loaded at a time
    const int DS = D / W;
    float* zpart = reinterpret_cast<float*>(area);
    for (int o0 = 0; o0 < NO; o0 += kWave) {
      const int o = min(o0 + lane, NO - 1);
      const int r = R == 1 ? 0 : o / (RK + 1), m = o % (RK + 1);
      const int rho = min(row0 + r, n_rho - 1);
      const int h = ih * gq + rho % gq;
      const int stride = m < RK ? RK : 1;
      const float* qv = q + ((b * H_q + h) * Q + rho / gq) * D + wave * DS;
      const float* col = (m < RK ? Bq + (size_t)h * D * RK + m : mu + (size_t)(h / (H_q / H_kv)) * D) +
                         (size_t)wave * DS * stride;
      float acc = 0.f;
      for (int c0 = 0; c0 < DS; c0 += DB) {
        float qa[DB], ba[DB];
#pragma unroll
        for (int u = 0; u < DB; ++u) {
          qa[u] = qv[c0 + u];
          ba[u] = col[(size_t)(c0 + u) * stride];
        }
#pragma unroll
        for (int u = 0; u < DB; ++u) acc = fmaf(qa[u], ba[u], acc);
      }
      zpart[wave * NO + o] = acc;
    }
    if (tid < R) cnt[tid] = 0;
    __syncthreads();
    for (int o = tid; o < NO; o += W * kWave) {
      float v = zpart[o];
      for (int w = 1; w < W; ++w) v += zpart[w * NO + o];
      const int r = o / (RK + 1), m = o % (RK + 1);
      zs[r][m] = ST != kStF32 && m < RK ? bf16_round(v) : v;
    }
    __syncthreads();
  }
  // z (as pairs for bf16 and fp8 codes) in scalar registers when it fits (it is
  // the same in every lane), else read from LDS with the pieces
  uint32_t zp[kScalarZ ? R : 1][kScalarZ ? ZW : 1];
  if constexpr (ST == kStF32 && kScalarZ) {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int m = 0; m < RK; ++m)
        zp[r][m] = (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(zs[r][m]));
  } else if constexpr (ST != kStF32) {
    auto pair = [&](int r, int m) {
      return (__float_as_uint(zs[r][2 * m]) >> 16) | (__float_as_uint(zs[r][2 * m + 1]) & 0xffff0000u);
    };
    if constexpr (kScalarZ) {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int m = 0; m < RK / 2; ++m)
          zp[r][m] = (uint32_t)__builtin_amdgcn_readfirstlane((int)pair(r, m));
    } else {
      for (int o = tid; o < R * RK / 2; o += W * kWave) zw[o / (RK / 2)][o % (RK / 2)] = pair(o / (RK / 2), o % (RK / 2));
      __syncthreads();
    }
  }
  float bb[R];
#pragma unroll
  for (int r = 0; r < R; ++r) bb[r] = zs[r][RK];

  // scores of this lane's key of tile t < tend (-inf past a row's limit)
  auto score = [&](int t, const Raw& x, float* out) {
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.f;
    auto piece = [&](int p, const uint4& v) {
      if constexpr (ST == kStF32) {
        const float c[4] = {__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)};
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[r] = fmaf(kScalarZ ? __uint_as_float(zp[kScalarZ ? r : 0][kScalarZ ? 4 * p + e : 0]) : zs[r][4 * p + e],
                          c[e], acc[r]);
      } else {
        constexpr int WP = CPP / 2;  // words of bf16 pairs
        uint32_t w[WP];
        const uint32_t vv[4] = {v.x, v.y, v.z, v.w};
        if constexpr (ST == kStFp8) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint2 bw = e4m3x4_to_bf16(vv[e]);
            w[2 * e] = bw.x;
            w[2 * e + 1] = bw.y;
          }
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = vv[e];
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int e = 0; e < WP; ++e) {
            const uint32_t z = kScalarZ ? zp[kScalarZ ? r : 0][kScalarZ ? WP * p + e : 0] : zw[r][WP * p + e];
            acc[r] = __builtin_amdgcn_fdot2_f32_bf16(as_bf16x2(w[e]), as_bf16x2(z), acc[r], false);
          }
      }
    };
    if constexpr (PF > 0) {
#pragma unroll
      for (int p = 0; p < NP; ++p) piece(p, x.v[p]);
    } else {
      // pieces at a time: with z from LDS, at most 64 registers of it and at
      // least two rounds (a loop that is not unrolled, so that z is not kept)
      constexpr int PZ = std::min(64 / (R * (ST == kStFp8 ? 8 : 4)), NP / 2);
      constexpr int PB = kScalarZ ? std::min(NP, 8) : std::max(PZ, 1);
      const uint8_t* tb = tile_ptr(t);
      auto batch = [&](int p0) {
        uint4 v[PB];
#pragma unroll
        for (int p = 0; p < PB; ++p) v[p] = *reinterpret_cast<const uint4*>(tb + (size_t)(p0 + p) * kTile * 16);
#pragma unroll
        for (int p = 0; p < PB; ++p) piece(p0 + p, v[p]);
      };
      if constexpr (kScalarZ) {
#pragma unroll
        for (int p0 = 0; p0 < NP; p0 += PB) batch(p0);
      } else {
#pragma unroll 1
        for (int p0 = 0; p0 < NP; p0 += PB) batch(p0);
      }
    }
    const int j = t * kTile + lane;
#pragma unroll
    for (int r = 0; r < R; ++r) out[r] = j < lim[r] ? acc[r] + bb[r] : -INFINITY;
  };
  auto append = [&](int r, bool take, float sv, int t) {
    const uint64_t mask = __ballot(take);
    if (mask == 0) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(&cnt[r], __popcll(mask));
    at = __builtin_amdgcn_readfirstlane(at) + prefix_count(mask);
    if (take && at < CAP) buf[r][at] = KO::make(sv, t * kTile + lane);
  };

  // ---- the head
  float s[T][R];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const int t = t_first + i * W;
    if (t < tend) {
      score(t, (i & 1) ? rb : ra, s[i]);
      load(t + 2 * W, (i & 1) ? rb : ra);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) s[i][r] = -INFINITY;
    }
  }
  float thr[R];  // the gate (-inf: every key is a candidate)
#pragma unroll
  for (int r = 0; r < R; ++r) thr[r] = -INFINITY;
  if (tend - tbeg > CAP / kTile) {
    uint32_t* mx = reinterpret_cast<uint32_t*>(area);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float m = -INFINITY;  // a lane whose scores are no numbers has no part in the gate
#pragma unroll
      for (int i = 0; i < T; ++i) m = fmaxf(m, s[i][r]);
      uint32_t o = ord_f32(m);
      wave_sort<KeysU32>(o);
      mx[(r * W + wave) * kWave + lane] = o;
    }
    __syncthreads();
    merge_tree<KeysU32, R>(mx, W, W, wave, W, lane);
#pragma unroll
    for (int r = 0; r < R; ++r) thr[r] = unord_f32(mx[r * W * kWave + kWave - 1]);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // at or above the gate, compared as floats (a gate of +0 takes every zero); scores of -inf never
    const float least = thr[r] == -INFINITY ? -__FLT_MAX__ : thr[r];
#pragma unroll
    for (int i = 0; i < T; ++i) append(r, s[i][r] >= least, s[i][r], t_first + i * W);
  }

  // ---- the tail
  auto tail = [&](int t, Raw& x) {
    float v[R];
    score(t, x, v);
    load(t + 2 * W, x);
#pragma unroll
    for (int r = 0; r < R; ++r) append(r, v[r] > thr[r], v[r], t);
  };
  // the row's candidates -> sorted, the best 64 first (every wave takes part)
  auto most_candidates = [&]() {
    int n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) n = max(n, cnt[r]);
    return n;
  };
  auto sort_candidates = [&](int most) {
    const int segs = max(1, (most + kWave - 1) / kWave);
    for (int t = wave; t < R * segs; t += W) {
      const int r = t % R, at = (t / R) * kWave + lane;
      K x = at < cnt[r] ? buf[r][at] : KO::pad();
      wave_sort<KO>(x);
      buf[r][at] = x;
    }
    __syncthreads();
    merge_tree<KO, R>(&buf[0][0], CAP / kWave, segs, wave, W, lane);
  };
  const int round = W * kDecodeRound;
  for (int r0 = tbeg + W * T; r0 < tend; r0 += round) {
    for (int t = r0 + wave; t < min(tend, r0 + round); t += 2 * W) {
      tail(t, ra);
      if (t + W < tend) tail(t + W, rb);
    }
    if (r0 + round >= tend) break;
    __syncthreads();
    const int most = most_candidates();
    if (most > CAP) break;
    if (most > CAP / 2) {
      sort_candidates(most);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (cnt[r] >= kWave) thr[r] = fmaxf(thr[r], KO::score(buf[r][kWave - 1]));
      __syncthreads();  // every wave has read the counts
      if (tid < R) cnt[tid] = min(cnt[tid], kWave);
    }
    __syncthreads();  // before the next round's candidates
  }
  __syncthreads();

  auto out_row = [&](int r, K e) {
    if (row0 + r >= n_rho) return;
    if (n_chunks == 1) {
      if (lane < k) {
        const size_t o = flat[r] * k + lane;
        top_idx[o] = out_index<KO>(e);
        if (top_score) top_score[o] = KO::score(e);
      }
    } else {
      part[(flat[r] * n_chunks + ch) * kMaxK + lane] = e;
    }
  };
  const int most = most_candidates();
  if (most <= CAP) {
    sort_candidates(most);
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (wave == r) out_row(r, buf[r][lane]);
    return;
  }
  // ---- too many candidates: an online top-64 per wave, row by row
  K* lists = reinterpret_cast<K*>(area);  // [W][64], then the waves' buffers [W][64]
#pragma unroll 1
  for (int r = 0; r < R; ++r) {
    __syncthreads();
    RowLists<KO, 1> top;
    top.init(lists + wave * kWave, lists + (W + wave) * kWave);
    for (int t = t_first; t < tend; t += W) {
      float v[R];
      load(t, ra);
      score(t, ra, v);
      float sv = v[0];
#pragma unroll
      for (int x = 1; x < R; ++x) sv = x == r ? v[x] : sv;
      top.offer(0, sv, t * kTile + lane);
    }
    top.finish(0);
    __syncthreads();
    merge_tree<KO, 1>(lists, W, W, wave, W, lane);
#pragma unroll
    for (int x = 0; x < R; ++x)
      if (x == r && wave == 0) out_row(x, lists[lane]);
  }
}

// ---------------------------------------------------------------- sketch scoring, MFMA

// Query blocks of 16 rows per wave, the column count of the 16x16 MFMA tiles.
// A = 16 keys of the current tile (rows), B = the wave's 16 queries (columns),
// so each lane holds scores of one query (lane % 16) against 16 keys of every
// 64-key tile.  The scorer and the query-sketch prologue below serve the
// batched kernel (score_batch_kernel), the one-pass kernel for long rows
// (score_scan_kernel) and the exact-recall kernels.

// Pack 8 floats that already hold bf16 values into a bf16x8 operand.
__device__ __forceinline__ uint4 pack_bf16x8(const float* f) {
  uint4 u;
  u.x = (__float_as_uint(f[0]) >> 16) | (__float_as_uint(f[1]) & 0xffff0000u);
  u.y = (__float_as_uint(f[2]) >> 16) | (__float_as_uint(f[3]) & 0xffff0000u);
  u.z = (__float_as_uint(f[4]) >> 16) | (__float_as_uint(f[5]) & 0xffff0000u);
  u.w = (__float_as_uint(f[6]) >> 16) | (__float_as_uint(f[7]) & 0xffff0000u);
  return u;
}
__device__ __forceinline__ float xor_shfl_f32(float v, int m) {
  return __uint_as_float(xor_shfl_u32(__float_as_uint(v), m));
}
// Sum over the four lanes that share lane % 16.
__device__ __forceinline__ float sum_lane_groups(float v) {
  v += xor_shfl_f32(v, 16);
  return v + xor_shfl_f32(v, 32);
}

// Upper-tail standard normal quantile: z with P(X > z) = tail, tail in (0, 0.5]
// (Abramowitz & Stegun 26.2.23, absolute error below 4.5e-4).  Only used to
// predict where a row's 64th score lies.
__device__ __forceinline__ float normal_upper_quantile(float tail) {
  const float t = sqrtf(-2.f * __logf(tail));
  return t - (2.515517f + t * (0.802853f + t * 0.010328f)) /
                 (1.f + t * (1.432788f + t * (0.189269f + t * 0.001308f)));
}

constexpr int kBins = 64;
constexpr int kCollect = 128;
constexpr int kSampleTiles = 8;   // moments from at least this many tiles per chunk
constexpr float kWinLo = 1.25f;   // histogram window around the predicted 64th score (sd)
constexpr float kWinHi = 0.75f;
constexpr int kCandRow = kCollect + 1;  // padded row strides (LDS bank spread)
constexpr int kHistRow = kBins + 5;  // 64 bins, 4 private overflow slots, 1 pad
enum RowMode : int { kModeAll = 0, kModeHist = 1, kModeFallback = 2 };

// Scores of one 64-key tile for the wave's 16 queries: acc[sub][v] is query
// (lane % 16) against key t0 + 16*sub + 4*(lane/16) + v, plus `init` (the
// kernels set it to the row's mean term b).
// bf16 and fp8 codes run on the bf16 MFMA (fp8 widened exactly to bf16 in
// registers), float32 codes on the f32 MFMA.
template <int RK, int ST>
struct MfmaScorer {
  static constexpr bool SBF = ST != kStF32;  // bf16 operands
  static constexpr bool F8 = ST == kStFp8;
  static constexpr int NKB = (SBF && RK >= 32) ? RK / 32 : 1;
  static constexpr int NKF = SBF ? 1 : RK / 4;
  static constexpr size_t TB = (size_t)kTile * RK * code_bytes<ST>();
  bf16x8_t zb[NKB];
  i16x4_t zb4;
  float zf[NKF];
  float init = 0.f;  // accumulator start (this lane's query column)

  // zs: this lane's query sketch row (RK floats, bf16 values for bf16 / fp8 codes)
  __device__ void load_operand(const float* zs, int g) {
    if constexpr (SBF) {
      if constexpr (RK == 16) {
        uint2 u;
        u.x = (__float_as_uint(zs[4 * g + 0]) >> 16) | (__float_as_uint(zs[4 * g + 1]) & 0xffff0000u);
        u.y = (__float_as_uint(zs[4 * g + 2]) >> 16) | (__float_as_uint(zs[4 * g + 3]) & 0xffff0000u);
        zb4 = as_i16x4(u);
      } else {
#pragma unroll
        for (int kk = 0; kk < NKB; ++kk) zb[kk] = as_bf16x8(pack_bf16x8(zs + 32 * kk + 8 * g));
      }
    } else {
#pragma unroll
      for (int m = 0; m < RK / 16; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e) zf[4 * m + e] = zs[4 * (g + 4 * m) + e];
    }
  }

  // zr: this lane's query sketch row as query_sketch_kernel writes it (RK
  // bf16 values for bf16 / fp8 codes, RK floats for float32 codes)
  __device__ void load_operand_row(const uint8_t* zr, int g) {
    if constexpr (SBF) {
      if constexpr (RK == 16) {
        zb4 = as_i16x4(*reinterpret_cast<const uint2*>(zr + 8 * g));
      } else {
#pragma unroll
        for (int kk = 0; kk < NKB; ++kk)
          zb[kk] = as_bf16x8(*reinterpret_cast<const uint4*>(zr + 2 * (32 * kk + 8 * g)));
      }
    } else {
#pragma unroll
      for (int m = 0; m < RK / 16; ++m) {
        const float4 v = *reinterpret_cast<const float4*>(zr + 4 * (4 * (g + 4 * m)));
        zf[4 * m] = v.x;
        zf[4 * m + 1] = v.y;
        zf[4 * m + 2] = v.z;
        zf[4 * m + 3] = v.w;
      }
    }
  }

  // raw operands of one tile: NL 16-byte loads per 16-key sub-block
  static constexpr int NL = SBF ? (RK == 16 ? 1 : RK / 32) : RK / 16;
  struct Raw {
    uint4 v[4][NL];
  };
  // the next tile is loaded while the current one is scored when its raw
  // operands fit in 32 registers (in for_tiles_deep 64, see there)
  static constexpr bool kPrefetch = 4 * NL <= 8;
  static constexpr bool kPrefetchWide = 4 * NL <= 16;
  // scores good to a bf16 rounding of both operands from the bf16 MFMA
  static constexpr bool kApprox = !SBF && RK >= 32;

  __device__ __forceinline__ void load(const uint8_t* tb, int qi, int g, Raw& r) const {
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      const int key = 16 * sub + qi;
      if constexpr (F8 && RK == 16) {  // dims 4g .. 4g+3: bytes 4g.. of piece 0
        const uint32_t raw = *reinterpret_cast<const uint32_t*>(tb + (size_t)key * 16 + 4 * g);
        r.v[sub][0] = uint4{raw, 0u, 0u, 0u};
      } else if constexpr (F8) {  // dims 32kk + 8g .. +7: piece 2kk + g/2, bytes 8(g%2)..
#pragma unroll
        for (int kk = 0; kk < NL; ++kk) {
          const uint2 raw = *reinterpret_cast<const uint2*>(
              tb + (size_t)(2 * kk + g / 2) * kTile * 16 + (size_t)key * 16 + (g % 2) * 8);
          r.v[sub][kk] = uint4{raw.x, raw.y, 0u, 0u};
        }
      } else if constexpr (SBF && RK == 16) {
        const uint2 raw = *reinterpret_cast<const uint2*>(tb + (size_t)(g / 2) * kTile * 16 +
                                                         (size_t)key * 16 + (g % 2) * 8);
        r.v[sub][0] = uint4{raw.x, raw.y, 0u, 0u};
      } else if constexpr (SBF) {
#pragma unroll
        for (int kk = 0; kk < NL; ++kk)
          r.v[sub][kk] = *reinterpret_cast<const uint4*>(tb + (size_t)(4 * kk + g) * kTile * 16 +
                                                         (size_t)key * 16);
      } else {
#pragma unroll
        for (int m = 0; m < NL; ++m)
          r.v[sub][m] = *reinterpret_cast<const uint4*>(tb + (size_t)(g + 4 * m) * kTile * 16 +
                                                        (size_t)key * 16);
      }
    }
  }

  __device__ __forceinline__ void mma(const Raw& r, f32x4_t acc[4]) const {
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      f32x4_t a = {init, init, init, init};
      if constexpr (F8 && RK == 16) {
        a = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_i16x4(e4m3x4_to_bf16(r.v[sub][0].x)), zb4,
                                                     a, 0, 0, 0);
      } else if constexpr (F8) {
#pragma unroll
        for (int kk = 0; kk < NL; ++kk) {
          const uint2 w0 = e4m3x4_to_bf16(r.v[sub][kk].x), w1 = e4m3x4_to_bf16(r.v[sub][kk].y);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(uint4{w0.x, w0.y, w1.x, w1.y}),
                                                      zb[kk], a, 0, 0, 0);
        }
      } else if constexpr (SBF && RK == 16) {
        a = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(as_i16x4(uint2{r.v[sub][0].x, r.v[sub][0].y}),
                                                     zb4, a, 0, 0, 0);
      } else if constexpr (SBF) {
#pragma unroll
        for (int kk = 0; kk < NL; ++kk)
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(r.v[sub][kk]), zb[kk], a, 0, 0, 0);
      } else {
#pragma unroll
        for (int m = 0; m < NL; ++m) {
          const uint4 raw = r.v[sub][m];
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(raw.x), zf[4 * m + 0], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(raw.y), zf[4 * m + 1], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(raw.z), zf[4 * m + 2], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(raw.w), zf[4 * m + 3], a, 0, 0, 0);
        }
      }
      acc[sub] = a;
    }
  }

  // The same for float32 codes with both operands rounded to bf16: a step of
  // the bf16 MFMA takes dims 32 kk + 4 g .. + 3 and 32 kk + 16 + 4 g .. + 3 of
  // lane group g, two of the raw pieces, in a 16th of the float32 MFMA's time.
  __device__ __forceinline__ void mma_approx(const Raw& r, f32x4_t acc[4]) const {
    if constexpr (kApprox) {
      bf16x8_t z[RK / 32];
#pragma unroll
      for (int kk = 0; kk < RK / 32; ++kk)
        z[kk] = as_bf16x8(uint4{bf16x2_bits(zf[8 * kk], zf[8 * kk + 1]), bf16x2_bits(zf[8 * kk + 2], zf[8 * kk + 3]),
                                bf16x2_bits(zf[8 * kk + 4], zf[8 * kk + 5]), bf16x2_bits(zf[8 * kk + 6], zf[8 * kk + 7])});
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        f32x4_t a = {init, init, init, init};
#pragma unroll
        for (int kk = 0; kk < RK / 32; ++kk) {
          const uint4 x = r.v[sub][2 * kk], y = r.v[sub][2 * kk + 1];
          auto two = [](uint32_t lo, uint32_t hi) { return bf16x2_bits(__uint_as_float(lo), __uint_as_float(hi)); };
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              as_bf16x8(uint4{two(x.x, x.y), two(x.z, x.w), two(y.x, y.y), two(y.z, y.w)}), z[kk], a, 0, 0, 0);
        }
        acc[sub] = a;
      }
    } else {
      mma(r, acc);
    }
  }

  // body(t0, acc) for the tiles t0 = t_beg, t_beg + step, ... < t_end
  template <class F>
  __device__ __forceinline__ void for_tiles(const uint8_t* hbase, int t_beg, int t_end, int step,
                                            int qi, int g, F&& body) const {
    if constexpr (kPrefetch) {
      // two register buffers taken in turn; the load past the last tile is
      // clamped to it (a valid, unused reload) so that no load is conditional
      if (t_beg >= t_end) return;
      const int last = t_beg + ((t_end - 1 - t_beg) / step) * step;
      auto at = [&](int t) { return hbase + (size_t)(min(t, last) / kTile) * TB; };
      Raw ra, rb;
      load(at(t_beg), qi, g, ra);
      for (int t0 = t_beg; t0 < t_end; t0 += 2 * step) {
        load(at(t0 + step), qi, g, rb);
        f32x4_t acc[4];
        mma(ra, acc);
        body(t0, acc);
        if (t0 + step >= t_end) break;
        load(at(t0 + 2 * step), qi, g, ra);
        mma(rb, acc);
        body(t0 + step, acc);
      }
    } else {
      for (int t0 = t_beg; t0 < t_end; t0 += step) {
        Raw cur;
        load(hbase + (size_t)(t0 / kTile) * TB, qi, g, cur);
        f32x4_t acc[4];
        mma(cur, acc);
        body(t0, acc);
      }
    }
  }

  // body(t0, acc) for every tile of [t_beg, t_end) in order, with the loads
  // of the next DEPTH - 1 tiles in flight while one is scored (a ring of
  // DEPTH register buffers) when a tile's operands fit in 32 registers, of the
  // next one when they fit in 64; otherwise as for_tiles.  Loads past the last
  // tile are clamped to it.  APPROX: scores of mma_approx.
  template <int DEPTH = 3, bool APPROX = false, class F>
  __device__ __forceinline__ void for_tiles_deep(const uint8_t* hbase, int t_beg, int t_end,
                                                 int qi, int g, F&& body) const {
    auto form = [&](const Raw& r, f32x4_t* acc) {
      if constexpr (APPROX)
        mma_approx(r, acc);
      else
        mma(r, acc);
    };
    if (t_beg >= t_end) return;
    if constexpr (kPrefetchWide) {
      constexpr int N = kPrefetch ? DEPTH : 2;
      const int last = t_beg + ((t_end - 1 - t_beg) / kTile) * kTile;
      auto at = [&](int t) { return hbase + (size_t)(min(t, last) / kTile) * TB; };
      Raw r[N];
#pragma unroll
      for (int d = 0; d + 1 < N; ++d) load(at(t_beg + d * kTile), qi, g, r[d]);
      for (int t0 = t_beg;; t0 += N * kTile) {
#pragma unroll
        for (int d = 0; d < N; ++d) {
          const int t = t0 + d * kTile;
          load(at(t + (N - 1) * kTile), qi, g, r[(d + N - 1) % N]);
          f32x4_t acc[4];
          form(r[d], acc);
          body(t, acc);
          if (t + kTile >= t_end) return;
        }
      }
    } else {
      for (int t0 = t_beg; t0 < t_end; t0 += kTile) {
        Raw cur;
        load(hbase + (size_t)(t0 / kTile) * TB, qi, g, cur);
        f32x4_t acc[4];
        form(cur, acc);
        body(t0, acc);
      }
    }
  }
};

// The query sketch of a wave's 16 rows (lane (qi, g) = lane % 16, lane / 16)
// on the f32 MFMA: D[m][qi] = sum_c B_q[c][m] q[qi][c] with lane group g
// feeding dims c = 4s + g, rounded to bf16 for bf16 and fp8 codes and staged
// through zs (16 x RK floats of LDS) into the scorer's operand.  Returns
// b = q . mu of row qi (the same in its four lanes).  qr: row qi's query (any
// valid row when !row_ok, whose query counts as zero).
template <int RK, int ST>
__device__ __forceinline__ float mfma_query_sketch(const float* __restrict__ qr, bool row_ok,
                                                   const float* __restrict__ bq,
                                                   const float* __restrict__ mr, float* zs, int qi,
                                                   int g, MfmaScorer<RK, ST>& sc) {
  constexpr int D = saki::kHeadDim;
  f32x4_t za[RK / 16];
#pragma unroll
  for (int mb = 0; mb < RK / 16; ++mb) za[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float bp = 0.f;
  // the loads of SB steps are issued together, then their products taken
  constexpr int SB = RK <= 32 ? 16 : RK <= 64 ? 8 : 4;
#pragma unroll 1
  for (int s0 = 0; s0 < D / 4; s0 += SB) {
    float qa[SB], ma[SB], ba[SB][RK / 16];
#pragma unroll
    for (int u = 0; u < SB; ++u) {
      const int c = 4 * (s0 + u) + g;
      qa[u] = qr[c];
      ma[u] = mr[c];
#pragma unroll
      for (int mb = 0; mb < RK / 16; ++mb) ba[u][mb] = bq[c * RK + 16 * mb + qi];
    }
#pragma unroll
    for (int u = 0; u < SB; ++u) {
      const float qv = row_ok ? qa[u] : 0.f;
      bp = fmaf(qv, ma[u], bp);
#pragma unroll
      for (int mb = 0; mb < RK / 16; ++mb)
        za[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ba[u][mb], qv, za[mb], 0, 0, 0);
    }
  }
  const float b = sum_lane_groups(bp);
#pragma unroll
  for (int mb = 0; mb < RK / 16; ++mb)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float zv = za[mb][v];
      zs[qi * RK + 16 * mb + 4 * g + v] = ST != kStF32 ? bf16_round(zv) : zv;
    }
  wave_lds_sync();
  sc.load_operand(zs + qi * RK, g);
  wave_lds_sync();
  return b;
}

// ---------------------------------------------------------------- query sketches of a batch of rows

// query_sketch_kernel: z = B_q^T q and b = q . mu (equation (5): the query
// side of the factored score) of every row, written once so that the
// two-pass scoring kernel loads each wave's 16 rows as one contiguous block.
// z is rounded to bf16 for bf16 and fp8 codes (the MFMA operand) and kept in
// float32 for float32 codes; row layout zq[(bh * Q + i) * RK + m], b[bh * Q + i].
// The f32 MFMA forms D[m][qi] = sum_c B_q[c][m] q[qi][c]: lane (qi, g) loads
// q[qi][16j + 4g .. 16j + 4g + 3] for j = 0..7 as float4 (each row read as
// 64-byte runs) and feeds dims c = 16j + 4g + e at step 4j + e.  B_q of the
// head waits in LDS in that operand order, one float4 per (j, mb) and lane.
// grid: 1-D, work-group (bh, part) covers rows [part * rows_per, ...) of (b, h).
// Few long heads are cut into shorter parts so that every CU has some: the
// 32 x 4,032 rows of a layer take 10 us in 512 parts, 32 us in 128 of 1,024 rows.
constexpr int kQsWaves = 4;
constexpr int kQsRows = 1024;   // rows per work-group, at most
constexpr int kQsGroups = 512;  // work-groups wanted before a work-group takes more than 64 rows

template <int RK, int ST>
__global__ __launch_bounds__(kQsWaves * kWave) void query_sketch_kernel(
    const float* __restrict__ q, const float* __restrict__ Bq, const float* __restrict__ mu,
    int Q, int H_q, int H_kv, int n_bh, int parts, int rows_per, uint8_t* __restrict__ zq,
    float* __restrict__ bout) {
  constexpr int D = saki::kHeadDim;
  constexpr int MB = RK / 16;
  __shared__ __align__(16) float bl[D * RK];
  const long long lb = xcd_logical_block((long long)n_bh * parts);
  if (lb < 0) return;
  const size_t bh = (size_t)(lb / parts);
  const int part = (int)(lb % parts);
  const int h = (int)(bh % H_q);
  const int gkv = h / (H_q / H_kv);
  // B_q[h] (row-major D x RK) -> bl[((j * MB + mb) * 64 + 16 g + qi) * 4 + e]
  // = B_q[16j + 4g + e][16mb + qi]
  const float* bsrc = Bq + (size_t)h * D * RK;
  for (int i = threadIdx.x; i < D * RK; i += kQsWaves * kWave) {
    const int c = i / RK, m = i % RK;
    bl[(((c / 16) * MB + m / 16) * 64 + 16 * ((c % 16) / 4) + m % 16) * 4 + c % 4] = bsrc[i];
  }
  __syncthreads();
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int qi = lane % 16, g = lane / 16;
  const float* mr = mu + (size_t)gkv * D;
  float4 mv[8];  // this lane's dims of mu
#pragma unroll
  for (int j = 0; j < 8; ++j) mv[j] = *reinterpret_cast<const float4*>(mr + 16 * j + 4 * g);
  const int r_end = min(Q, (part + 1) * rows_per);
  for (int row0 = part * rows_per + wave * kMR; row0 < r_end; row0 += kQsWaves * kMR) {
    const int row = row0 + qi;
    const bool ok = row < r_end;
    const float* qr = q + (bh * Q + (ok ? row : row0)) * D;
    float4 qv[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      qv[j] = *reinterpret_cast<const float4*>(qr + 16 * j + 4 * g);
      if (!ok) qv[j] = float4{0.f, 0.f, 0.f, 0.f};
    }
    float bp = 0.f;
    f32x4_t za[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) za[mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      bp = fmaf(qv[j].x, mv[j].x, bp);
      bp = fmaf(qv[j].y, mv[j].y, bp);
      bp = fmaf(qv[j].z, mv[j].z, bp);
      bp = fmaf(qv[j].w, mv[j].w, bp);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const float4 a = *reinterpret_cast<const float4*>(bl + ((j * MB + mb) * 64 + lane) * 4);
        za[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, qv[j].x, za[mb], 0, 0, 0);
        za[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, qv[j].y, za[mb], 0, 0, 0);
        za[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, qv[j].z, za[mb], 0, 0, 0);
        za[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, qv[j].w, za[mb], 0, 0, 0);
      }
    }
    const float b = sum_lane_groups(bp);
    if (!ok) continue;
    const size_t base = (bh * Q + row) * RK;
    // lane (qi, g) holds z[row][16mb + 4g + v], v = 0..3
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      if constexpr (ST != kStF32) {
        const uint2 u{bf16_bits(za[mb][0]) | (bf16_bits(za[mb][1]) << 16),
                      bf16_bits(za[mb][2]) | (bf16_bits(za[mb][3]) << 16)};
        *reinterpret_cast<uint2*>(zq + (base + 16 * mb + 4 * g) * 2) = u;
      } else {
        *reinterpret_cast<float4*>(zq + (base + 16 * mb + 4 * g) * 4) =
            float4{za[mb][0], za[mb][1], za[mb][2], za[mb][3]};
      }
    }
    if (g == 0) bout[bh * Q + row] = b;
  }
}

// ---------------------------------------------------------------- sketch scoring, MFMA, block-maximum gate

// score_batch_kernel: one wave per work-group (its LDS is released the moment
// it ends, where a wave of a larger work-group would hold its slot until the
// slowest of its siblings ends), each with a block of 16 query rows and that
// block's keys of one chunk (at most 4,096 keys), and the exact top-64 per row
// in two passes over the codes (the MFMA recomputes the scores in the second).  Rows are ranked by s' = z . c: b is
// the same for all keys of a row and is added to the 64 kept scores.
//   A. each lane records the maxima of its keys in blocks of 8, 4, 2 or 1
//      keys, the size set by the wave's longest row (at least 2,048, 1,024,
//      512 keys, or fewer), so that a row of at least about 256 keys has
//      about 256 blocks or more and the rows of a wave below 512 keys have
//      one block per key.  A maximum is stored as the top 16 bits of its
//      ordered float32 bits, which rounds it down.
//   threshold: per row, a histogram of the stored maxima over 64 equal bins
//      of score around the predicted 64th largest (from their mean and
//      spread and a normal quantile; moved above or below when the crossing
//      falls outside) gives tau, the lower edge of the bin below the highest
//      bin whose count from the top reaches 64.  At least 64 blocks then
//      have a maximum >= tau, so at least 64 keys score >= tau and all of
//      the row's top-64 do; with 256 blocks or more about 64-90 keys pass.
//      A row with fewer than 64 blocks keeps every key.
//   B. every key that scores >= tau goes to its lane's candidate slots (39
//      per lane usable, 156 per row), and the row's count is checked to be
//      >= 64.
// With that check any tau is safe, so pass A may take rounded scores: float32
// codes of 32 and more dims go through the bf16 MFMA there (the float32 one
// bounds this kernel for them: at r = 64, 64 instructions of 32 clocks a tile
// against 8 of 16).
// The candidates are then sorted by a bitonic network that holds 16 entries
// per lane, and the best 64 are kept.  A row whose candidates overflow its
// slots (many equal scores, or rows of very different lengths in one wave)
// or fall short sends its wave to the online selection of saki_topk.h.

constexpr int kBWaves = saki::kBatchWaves;  // independent waves per work-group
constexpr int kBEnt = 512;                 // block-maximum entries per row
constexpr int kBBins = 64;                 // histogram bins per row
constexpr int kBSlots = 40;                // candidate slots per lane
constexpr int kBDepth = 3;                 // code tiles whose loads are in flight, plus one
constexpr int kBWaveBytes = kMR * 4 * kBSlots * 8;  // 20 KiB of LDS per wave
static_assert(saki::kBatchMaxChunk / 8 <= kBEnt, "a chunk's 8-key blocks fit");
static_assert(kMR * kBEnt * 2 + kMR * kBBins * 4 <= kBWaveBytes, "entries and bins fit");
static_assert(kMR * kTile * 4 + 2 * (kMR / 2) * kList * 8 <= kBWaveBytes, "fallback fits");

// Top 16 bits of the ordered float32 bits: rounds down, finite values map to
// 0x0080 and above, and -inf (a masked key) to 0.
__device__ __forceinline__ uint32_t ord16(float x) {
  return x == -INFINITY ? 0u : (ord_f32(x) >> 16);
}
// The float an entry stands for (at most the maximum it was taken from).
__device__ __forceinline__ float unord16(uint32_t v) { return unord_f32(v << 16); }
// ord16(a) | ord16(b) << 16 for finite a and b.
__device__ __forceinline__ uint32_t pack_ord16(float a, float b) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  const uint32_t oa = ua ^ ((uint32_t)((int32_t)ua >> 31) | 0x80000000u);
  const uint32_t ob = ub ^ ((uint32_t)((int32_t)ub >> 31) | 0x80000000u);
  return __builtin_amdgcn_perm(ob, oa, 0x07060302u);  // bytes 2, 3 of oa, then of ob
}

// Bitonic sort of one row's 64 entries held 16 per lane by the row's four
// lanes (lane groups g = lane / 16): entry e = 16 g + i is x[i] of lane group
// g.  Leaves the entries in descending order of e.
template <class KO>
__device__ __forceinline__ void sort64_x16(typename KO::K (&x)[16], int g) {
  using K = typename KO::K;
#pragma unroll
  for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
    for (int m = k >> 1; m > 0; m >>= 1) {
      if (m >= 16) {  // partner in lane group g ^ (m / 16): lane xor m
        const bool lower = (g & (m >> 4)) == 0;
        const bool desc = k == 64 || (g & (k >> 4)) == 0;
        const bool keep_better = lower == desc;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const K o = KO::shfl_xor(x[i], m);
          x[i] = KO::sel(KO::gt(x[i], o) == keep_better, x[i], o);
        }
      } else {  // partner in the same lane
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          if (i & m) continue;
          const int j = i | m;
          const bool desc = k >= 64 ? true : k >= 16 ? (g & (k >> 4)) == 0 : (i & k) == 0;
          const K a = x[i], b = x[j];
          const bool sw = KO::gt(a, b) != desc;  // the lower position takes the better when descending
          x[i] = KO::sel(sw, b, a);
          x[j] = KO::sel(sw, a, b);
        }
      }
    }
  }
}

// x <- the best 64 of x and y (both sorted descending as left by sort64_x16).
template <class KO>
__device__ __forceinline__ void merge64_x16(typename KO::K (&x)[16], const typename KO::K (&y)[16],
                                            int g) {
  using K = typename KO::K;
  // entry e against y's entry 63 - e = 16 (3 - g) + (15 - i): lane group g ^ 3
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const K r = KO::shfl_xor(KO::shfl_xor(y[15 - i], 16), 32);
    x[i] = KO::sel(KO::gt(r, x[i]), r, x[i]);
  }
  // x is now bitonic: half-cleaners, all descending
#pragma unroll
  for (int m = 32; m >= 16; m >>= 1) {
    const bool lower = (g & (m >> 4)) == 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const K o = KO::shfl_xor(x[i], m);
      x[i] = KO::sel(KO::gt(x[i], o) == lower, x[i], o);
    }
  }
#pragma unroll
  for (int m = 8; m > 0; m >>= 1) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i & m) continue;
      const int j = i | m;
      const K a = x[i], b = x[j];
      const bool sw = KO::gt(b, a);
      x[i] = KO::sel(sw, b, a);
      x[j] = KO::sel(sw, a, b);
    }
  }
}

// ---- 32-bit keys, 64 per row held 16 per lane as in sort64_x16

__device__ __forceinline__ uint32_t umax32(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t umin32(uint32_t a, uint32_t b) { return a < b ? a : b; }
// a takes the larger key, b the smaller
__device__ __forceinline__ void cx_u32(uint32_t& a, uint32_t& b) {
  const uint32_t hi = umax32(a, b);
  b = umin32(a, b);
  a = hi;
}
// Compare-exchange of entry X of lane groups g and g ^ (M / 16), and the same
// for entry Y; the lower lane group keeps the larger key.  The first permlane
// swap hands every lane one such pair (of X in half of the lane groups, of Y
// in the others), and the second sends the larger and the smaller back.
template <int M>
__device__ __forceinline__ void cx_rows_u32(uint32_t& X, uint32_t& Y) {
  if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(X, Y, false, false);
    const auto t = __builtin_amdgcn_permlane16_swap(umax32(r[0], r[1]), umin32(r[0], r[1]), false, false);
    X = t[0];
    Y = t[1];
  } else {
    const auto r = __builtin_amdgcn_permlane32_swap(X, Y, false, false);
    const auto t = __builtin_amdgcn_permlane32_swap(umax32(r[0], r[1]), umin32(r[0], r[1]), false, false);
    X = t[0];
    Y = t[1];
  }
}
// Stages m = 8, 4, 2, 1 of a descending bitonic merge inside each lane.
__device__ __forceinline__ void lane_merge_desc_u32(uint32_t (&x)[16]) {
#pragma unroll
  for (int m = 8; m > 0; m >>= 1)
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (!(i & m)) cx_u32(x[i], x[i | m]);
}
// Bitonic sort of one row's 64 keys into descending order of e = 16 g + i.
// Blocks whose direction depends on the lane group (levels 16 and 32) are
// sorted as complemented keys, so every stage there is descending.
__device__ __forceinline__ void sort64_u32(uint32_t (&x)[16], int g) {
#pragma unroll
  for (int k = 2; k <= 8; k <<= 1)
#pragma unroll
    for (int m = k >> 1; m > 0; m >>= 1)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i & m) continue;
        if ((i & k) == 0)
          cx_u32(x[i], x[i | m]);
        else
          cx_u32(x[i | m], x[i]);
      }
  const uint32_t c1 = (g & 1) ? ~0u : 0u, c2 = (g & 2) ? ~0u : 0u;
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] ^= c1;
  lane_merge_desc_u32(x);  // level 16
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] ^= c1 ^ c2;
#pragma unroll
  for (int i = 0; i < 16; i += 2) cx_rows_u32<16>(x[i], x[i + 1]);  // level 32
  lane_merge_desc_u32(x);
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] ^= c2;
#pragma unroll
  for (int i = 0; i < 16; i += 2) cx_rows_u32<32>(x[i], x[i + 1]);  // level 64
#pragma unroll
  for (int i = 0; i < 16; i += 2) cx_rows_u32<16>(x[i], x[i + 1]);
  lane_merge_desc_u32(x);
}
// x <- the best 64 of x (descending) and y (ascending); dmax <- the largest
// key left out so far.  The elementwise maxima form a bitonic sequence.
__device__ __forceinline__ void merge64_u32(uint32_t (&x)[16], const uint32_t (&y)[16],
                                            uint32_t& dmax) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    dmax = umax32(dmax, umin32(x[i], y[i]));
    x[i] = umax32(x[i], y[i]);
  }
#pragma unroll
  for (int i = 0; i < 16; i += 2) cx_rows_u32<32>(x[i], x[i + 1]);
#pragma unroll
  for (int i = 0; i < 16; i += 2) cx_rows_u32<16>(x[i], x[i + 1]);
  lane_merge_desc_u32(x);
}

// grid: 1-D, 8 * ceil(groups * n_chunks * n_bh / 8) work-groups of kBWaves
// waves; work-group (bh, chunk, group) takes the 16-row blocks kBWaves * group
// .. kBWaves * group + kBWaves - 1 of (sequence, head) bh, the longest causal
// rows first.
template <int RK, int ST>
__global__ __launch_bounds__(kBWaves * kWave) void score_batch_kernel(
    const uint8_t* __restrict__ index, int n_tiles, int N_valid, int Q,
    const int* __restrict__ q_pos, const uint8_t* __restrict__ zq,
    const float* __restrict__ zb, int H_q, int gq, int n_bh, int groups, int chunk,
    int n_chunks, int k, int* __restrict__ top_idx, float* __restrict__ top_score,
    uint64_t* __restrict__ part) {
  constexpr int D = saki::kHeadDim;
  using KO = KeysF32;
  using K = uint64_t;
  using Scorer = MfmaScorer<RK, ST>;
  __shared__ __align__(16) uint8_t lds_mem[kBWaves][kBWaveBytes];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const long long lb = xcd_logical_block((long long)groups * n_chunks * n_bh);
  if (lb < 0) return;
  const int gb = groups - 1 - (int)(lb % groups);
  const int ch = (int)((lb / groups) % n_chunks);
  const size_t bh = (size_t)(lb / ((long long)groups * n_chunks));
  const int h = (int)(bh % H_q);
  const int row0 = (gb * kBWaves + wave) * kMR;
  if (row0 >= Q) return;  // the waves never synchronise with each other
  const int qi = lane % 16, g = lane / 16;
  const int my_row = row0 + qi;
  const bool row_ok = my_row < Q;
  const int my_lim = row_limit(my_row, Q, N_valid, q_pos);  // 0 for rows past Q
  const int kmax = wave_max_i(my_lim);
  const int kmin = wave_min_i(my_lim);
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  uint8_t* wl = lds_mem[wave];

  // ---- query sketch, formed by query_sketch_kernel.  b = q . mu is the same
  // for every key of a row, so the selection ranks s' = z . c (accumulators
  // starting at zero) and b is added to the 64 scores that are kept.
  Scorer sc;
  const size_t zrow = bh * Q + (row_ok ? my_row : row0);
  sc.load_operand_row(zq + zrow * RK * (ST != kStF32 ? 2 : 4), g);
  const float my_b = zb[zrow];
  const size_t code_set = (bh / H_q) * (H_q / gq) + h / gq;
  const uint8_t* hbase = index + code_set * n_tiles * Scorer::TB;

  // keys past a row's limit score -inf (tiles crossing some row's limit only)
  auto mask_tile = [&](int t0, f32x4_t* acc) {
    if (t0 + kTile > kmin) {
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (t0 + 16 * sub + 4 * g + v >= my_lim) acc[sub][v] = -INFINITY;
    }
  };

  // ---- pass A: block maxima of this lane's keys
  const int n_row = max(0, min(my_lim, kend) - kbeg);
  const int row_tiles = (n_row + kTile - 1) / kTile;
  // entries of one lane per tile: 2, 4, 8 or 16 blocks of 8, 4, 2 or 1 keys,
  // by the wave's longest row (kend - kbeg keys), so that no row has more
  // than kBEnt entries
  const int n_wave = kend - kbeg;
  const int lane_ent = n_wave >= 2048 ? 2 : n_wave >= 1024 ? 4 : n_wave >= 512 ? 8 : 16;
  // row qi's entries and histogram bins have their 16-byte groups permuted
  // (word offset xor 4 qi), so that the rows' accesses spread over the banks
  uint32_t* ent = reinterpret_cast<uint32_t*>(wl) + qi * (kBEnt / 2);
  const int sw = 4 * qi;
  float bsum = 0.f, bsq = 0.f, bmax = -INFINITY, bmin = INFINITY, bcnt = 0.f;
  auto stat = [&](float x) {  // x: a block maximum (-inf: no key of the row)
    const bool ok = x != -INFINITY;
    const float y = ok ? x : 0.f;
    bcnt += ok ? 1.f : 0.f;
    bsum += y;
    bsq = fmaf(y, y, bsq);
    bmax = vmax(bmax, x);
    bmin = ok ? vmin(bmin, x) : bmin;
  };
  sc.template for_tiles_deep<kBDepth, Scorer::kApprox>(hbase, kbeg, kend, qi, g, [&](int t0, f32x4_t* acc) {
    const int tl = (t0 - kbeg) / kTile;
    const int wo = (tl * 4 * lane_ent + g * lane_ent) / 2;  // this lane's first word
    if (t0 + kTile <= kmin && lane_ent <= 4) {
      // every key of the tile lies below every row's limit: no -inf
      if (lane_ent == 2) {
        const float a = vmax(vmax(vmax(acc[0][0], acc[0][1]), vmax(acc[0][2], acc[0][3])),
                             vmax(vmax(acc[1][0], acc[1][1]), vmax(acc[1][2], acc[1][3])));
        const float b = vmax(vmax(vmax(acc[2][0], acc[2][1]), vmax(acc[2][2], acc[2][3])),
                             vmax(vmax(acc[3][0], acc[3][1]), vmax(acc[3][2], acc[3][3])));
        ent[wo ^ sw] = pack_ord16(a, b);
        bsum += a + b;
        bsq = fmaf(a, a, fmaf(b, b, bsq));
        bmax = vmax(bmax, vmax(a, b));
        bmin = vmin(bmin, vmin(a, b));
        bcnt += 2.f;
      } else {
        float m4[4];
#pragma unroll
        for (int sub = 0; sub < 4; ++sub)
          m4[sub] = vmax(vmax(acc[sub][0], acc[sub][1]), vmax(acc[sub][2], acc[sub][3]));
        *reinterpret_cast<uint2*>(ent + (wo ^ sw)) = uint2{pack_ord16(m4[0], m4[1]), pack_ord16(m4[2], m4[3])};
        bsum += (m4[0] + m4[1]) + (m4[2] + m4[3]);
        bsq = fmaf(m4[0], m4[0], fmaf(m4[1], m4[1], fmaf(m4[2], m4[2], fmaf(m4[3], m4[3], bsq))));
        bmax = vmax(vmax(bmax, vmax(m4[0], m4[1])), vmax(m4[2], m4[3]));
        bmin = vmin(vmin(bmin, vmin(m4[0], m4[1])), vmin(m4[2], m4[3]));
        bcnt += 4.f;
      }
      return;
    }
    mask_tile(t0, acc);
    if (tl >= row_tiles) return;  // nothing of this row: no entries
    float m2[8];  // maxima of the pairs (sub, v = 0..1), (sub, v = 2..3)
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      m2[2 * sub] = vmax(acc[sub][0], acc[sub][1]);
      m2[2 * sub + 1] = vmax(acc[sub][2], acc[sub][3]);
    }
    if (lane_ent == 2) {
      const float a = vmax(vmax(m2[0], m2[1]), vmax(m2[2], m2[3]));
      const float b = vmax(vmax(m2[4], m2[5]), vmax(m2[6], m2[7]));
      ent[wo ^ sw] = ord16(a) | (ord16(b) << 16);
      stat(a);
      stat(b);
    } else if (lane_ent == 4) {
      uint32_t u[4];
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        const float m4 = vmax(m2[2 * sub], m2[2 * sub + 1]);
        u[sub] = ord16(m4);
        stat(m4);
      }
      *reinterpret_cast<uint2*>(ent + (wo ^ sw)) = uint2{u[0] | (u[1] << 16), u[2] | (u[3] << 16)};
    } else if (lane_ent == 8) {
      uint32_t u[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        u[j] = ord16(m2[j]);
        stat(m2[j]);
      }
      *reinterpret_cast<uint4*>(ent + (wo ^ sw)) =
          uint4{u[0] | (u[1] << 16), u[2] | (u[3] << 16), u[4] | (u[5] << 16), u[6] | (u[7] << 16)};
    } else {
      uint32_t u[16];
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          u[4 * sub + v] = ord16(acc[sub][v]);
          stat(acc[sub][v]);
        }
      *reinterpret_cast<uint4*>(ent + (wo ^ sw)) =
          uint4{u[0] | (u[1] << 16), u[2] | (u[3] << 16), u[4] | (u[5] << 16), u[6] | (u[7] << 16)};
      *reinterpret_cast<uint4*>(ent + ((wo + 4) ^ sw)) = uint4{u[8] | (u[9] << 16), u[10] | (u[11] << 16),
                                                             u[12] | (u[13] << 16), u[14] | (u[15] << 16)};
    }
  });
  wave_lds_sync();

  // ---- threshold per row
  bsum = sum_lane_groups(bsum);
  bsq = sum_lane_groups(bsq);
  bcnt = sum_lane_groups(bcnt);
  bmax = fmaxf(bmax, xor_shfl_f32(bmax, 16));
  bmax = fmaxf(bmax, xor_shfl_f32(bmax, 32));
  bmin = fminf(bmin, xor_shfl_f32(bmin, 16));
  bmin = fminf(bmin, xor_shfl_f32(bmin, 32));
  const int n_ent = row_tiles * 4 * lane_ent;
  // rows with fewer than 64 blocks keep every key, and so do rows of up to two
  // tiles, whose keys (32 a lane) have room: of 64 of them a threshold from
  // rounded scores may leave out one, and the fallback takes the wave (16
  // queries over 64 float32 keys of r = 32, 32 heads: 31 us, now 13)
  float tau = -FLT_MAX;
  static_assert(2 * kTile / 4 < kBSlots, "two tiles of candidates fit a lane");
  bool done = bcnt < (float)kList || row_tiles <= 2;
  float lo = 0.f, hi = 0.f;
  if (!done) {
    const float mean = bsum / bcnt;
    const float sd = sqrtf(fmaxf(bsq / bcnt - mean * mean, 0.f));
    const float tail = (float)kList / bcnt;  // in (0, 1]
    const float zq = tail <= 0.5f ? normal_upper_quantile(tail)
                                  : (tail < 1.f ? -normal_upper_quantile(1.f - tail) : -4.f);
    const float pred = mean + sd * zq;  // predicted 64th largest maximum
    lo = fmaxf(pred - 1.5f * sd, bmin);
    hi = fminf(pred + 0.5f * sd, bmax);
    if (!(hi > lo)) {  // all maxima (nearly) equal
      tau = bmin;
      done = true;
    }
  }
  uint32_t* hist = reinterpret_cast<uint32_t*>(wl + kMR * kBEnt * 2) + qi * kBBins;  // bin b at word b ^ sw
  for (int round = 0; __ballot(!done) != 0; ++round) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      *reinterpret_cast<uint4*>(hist + ((16 * g + 4 * u) ^ sw)) = uint4{0u, 0u, 0u, 0u};
    wave_lds_sync();
    const float inv_w = (float)(kBBins - 1) / (hi - lo);  // bins 0..62 over [lo, hi), 63 above
    const float off = -lo * inv_w;
    if (!done) {
      // an entry (in the top 16 bits of o) counts in bin (its value - lo) * inv_w,
      // cut to 63, unless that is below 0; an empty entry reads as NaN and
      // does not count
      auto count = [&](uint32_t o) {
        const uint32_t bits = o ^ (~(uint32_t)((int32_t)o >> 31) | 0x80000000u);
        const float x = fmaf(__uint_as_float(bits), inv_w, off);
        const int b = min((int)x, kBBins - 1);
        if (x >= 0.f) atomicAdd(&hist[b ^ sw], 1u);
      };
#pragma unroll 2
      for (int e0 = 8 * g; e0 < n_ent; e0 += 32) {  // this lane's quarter of the row's entries
        const uint4 w = *reinterpret_cast<const uint4*>(ent + ((e0 / 2) ^ sw));
        const uint32_t ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          count(ww[u] << 16);
          count(ww[u] & 0xffff0000u);
        }
      }
    }
    wave_lds_sync();
    // bins 16 g .. 16 g + 15 of this lane's row: counts from the top
    uint32_t c[16];
    {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint4 t = *reinterpret_cast<const uint4*>(hist + ((16 * g + 4 * u) ^ sw));
        c[4 * u] = t.x;
        c[4 * u + 1] = t.y;
        c[4 * u + 2] = t.z;
        c[4 * u + 3] = t.w;
      }
    }
    uint32_t run = 0;
#pragma unroll
    for (int i = 15; i >= 0; --i) {
      run += c[i];
      c[i] = run;
    }
    const uint32_t t1 = xor_shfl_u32(run, 16), t2 = xor_shfl_u32(run, 32), t3 = xor_shfl_u32(t1, 32);
    // totals of the lane groups above g (groups g ^ 1, g ^ 2, g ^ 3 hold t1, t2, t3)
    const uint32_t above = g == 0 ? t1 + t2 + t3 : g == 1 ? t2 + t3 : g == 2 ? t1 : 0u;
    int n_ge = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) n_ge += (c[i] + above >= (uint32_t)kList) ? 1 : 0;
    int b = n_ge > 0 ? 16 * g + n_ge - 1 : -1;
    b = max(b, (int)xor_shfl_u32((uint32_t)b, 16));
    b = max(b, (int)xor_shfl_u32((uint32_t)b, 32));
    if (!done) {
      const float w = (hi - lo) / (float)(kBBins - 1);
      if (round >= 3) {  // no usable window: keep every key (the count check decides)
        done = true;
      } else if (b < 0) {  // the 64th largest maximum lies below the window
        hi = lo;
        lo = bmin;
        done = !(hi > lo);
      } else if (b == kBBins - 1 && hi < bmax) {  // or above it
        lo = hi;
        hi = bmax;
      } else {
        // one bin lower than the crossing: rounding in the bin index never
        // puts a maximum below tau
        tau = lo + (float)(b - 1) * w;
        done = true;
      }
    }
    wave_lds_sync();
  }

  // ---- pass B: candidates, every key scoring >= tau
  // Slot j of a lane holds a score bits at word 128 j + lane and its key at
  // word 128 j + 64 + lane (so that the lanes' writes spread over the banks
  // and a pair is one two-address write).  Every score is written to the
  // lane's next free slot and the pointer moves on only past one >= tau, so
  // no lane branches; a lane whose count reaches the last slot keeps
  // counting and overwrites it (and the wave then takes the fallback below).
  uint32_t* const cw = reinterpret_cast<uint32_t*>(wl) + lane;
  uint32_t* wp = cw;
  int cnt = 0;
  sc.template for_tiles_deep<kBDepth>(hbase, kbeg, kend, qi, g, [&](int t0, f32x4_t* acc) {
    mask_tile(t0, acc);
    const uint32_t kb = (uint32_t)(t0 + 4 * g);
    if (__ballot(cnt > kBSlots - 16) == 0) {  // room for the whole tile in every lane
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          wp[0] = __float_as_uint(acc[sub][v]);
          wp[kWave] = kb + (uint32_t)(16 * sub + v);
          wp += acc[sub][v] >= tau ? 2 * kWave : 0;
        }
      cnt = (int)(wp - cw) / (2 * kWave);
    } else {
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          uint32_t* sp = cw + 2 * kWave * min(cnt, kBSlots - 1);
          sp[0] = __float_as_uint(acc[sub][v]);
          sp[kWave] = kb + (uint32_t)(16 * sub + v);
          cnt += acc[sub][v] >= tau ? 1 : 0;
        }
      wp = cw + 2 * kWave * min(cnt, kBSlots - 1);
    }
  });

  // the row's candidates: at least 64 unless every key of the row is one
  int row_cnt = cnt + (int)xor_shfl_u32((uint32_t)cnt, 16);
  row_cnt += (int)xor_shfl_u32((uint32_t)row_cnt, 32);
  const bool short_row = tau > -FLT_MAX && row_cnt < kList;
  if (__ballot(cnt >= kBSlots || short_row) == 0) {
    // ---- sort the candidates, keep the best 64
    wave_lds_sync();
    const uint32_t* const wbase = cw - lane;  // word 0 of the wave's slots
    // 32-bit keys: the top 24 bits of the ordered score s', then the
    // candidate's id 4 slot + g (0 past the lane's count)
    auto key32 = [&](int j) -> uint32_t {
      const uint32_t sb = cw[2 * kWave * min(j, kBSlots - 1)];
      const uint32_t o = sb ^ ((uint32_t)((int32_t)sb >> 31) | 0x80000000u);
      return j < cnt ? (o & 0xffffff00u) | (uint32_t)(4 * j + g) : 0u;
    };
    uint32_t x32[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x32[i] = key32(i);
    sort64_u32(x32, g);
    uint32_t dmax = 0u;  // the best key left out
    // the slots past the first 16 of each lane, 16 at a time, sorted
    // ascending (as complemented keys) and merged
#pragma unroll 1
    for (int set = 1; 16 * set < kBSlots && __ballot(cnt > 16 * set) != 0; ++set) {
      uint32_t y[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = ~key32(16 * set + i);
      sort64_u32(y, g);
#pragma unroll
      for (int i = 0; i < 16; ++i) y[i] = ~y[i];
      merge64_u32(x32, y, dmax);
    }
    // the kept set is certain unless the 64th kept key and the best one left
    // out share their top 24 bits
    dmax = umax32(dmax, xor_shfl_u32(dmax, 16));
    dmax = umax32(dmax, xor_shfl_u32(dmax, 32));
    // entry 63 of the row (x32[15] of lane group 3) in all four lanes; every
    // lane takes part in both swaps
    const uint32_t s32 = xor_shfl_u32(x32[15], 32);
    const uint32_t t32 = (g & 2) ? x32[15] : s32;
    const uint32_t s16 = xor_shfl_u32(t32, 16);
    const uint32_t k64 = (g & 1) ? t32 : s16;
    const bool unsure = dmax != 0u && (dmax >> 8) == (k64 >> 8);
    K x[16];
    if (__ballot(unsure) == 0) {
      // the kept entries as exact keys of (s' + b, index), in key order up to
      // runs of equal top 24 bits; two odd-even transposition steps put runs
      // of two in order (what is left is found below)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const uint32_t id = x32[i] & 0xffu;
        const uint32_t* c = wbase + 2 * kWave * (id >> 2) + 16 * (id & 3) + qi;
        x[i] = x32[i] == 0u ? KO::pad() : KO::make(__uint_as_float(c[0]) + my_b, (int)c[kWave]);
      }
      auto cx64 = [](K& a, K& b2) {
        const bool sw = KO::gt(b2, a);
        const K t = a;
        a = KO::sel(sw, b2, a);
        b2 = KO::sel(sw, t, b2);
      };
#pragma unroll
      for (int i = 0; i < 16; i += 2) cx64(x[i], x[i + 1]);
#pragma unroll
      for (int i = 1; i < 15; i += 2) cx64(x[i], x[i + 1]);
      {  // entries 16 g + 15 and 16 (g + 1), held by lanes 16 apart
        const K nxt = ((uint64_t)(uint32_t)__shfl_down((int)(uint32_t)(x[0] >> 32), 16, kWave) << 32) |
                      (uint32_t)__shfl_down((int)(uint32_t)x[0], 16, kWave);
        const K prv = ((uint64_t)(uint32_t)__shfl_up((int)(uint32_t)(x[15] >> 32), 16, kWave) << 32) |
                      (uint32_t)__shfl_up((int)(uint32_t)x[15], 16, kWave);
        if (g < 3 && KO::gt(nxt, x[15])) x[15] = nxt;
        if (g > 0 && KO::gt(x[0], prv)) x[0] = prv;
      }
    } else {
      // exact 64-bit keys of (s', index) over all slots
      auto slot = [&](int j) {
        const uint32_t* c = cw + 2 * kWave * min(j, kBSlots - 1);
        return j < min(cnt, kBSlots) ? KO::make(__uint_as_float(c[0]), (int)c[kWave]) : KO::pad();
      };
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = slot(i);
      sort64_x16<KO>(x, g);
#pragma unroll 1
      for (int set = 1; 16 * set < kBSlots && __ballot(cnt > 16 * set) != 0; ++set) {
        K y[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) y[i] = slot(16 * set + i);
        sort64_x16<KO>(y, g);
        merge64_x16<KO>(x, y, g);
      }
      // x holds the best 64 by s', sorted; b is added (the scores stay
      // non-increasing, and ties that arise are put in order below)
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i] = KO::make(KO::score(x[i]) + my_b, KO::index(x[i]));
    }
    // two entries whose scores are equal must stand in index order: the rare
    // row where some do not is sorted again
    bool disorder = false;
#pragma unroll
    for (int i = 1; i < 16; ++i) disorder |= KO::gt(x[i], x[i - 1]);
    {  // entry 16 (g + 1) of the row, held by the lane 16 above
      const uint32_t hi = (uint32_t)__shfl_down((int)(uint32_t)(x[0] >> 32), 16, kWave);
      const uint32_t lo = (uint32_t)__shfl_down((int)(uint32_t)x[0], 16, kWave);
      disorder |= g < 3 && KO::gt(((uint64_t)hi << 32) | lo, x[15]);
    }
    if (__ballot(disorder) != 0) sort64_x16<KO>(x, g);
    if (row_ok) {
      const size_t rw = bh * Q + my_row;
      // a lane's 16 entries are 64 contiguous bytes of its row
      const bool vec = k == kMaxK && ((reinterpret_cast<uintptr_t>(top_idx) |
                                       reinterpret_cast<uintptr_t>(top_score)) & 15) == 0;
      if (n_chunks == 1 && vec) {
        int4* ip = reinterpret_cast<int4*>(top_idx + rw * kMaxK + 16 * g);
#pragma unroll
        for (int u = 0; u < 4; ++u)
          ip[u] = int4{out_index<KO>(x[4 * u]), out_index<KO>(x[4 * u + 1]),
                       out_index<KO>(x[4 * u + 2]), out_index<KO>(x[4 * u + 3])};
        if (top_score) {
          float4* sp = reinterpret_cast<float4*>(top_score + rw * kMaxK + 16 * g);
#pragma unroll
          for (int u = 0; u < 4; ++u)
            sp[u] = float4{KO::score(x[4 * u]), KO::score(x[4 * u + 1]), KO::score(x[4 * u + 2]),
                           KO::score(x[4 * u + 3])};
        }
      } else if (n_chunks == 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int e = 16 * g + i;
          if (e < k) {
            top_idx[rw * k + e] = out_index<KO>(x[i]);
            if (top_score) top_score[rw * k + e] = KO::score(x[i]);
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) part[(rw * n_chunks + ch) * kMaxK + 16 * g + i] = x[i];
      }
    }
    return;
  }

  // ---- fallback: online selection over the chunk, in two halves of 8 rows,
  // scores formed whole (accumulators starting at b)
  sc.init = my_b;
  wave_lds_sync();
  float* stage = reinterpret_cast<float*>(wl);  // [16][64], key column swizzled
  K* lists = reinterpret_cast<K*>(wl + kMR * kTile * 4);
  constexpr int kHalf = kMR / 2;
  for (int half = 0; half < 2; ++half) {
    RowLists<KO, kHalf> top;
    top.init(lists, lists + kHalf * kList);
    sc.for_tiles(hbase, kbeg, kend, kTile, qi, g, [&](int t0, f32x4_t* acc) {
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        const f32x4_t sv = acc[sub];
        *reinterpret_cast<f32x4_t*>(&stage[qi * kTile + ((16 * sub + 4 * g) ^ (qi << 2))]) = sv;
      }
      wave_lds_sync();
      const bool need_mask = t0 + kTile > kmin;
      for (int rr = 0; rr < kHalf; ++rr) {
        const int r = kHalf * half + rr;
        float sv = stage[r * kTile + (lane ^ (r << 2))];
        const int j = t0 + lane;
        if (need_mask && j >= __builtin_amdgcn_readlane(my_lim, r)) sv = -INFINITY;
        top.offer(rr, sv, j);
      }
      wave_lds_sync();
    });
    for (int rr = 0; rr < kHalf; ++rr) {
      top.finish(rr);
      const int i = row0 + kHalf * half + rr;
      if (i >= Q) continue;
      const K e = top.entry(rr);
      const size_t rw = bh * Q + i;
      if (n_chunks == 1) {
        if (lane < k) {
          top_idx[rw * k + lane] = out_index<KO>(e);
          if (top_score) top_score[rw * k + lane] = KO::score(e);
        }
      } else {
        part[(rw * n_chunks + ch) * kMaxK + lane] = e;
      }
    }
    wave_lds_sync();
  }
}

// ---------------------------------------------------------------- sketch scoring, MFMA, one pass

// Long rows (a batch of decode queries over a long cache) read each code once.
// A wave scores its 16 query rows against one key chunk on the MFMA (the
// layout of MfmaScorer, the mean term b folded into the accumulator) and
// keeps a running top-64 per row: a sorted 64-entry list and a 64-slot
// buffer of unsorted candidates, both in LDS.  A score is a candidate when it
// beats the row's threshold; a buffer that would overflow is sorted and
// merged into the list, which raises the threshold to the list's 64th score.
// Tiles are visited in increasing key order and buffers are flushed only
// between tiles, so a later key that merely ties the threshold ranks below
// every list entry: the strict test loses nothing.
//
// The threshold starts at a gate read off a sample of the chunk (8 tiles
// spread over it): the least, over the row's four lanes, of each lane's
// second-best sampled score, so that at least 8 sampled keys reach it.  The
// gate only bounds which keys are kept: a row whose list ends with 64
// entries above it holds the exact top-64 of the chunk.  A row that kept
// fewer (the gate was above its 64th score) still holds every key of the
// chunk above the gate.  With one chunk per row the wave scans such rows
// again without a gate.  With several, it records the gate in `gates` (-inf
// for rows that need none) and merge_kernel checks that the row's merged
// k-th score lies above every recorded gate, which makes the merged list
// exact.  Rows that fail the check are flagged; a second launch of this
// kernel with `only` = the flags rescans their chunks without a gate (its
// waves without a flagged row exit at once) and a second merge of just those
// rows follows.  A chunk's gate sits near its 200th-best key while the
// merged k-th score sits near each chunk's (64 / chunks)-th best, so rows
// fail only when several of their best keys fall in one chunk's sample (the
// queries of a sequence can share a few dominant keys).
//
// grid: 8 * ceil(ceil(units / kScanWaves) / 8) work-groups (XCD-ordered, as
// for xcd_logical_block), units = n_bh * wave_rows * n_chunks, one unit
// (head, 16-row block, chunk) per wave, chunks fastest.
using saki::kScanWaves;
constexpr int kScanBuf = 64;            // candidate slots per row
constexpr int kScanSample = 8;          // sampled tiles per chunk
constexpr int kScanGateKeys = 16 * kTile;  // rows with fewer keys in the chunk start ungated

template <int RK, int ST>
__global__ __launch_bounds__(kScanWaves * kWave) void score_scan_kernel(
    const uint8_t* __restrict__ index, int n_tiles, int N_valid, int Q,
    const int* __restrict__ q_pos, const float* __restrict__ q, const float* __restrict__ Bq,
    const float* __restrict__ mu, int H_q, int H_kv, int gq, int n_bh, int wave_rows, int chunk,
    int n_chunks, int k, int* __restrict__ top_idx, float* __restrict__ top_score,
    uint64_t* __restrict__ part, float* __restrict__ gates, const int* __restrict__ only) {
  constexpr int D = saki::kHeadDim;
  using KO = KeysF32;
  using K = KO::K;
  using Scorer = MfmaScorer<RK, ST>;
  __shared__ K list_mem[kScanWaves][kMR * kList];
  __shared__ K buf_mem[kScanWaves][kMR * kScanBuf];  // first the sketch staging [16][RK] floats
  static_assert(kMR * RK * sizeof(float) <= kMR * kScanBuf * sizeof(K), "sketch staging fits");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  const long long units = (long long)n_bh * wave_rows * n_chunks;
  const long long lb = xcd_logical_block((units + kScanWaves - 1) / kScanWaves);
  if (lb < 0) return;
  const long long unit = lb * kScanWaves + wave;
  if (unit >= units) return;
  const int ch = (int)(unit % n_chunks);
  const int wr = (int)((unit / n_chunks) % wave_rows);
  const size_t bh = (size_t)(unit / ((long long)n_chunks * wave_rows));
  const int h = (int)(bh % H_q);
  const int qi = lane % 16, g = lane / 16;
  const int row0 = wr * kMR;
  const int my_row = row0 + qi;
  const bool row_ok = my_row < Q;
  // with `only`, the rows to redo (a wave with none has nothing to do)
  const bool want = row_ok && (!only || only[bh * Q + my_row] != 0);
  if (only && __ballot(want) == 0) return;
  // keys are counted from the chunk's first one: steps past the last of nearly
  // 2^31 keys would not fit an int
  const int kbeg = ch * chunk;
  const int my_lim = min(row_limit(my_row, Q, N_valid, q_pos) - kbeg, chunk);
  const int kend = wave_max_i(my_lim);
  const int kmin = wave_min_i(row_ok ? my_lim : INT_MAX);
  K* list = list_mem[wave];
  K* buf = buf_mem[wave];

  const size_t code_set = (bh / H_q) * (H_q / gq) + h / gq;
  const uint8_t* hbase = index + (code_set * n_tiles + kbeg / kTile) * Scorer::TB;
  // the gate's sample: every stride-th tile of the chunk, at most kScanSample;
  // the first kSA of them are requested before the query sketch is formed
  const int n_row = row_ok ? max(0, my_lim) : 0;
  const bool gated = !only && wave_max_i(n_row) >= kScanGateKeys;
  const int stride = max(1, kend / (kTile * kScanSample)) * kTile;
  const int n_samp = gated ? min(kScanSample, (kend - 1) / stride + 1) : 0;
  constexpr int kSA = Scorer::NL == 1 ? 4 : Scorer::kPrefetch ? 2 : 1;
  Scorer sc;
  typename Scorer::Raw sraw[kSA];
  auto sample_at = [&](int i) { return hbase + (size_t)(i * stride / kTile) * Scorer::TB; };
#pragma unroll
  for (int u = 0; u < kSA; ++u)
    if (u < n_samp) sc.load(sample_at(u), qi, g, sraw[u]);

  sc.init = mfma_query_sketch<RK, ST>(q + (bh * Q + (row_ok ? my_row : row0)) * D, row_ok,
                                      Bq + (size_t)h * D * RK, mu + (size_t)(h / (H_q / H_kv)) * D,
                                      reinterpret_cast<float*>(buf), qi, g, sc);
#pragma unroll 1
  for (int r = 0; r < kMR; ++r) list[r * kList + lane] = KO::pad();

  // ---- the gate
  float tau = -INFINITY;
  if (gated) {
    float m1 = -INFINITY, m2 = -INFINITY;
    for (int i0 = 0; i0 < n_samp; i0 += kSA) {
#pragma unroll
      for (int u = 0; u < kSA; ++u) {
        const int i = i0 + u;
        if (i >= n_samp) break;
        f32x4_t acc[4];
        sc.mma(sraw[u], acc);
        if (i + kSA < n_samp) sc.load(sample_at(i + kSA), qi, g, sraw[u]);
        const int t0 = i * stride;
#pragma unroll
        for (int sub = 0; sub < 4; ++sub)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float x = t0 + 16 * sub + 4 * g + v < my_lim ? acc[sub][v] : -INFINITY;
            m2 = fmaxf(m2, fminf(m1, x));
            m1 = fmaxf(m1, x);
          }
      }
    }
    // the least of the four lanes' second-best sampled scores: at least 8
    // sampled keys reach it
    float m = m2;
    m = fminf(m, xor_shfl_f32(m, 16));
    m = fminf(m, xor_shfl_f32(m, 32));
    if (n_row >= kScanGateKeys) tau = m;
  }

  // ---- the scan
  float thr = want ? tau : INFINITY;  // row qi's threshold (the same in its four lanes)
  int base = 0;                       // row qi's buffered candidates
  auto flush = [&](int r) {
    wave_lds_sync();
    const int c = __builtin_amdgcn_readlane(base, r);  // lane r: row r, lane group 0
    K b = lane < c ? buf[r * kScanBuf + lane] : KO::pad();
    wave_sort<KO>(b);
    K a = list[r * kList + lane];
    wave_merge<KO>(a, b);
    list[r * kList + lane] = a;
    const float t = KO::score(KO::readlane(a, kWave - 1));
    if (qi == r) {
      thr = fmaxf(thr, t);
      base = 0;
    }
    wave_lds_sync();
  };
  auto scan = [&]() {
    sc.for_tiles_deep(hbase, 0, kend, qi, g, [&](int t0, f32x4_t* acc) {
      uint32_t take = 0;
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) take |= (acc[sub][v] > thr ? 1u : 0u) << (4 * sub + v);
      if (t0 + kTile > kmin) {  // a tile crossing some row's limit
#pragma unroll
        for (int sub = 0; sub < 4; ++sub)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (t0 + 16 * sub + 4 * g + v >= my_lim) take &= ~(1u << (4 * sub + v));
      }
      if (__ballot(take != 0) == 0) return;
      // the four lanes of a row append at offsets from a prefix of their counts
      int c = __popc(take);
      int c1 = (int)xor_shfl_u32((uint32_t)c, 16);   // lane group g ^ 1
      int c2 = (int)xor_shfl_u32((uint32_t)c, 32);   // g ^ 2
      int c3 = (int)xor_shfl_u32((uint32_t)c1, 32);  // g ^ 3
      uint64_t full = __ballot(base + c + c1 + c2 + c3 > kScanBuf) & 0xffffull;
      if (full) {
        do {
          flush(__builtin_ctzll(full));
          full &= full - 1;
        } while (full);
#pragma unroll
        for (int sub = 0; sub < 4; ++sub)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (!(acc[sub][v] > thr)) take &= ~(1u << (4 * sub + v));
        c = __popc(take);
        c1 = (int)xor_shfl_u32((uint32_t)c, 16);
        c2 = (int)xor_shfl_u32((uint32_t)c, 32);
        c3 = (int)xor_shfl_u32((uint32_t)c1, 32);
      }
      int pos = base + (g == 1 ? c1 : g == 2 ? c2 + c3 : g == 3 ? c1 + c2 + c3 : 0);
      base += c + c1 + c2 + c3;
      // a lane rarely holds more than one or two candidates of a tile: take
      // them one per round, lowest element first, each picked out of the 16
      // scores by the bits of its element number
      while (__ballot(take != 0)) {
        const int e = __builtin_ctz(take | 0x10000u);
        // bit masks of e's bits: (m & x) | (~m & y) picks x where the bit is set
        const uint32_t m0 = 0u - (uint32_t)(e & 1), m1 = 0u - (uint32_t)((e >> 1) & 1);
        const uint32_t m2 = 0u - (uint32_t)((e >> 2) & 1), m3 = 0u - (uint32_t)((e >> 3) & 1);
        auto pick = [](uint32_t m, uint32_t x, uint32_t y) { return (m & x) | (~m & y); };
        uint32_t s8[8], s4[4], s2[2];
#pragma unroll
        for (int m = 0; m < 8; ++m)
          s8[m] = pick(m0, __float_as_uint(acc[m >> 1][(2 * m + 1) & 3]), __float_as_uint(acc[m >> 1][(2 * m) & 3]));
#pragma unroll
        for (int m = 0; m < 4; ++m) s4[m] = pick(m1, s8[2 * m + 1], s8[2 * m]);
#pragma unroll
        for (int m = 0; m < 2; ++m) s2[m] = pick(m2, s4[2 * m + 1], s4[2 * m]);
        const float sv = __uint_as_float(pick(m3, s2[1], s2[0]));
        if (take) {
          buf[qi * kScanBuf + pos] = KO::make(sv, kbeg + t0 + 16 * (e >> 2) + 4 * g + (e & 3));
          ++pos;
          take &= take - 1;
        }
      }
    });
    uint64_t left = __ballot(base > 0) & 0xffffull;
    while (left) {
      flush(__builtin_ctzll(left));
      left &= left - 1;
    }
  };
  scan();
  // rows whose gate kept fewer than 64 keys of the chunk
  wave_lds_sync();
  const bool short_row = tau > -INFINITY && KO::index(list[qi * kList + kList - 1]) == kPadIdx;
  if (n_chunks > 1) {
    if (g == 0 && want) gates[(bh * Q + my_row) * n_chunks + ch] = short_row ? tau : -INFINITY;
  } else if (__ballot(short_row) != 0) {  // one chunk: again, ungated; the other rows are done
    for (uint64_t m = __ballot(short_row) & 0xffffull; m; m &= m - 1)
      list[__builtin_ctzll(m) * kList + lane] = KO::pad();
    thr = short_row ? -INFINITY : INFINITY;
    wave_lds_sync();
    scan();
    wave_lds_sync();
  }

  for (int r = 0; r < kMR; ++r) {
    const int i = row0 + r;
    if (i >= Q) break;
    if (!__builtin_amdgcn_readlane((int)want, r)) continue;
    const K e = list[r * kList + lane];
    if (n_chunks == 1) {
      if (lane < k) {
        const size_t o = (bh * Q + i) * k + lane;
        top_idx[o] = out_index<KO>(e);
        if (top_score) top_score[o] = KO::score(e);
      }
    } else {
      part[((bh * Q + i) * n_chunks + ch) * kMaxK + lane] = e;
    }
  }
}

// ---------------------------------------------------------------- exact scores + recall

// Writes the exact top-k of a finished row, or its partial list.
template <class KO>
__device__ __forceinline__ void exact_row_out(typename KO::K e, size_t row, int ch, int n_chunks,
                                              int k, const int* approx, int* hits,
                                              int* exact_idx, typename KO::K* part) {
  const int lane = lane_id();
  if (n_chunks == 1) {
    const int ej = out_index<KO>(e);
    if (exact_idx && lane < k) exact_idx[row * k + lane] = ej;
    const int hsum = row_hits(ej, approx, row, k);
    if (lane == 0) hits[row] = hsum;
  } else {
    part[(row * n_chunks + ch) * kMaxK + lane] = e;
  }
}

// grid (row_blocks * n_chunks, B*H_q), block 64*waves.  Exact float64 scores
// with float64 FMAs, one key per lane, R rows per wave.
template <bool KBF, int R>
__global__ __launch_bounds__(256) void exact_stream_kernel(
    const void* __restrict__ keys, const float* __restrict__ q,
    const int* __restrict__ q_pos, int H_q, int H_kv, int N_cap, int N_valid, int Q,
    int row_blocks, int chunk, int n_chunks, int k, const int* __restrict__ approx,
    int* __restrict__ hits, int* __restrict__ exact_idx, KeyF64* __restrict__ part,
    const int* __restrict__ only) {
  constexpr int D = saki::kHeadDim;
  using KO = KeysF64;
  __shared__ double qsh[kStreamWaves][R][D];
  __shared__ KeyF64 lmem[kStreamWaves][R][kList];
  __shared__ KeyF64 bmem[kStreamWaves][R][kList];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int waves = blockDim.x / kWave;
  const int rb = blockIdx.x % row_blocks, ch = blockIdx.x / row_blocks;
  const size_t bh = blockIdx.y;
  const int b = (int)(bh / H_q), h = (int)(bh % H_q);
  const int gkv = h / (H_q / H_kv);
  const int row0 = (rb * waves + wave) * R;
  if (row0 >= Q) return;
  // with `only`, the rows flagged there (a wave with none has nothing to do)
  if (only && __ballot(lane < R && row0 + lane < Q && only[bh * Q + row0 + lane] != 0) == 0) return;
  int lim[R];
  int kmax = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    lim[r] = row_limit(row0 + r, Q, N_valid, q_pos);
    kmax = lim[r] > kmax ? lim[r] : kmax;
  }
  for (int i = lane; i < R * D; i += kWave) {
    const int r = i / D;
    qsh[wave][r][i % D] = (row0 + r < Q) ? (double)q[(bh * Q + row0 + r) * D + (i % D)] : 0.0;
  }
  RowLists<KO, R> top;
  top.init(&lmem[wave][0][0], &bmem[wave][0][0]);
  const size_t kbase = ((size_t)b * H_kv + gkv) * N_cap;
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  for (int t0 = kbeg; t0 < kend; t0 += kTile) {
    const int j = t0 + lane;
    const bool inb = j < N_valid;
    double acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0;
#pragma unroll 2
    for (int c0 = 0; c0 < D; c0 += 8) {
      double kv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) kv[e] = inb ? (double)load_key_elem<KBF>(keys, (kbase + j) * D + c0 + e) : 0.0;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[r] = fma(qsh[wave][r][c0 + e], kv[e], acc[r]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) top.offer(r, j < lim[r] ? acc[r] : -(double)INFINITY, j);
  }
  for (int r = 0; r < R; ++r) {
    top.finish(r);
    const int i = row0 + r;
    if (i >= Q || (only && only[bh * Q + i] == 0)) continue;
    exact_row_out<KO>(top.entry(r), bh * Q + i, ch, n_chunks, k, approx, hits, exact_idx, part);
  }
}

// Exact float64 scores on the f64 MFMA (16x16x4).  Lane group g feeds dims
// 32g .. 32g+31 of its key and query, one per k-step.  The f64 MFMA returns
// D[g + 4v][lane % 16] in register v.  grid (row_blocks * n_chunks, B*H_q) via
// xcd_grid, two waves of 16 rows per work-group.
template <bool KBF>
__global__ __launch_bounds__(128) void exact_mfma_kernel(
    const void* __restrict__ keys, const float* __restrict__ q,
    const int* __restrict__ q_pos, int H_q, int H_kv, int N_cap, int N_valid, int Q,
    int row_blocks, int chunk, int n_chunks, int k, const int* __restrict__ approx,
    int* __restrict__ hits, int* __restrict__ exact_idx, KeyF64* __restrict__ part, int n_bh,
    const int* __restrict__ redo) {
  constexpr int D = saki::kHeadDim;
  using KO = KeysF64;
  // staged scores [row][key], key column swizzled by the row index
  __shared__ double stage[kMfmaWaves][kMR][kTile];
  __shared__ KeyF64 lmem[kMfmaWaves][kMR][kList];
  __shared__ KeyF64 bmem[kMfmaWaves][kMR][kList];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int waves = blockDim.x / kWave;
  const long long lb = xcd_logical_block((long long)row_blocks * n_chunks * n_bh);
  if (lb < 0) return;
  const int rb = (int)(lb % row_blocks), ch = (int)((lb / row_blocks) % n_chunks);
  const size_t bh = (size_t)(lb / ((long long)row_blocks * n_chunks));
  const int b = (int)(bh / H_q), h = (int)(bh % H_q);
  const int gkv = h / (H_q / H_kv);
  const int row0 = (rb * waves + wave) * kMR;
  if (row0 >= Q) return;
  // as the fallback of exact_bf16_kernel: only the waves it flagged
  if (redo && redo[lb * kMfmaWaves + wave] == 0) return;
  const int qi = lane % 16, g = lane / 16;
  const int my_row = row0 + qi;
  const bool row_ok = my_row < Q;
  const int my_lim = row_limit(my_row, Q, N_valid, q_pos);
  const int kmax = wave_max_i(my_lim);
  const int kmin = wave_min_i(row_ok ? my_lim : INT_MAX);
  double qreg[32];
  {
    const float* qr = q + (bh * Q + (row_ok ? my_row : row0)) * D + 32 * g;
#pragma unroll
    for (int s4 = 0; s4 < 8; ++s4) {
      const float4 v = *reinterpret_cast<const float4*>(qr + 4 * s4);
      qreg[4 * s4 + 0] = row_ok ? (double)v.x : 0.0;
      qreg[4 * s4 + 1] = row_ok ? (double)v.y : 0.0;
      qreg[4 * s4 + 2] = row_ok ? (double)v.z : 0.0;
      qreg[4 * s4 + 3] = row_ok ? (double)v.w : 0.0;
    }
  }
  RowLists<KO, kMR> top;
  top.init(&lmem[wave][0][0], &bmem[wave][0][0]);
  const size_t kbase = ((size_t)b * H_kv + gkv) * N_cap;
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  for (int t0 = kbeg; t0 < kend; t0 += kTile) {
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      const int j = t0 + 16 * sub + qi;
      const bool inb = j < N_valid;
      float kf[32];
      if constexpr (KBF) {
        const uint16_t* kr = reinterpret_cast<const uint16_t*>(keys) + (kbase + (inb ? j : 0)) * D + 32 * g;
#pragma unroll
        for (int s8 = 0; s8 < 4; ++s8) {
          const uint4 v = *reinterpret_cast<const uint4*>(kr + 8 * s8);
          unpack_piece<true>(v, kf + 8 * s8);
        }
      } else {
        const float* kr = reinterpret_cast<const float*>(keys) + (kbase + (inb ? j : 0)) * D + 32 * g;
#pragma unroll
        for (int s4 = 0; s4 < 8; ++s4) {
          const float4 v = *reinterpret_cast<const float4*>(kr + 4 * s4);
          kf[4 * s4 + 0] = v.x;
          kf[4 * s4 + 1] = v.y;
          kf[4 * s4 + 2] = v.z;
          kf[4 * s4 + 3] = v.w;
        }
      }
      f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 32; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(inb ? (double)kf[s] : 0.0, qreg[s], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) stage[wave][qi][(16 * sub + g + 4 * v) ^ qi] = acc[v];
    }
    wave_lds_sync();
    const bool need_mask = t0 + kTile > kmin;
    for (int r = 0; r < kMR; ++r) {
      double sv = stage[wave][r][lane ^ r];
      const int j = t0 + lane;
      if (need_mask && j >= __builtin_amdgcn_readlane(my_lim, r)) sv = -(double)INFINITY;
      top.offer(r, sv, j);
    }
    wave_lds_sync();
  }
  for (int r = 0; r < kMR; ++r) {
    top.finish(r);
    const int i = row0 + r;
    if (i >= Q) continue;
    exact_row_out<KO>(top.entry(r), bh * Q + i, ch, n_chunks, k, approx, hits, exact_idx, part);
  }
}

// ---------------------------------------------------------------- exact scores, bound-and-rescore

// Keys rounded to bf16 in the MFMA tile layout of the codes (16 pieces of 8
// dims per key), and an upper bound of every key's Euclidean norm (rows of
// n_tiles * 64 per (b, g), so that aligned groups of four can be loaded).
// grid (n_tiles(N_valid), B*H_kv), block 256.
template <bool KBF>
__global__ __launch_bounds__(256) void keys_hi_kernel(const void* __restrict__ keys, int N_cap,
                                                      int N_valid, int n_tiles,
                                                      uint8_t* __restrict__ khi,
                                                      uint8_t* __restrict__ klo,
                                                      float* __restrict__ knorm) {
  constexpr int D = saki::kHeadDim;
  constexpr int NP = D / 8;
  __shared__ float part[4][kTile];
  const int tile = blockIdx.x;
  const size_t bg = blockIdx.y;
  const int t = threadIdx.x % kTile, pg = threadIdx.x / kTile;
  const int n = tile * kTile + t;
  const bool ok = n < N_valid;
  const size_t toff = (bg * n_tiles + tile) * (size_t)kTile * D * 2;
  float ss = 0.f;
  for (int p = pg; p < NP; p += 4) {
    float f[8], hi[8], lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      f[e] = ok ? load_key_elem<KBF>(keys, (bg * N_cap + n) * D + 8 * p + e) : 0.f;
      ss = fmaf(f[e], f[e], ss);
      hi[e] = bf16_round(f[e]);
      lo[e] = bf16_round(f[e] - hi[e]);  // exact difference, then rounded
    }
    const size_t o = toff + (size_t)p * kTile * 16 + (size_t)t * 16;
    *reinterpret_cast<uint4*>(khi + o) = pack_bf16x8(hi);
    *reinterpret_cast<uint4*>(klo + o) = pack_bf16x8(lo);
  }
  part[pg][t] = ss;
  __syncthreads();
  if (pg == 0)  // one row of n_tiles * 64 bounds per (b, g); 0 past N_valid
    knorm[bg * n_tiles * kTile + n] =
        ok ? sqrtf(part[0][t] + part[1][t] + part[2][t] + part[3][t]) * (1.f + 1e-5f) : 0.f;
}

// Exact top-64 and recall hits by bound-and-rescore.  With x = x_h + x_l + x_r
// (x_h = bf16(x), x_l = bf16(x - x_h)), the three bf16 MFMA products
// a3 = q_h.k_h + q_h.k_l + q_l.k_h miss q.k by the dropped terms (at most about
// 3 * 2^-16 sum|q_i k_i|) plus float32 accumulation (at most 384 * 2^-24 of the
// same sum), so |a3 - q.k| <= E = kExactEps3 * ||q|| ||k|| with 40% margin.
// Three passes run on these intervals: moments of the
// single product q_h.k_h (only a prediction), a histogram of the lower bounds
// a3 - E, and a gate on the upper bounds a3 + E at the bin where the
// lower-bound count reaches 64: every key whose exact score can reach the 64th
// exact score passes it.  Gated keys are rescored in float64 (float32 inputs,
// so every product is exact) and sorted.  A wave whose rows miss the
// prediction or gate more than 128 keys is flagged and redone by
// exact_mfma_kernel.  grid/block as exact_mfma_kernel.
constexpr float kExactEps3 = 1e-4f;

template <bool KBF>
__global__ __launch_bounds__(128) void exact_bf16_kernel(
    const void* __restrict__ keys, const uint8_t* __restrict__ khi,
    const uint8_t* __restrict__ klo, const float* __restrict__ knorm, const float* __restrict__ q,
    const int* __restrict__ q_pos, int H_q, int H_kv, int N_cap, int N_valid, int Q,
    int n_tiles_hi, int n_bh, int row_blocks, int chunk, int n_chunks, int k,
    const int* __restrict__ approx, int* __restrict__ hits, int* __restrict__ exact_idx,
    KeyF64* __restrict__ part, const int* __restrict__ only, int* __restrict__ redo) {
  constexpr int D = saki::kHeadDim;
  constexpr size_t TB = (size_t)kTile * D * 2;
  using KO = KeysF64;
  __shared__ int cand_mem[kMfmaWaves][kMR * kCandRow];
  __shared__ int hist_mem[kMfmaWaves][kMR * kHistRow];
  __shared__ float qrow_mem[kMfmaWaves][kMR * D];
  __shared__ int ccount[kMfmaWaves][kMR];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int waves = blockDim.x / kWave;
  const long long lb = xcd_logical_block((long long)row_blocks * n_chunks * n_bh);
  if (lb < 0) return;
  const int rb = (int)(lb % row_blocks), ch = (int)((lb / row_blocks) % n_chunks);
  const size_t bh = (size_t)(lb / ((long long)row_blocks * n_chunks));
  const int b = (int)(bh / H_q), h = (int)(bh % H_q);
  const int gkv = h / (H_q / H_kv);
  const size_t bg = (size_t)b * H_kv + gkv;
  const int row0 = (rb * waves + wave) * kMR;
  if (row0 >= Q) return;
  // as the second tier after exact_gate_kernel: only the waves it flagged
  if (only && only[lb * kMfmaWaves + wave] == 0) {
    if (lane == 0) redo[lb * kMfmaWaves + wave] = 0;
    return;
  }
  const int qi = lane % 16, g = lane / 16;
  const int my_row = row0 + qi;
  const bool row_ok = my_row < Q;
  const int my_lim = row_limit(my_row, Q, N_valid, q_pos);
  const int kmax = wave_max_i(my_lim);
  const int kmin = wave_min_i(row_ok ? my_lim : INT_MAX);
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  int* cand = cand_mem[wave];
  int* hist = hist_mem[wave];
  float* qrows = qrow_mem[wave];
  const size_t hoff = bg * n_tiles_hi * TB;
  const float* kn = knorm + bg * n_tiles_hi * kTile;

  // query: bf16 hi/lo operands (dims 32kk + 8g .. +7), float32 copy in LDS,
  // norm bound
  bf16x8_t qh[4], ql[4];
  float qn;
  {
    const float* qr = q + (bh * Q + (row_ok ? my_row : row0)) * D;
    float ss = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      float fh[8], fl[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float f = row_ok ? qr[32 * kk + 8 * g + e] : 0.f;
        ss = fmaf(f, f, ss);
        qrows[qi * D + 32 * kk + 8 * g + e] = f;
        fh[e] = bf16_round(f);
        fl[e] = bf16_round(f - fh[e]);
      }
      qh[kk] = as_bf16x8(pack_bf16x8(fh));
      ql[kk] = as_bf16x8(pack_bf16x8(fl));
    }
    qn = sqrtf(sum_lane_groups(ss)) * (1.f + 1e-5f);
  }
  const float eq = kExactEps3 * qn;
  wave_lds_sync();

  // THREE: a3 (three products) and its error radius; otherwise q_h.k_h only.
  auto tile = [&](int t0, f32x4_t acc[4], float e[4][4], auto three) {
    const size_t to = hoff + (size_t)(t0 / kTile) * TB;
#pragma unroll
    for (int sub = 0; sub < 4; ++sub) {
      const int key = 16 * sub + qi;
      f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const size_t o = to + (size_t)(4 * kk + g) * kTile * 16 + (size_t)key * 16;
        const bf16x8_t kh = as_bf16x8(*reinterpret_cast<const uint4*>(khi + o));
        a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, qh[kk], a, 0, 0, 0);
        if constexpr (decltype(three)::value) {
          const bf16x8_t kl = as_bf16x8(*reinterpret_cast<const uint4*>(klo + o));
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl, qh[kk], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, ql[kk], a, 0, 0, 0);
        }
      }
      acc[sub] = a;
      if constexpr (decltype(three)::value) {
        // radii of keys t0 + 16 sub + 4g .. +3 (keys past N_valid are masked)
        const int kb = t0 + 16 * sub + 4 * g;
#pragma unroll
        for (int v = 0; v < 4; ++v) e[sub][v] = (kb + v < N_valid) ? eq * kn[kb + v] : 0.f;
      }
    }
  };
  using One = std::integral_constant<bool, false>;
  using Three = std::integral_constant<bool, true>;

  // ---- pass 1: moments of the approximate scores
  float sum = 0.f, sumsq = 0.f;
  for (int t0 = kbeg; t0 < kend; t0 += kTile) {
    f32x4_t acc[4];
    float e[4][4];
    tile(t0, acc, e, One{});
    const bool need_mask = t0 + kTile > kmin;
#pragma unroll
    for (int sub = 0; sub < 4; ++sub)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float x = acc[sub][v];
        if (need_mask && t0 + 16 * sub + 4 * g + v >= my_lim) x = 0.f;
        sum += x;
        sumsq = fmaf(x, x, sumsq);
      }
  }
  sum = sum_lane_groups(sum);
  sumsq = sum_lane_groups(sumsq);
  const int n_row = row_ok ? max(0, min(my_lim, kend) - kbeg) : 0;
  int mode = kModeAll;
  float inv_w = 0.f, off = 0.f;
  if (n_row > kCollect) {
    const float mean = sum / (float)n_row;
    const float sd = sqrtf(fmaxf(sumsq / (float)n_row - mean * mean, 0.f));
    if (sd > 0.f && isfinite(sd) && isfinite(mean)) {
      const float t_hat = mean + sd * normal_upper_quantile((float)kList / (float)n_row);
      const float lo = t_hat - 2.f * sd;
      inv_w = (float)(kBins - 2) / (3.f * sd);
      off = 1.f - lo * inv_w;
      mode = kModeHist;
    } else {
      mode = kModeFallback;
    }
  }

  // ---- pass 2: histogram of the lower bounds
  float gate = -INFINITY;
  if (__ballot(mode == kModeHist) != 0) {
    for (int i = lane; i < kMR * kHistRow; i += kWave) hist[i] = 0;
    wave_lds_sync();
    for (int t0 = kbeg; t0 < kend; t0 += kTile) {
      f32x4_t acc[4];
      float e[4][4];
      tile(t0, acc, e, Three{});
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float x = fmaf(acc[sub][v] - e[sub][v], inv_w, off);
          if (mode == kModeHist && x >= 1.f && t0 + 16 * sub + 4 * g + v < my_lim)
            atomicAdd(&hist[qi * kHistRow + min((int)x, kBins - 1)], 1);
        }
    }
    wave_lds_sync();
    for (int r = 0; r < kMR; ++r) {
      if (__builtin_amdgcn_readlane(mode, r) != kModeHist) continue;
      int x = hist[r * kHistRow + (kBins - 1 - lane)];
      if (lane == kBins - 1) x = 0;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int t = __shfl_up(x, d, kWave);
        if (lane >= d) x += t;
      }
      const uint64_t reach = __ballot(x >= kList);
      const int new_mode = reach == 0 ? (int)kModeFallback : (int)kModeHist;
      const float bstar = reach == 0 ? 0.f : (float)(kBins - 1 - __builtin_ctzll(reach));
      if (qi == r) {
        mode = new_mode;
        gate = bstar;
      }
    }
  }

  // ---- pass 3: collect the keys whose upper bound reaches the gate
  bool fallback = __ballot(mode == kModeFallback) != 0;
  if (!fallback) {
    if (lane < kMR) ccount[wave][lane] = 0;
    wave_lds_sync();
    for (int t0 = kbeg; t0 < kend; t0 += kTile) {
      f32x4_t acc[4];
      float e[4][4];
      tile(t0, acc, e, Three{});
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int key = t0 + 16 * sub + 4 * g + v;
          const bool take = key < my_lim &&
                            (mode == kModeAll || fmaf(acc[sub][v] + e[sub][v], inv_w, off) >= gate);
          if (take) {
            const int pos = atomicAdd(&ccount[wave][qi], 1);
            if (pos < kCollect) cand[qi * kCandRow + pos] = key;
          }
        }
    }
    wave_lds_sync();
    fallback = __ballot(lane < kMR && ccount[wave][lane < kMR ? lane : 0] > kCollect) != 0;
  }
  if (lane == 0) redo[lb * kMfmaWaves + wave] = fallback ? 1 : 0;
  if (fallback) return;

  // ---- rescoring in float64 and the exact top-64 of each row
  const size_t kbase = bg * N_cap;
  for (int r = 0; r < kMR; ++r) {
    const int i = row0 + r;
    if (i >= Q) break;
    const int c = ccount[wave][r];
    KeyF64 best = KO::pad();
    for (int base = 0; base < c; base += kWave) {
      KeyF64 x = KO::pad();
      if (base + lane < c) {
        const int j = cand[r * kCandRow + base + lane];
        double acc = 0.0;
        if constexpr (KBF) {
          const uint16_t* kr = reinterpret_cast<const uint16_t*>(keys) + (kbase + j) * D;
#pragma unroll 4
          for (int d8 = 0; d8 < D; d8 += 8) {
            float f[8];
            unpack_piece<true>(*reinterpret_cast<const uint4*>(kr + d8), f);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fma((double)qrows[r * D + d8 + e], (double)f[e], acc);
          }
        } else {
          const float* kr = reinterpret_cast<const float*>(keys) + (kbase + j) * D;
#pragma unroll 4
          for (int d4 = 0; d4 < D; d4 += 4) {
            const float4 f = *reinterpret_cast<const float4*>(kr + d4);
            acc = fma((double)qrows[r * D + d4 + 0], (double)f.x, acc);
            acc = fma((double)qrows[r * D + d4 + 1], (double)f.y, acc);
            acc = fma((double)qrows[r * D + d4 + 2], (double)f.z, acc);
            acc = fma((double)qrows[r * D + d4 + 3], (double)f.w, acc);
          }
        }
        x = KO::make(acc, j);
      }
      wave_sort<KO>(x);
      if (base == 0) best = x;
      else wave_merge<KO>(best, x);
    }
    exact_row_out<KO>(best, bh * Q + i, ch, n_chunks, k, approx, hits, exact_idx, part);
  }
}

// ---------------------------------------------------------------- exact scores, gated by the candidate list

// The k-th best exact score among any k distinct visible keys is a lower
// bound of the row's exact k-th score, so the candidate list S_i itself gives
// every row a gate tau_i before the scan.  The gate is taken from float32 dot
// products, whose error is at most gamma_128 sum|q_e k_e| <= 7.7e-6 ||q|| ||k||.
constexpr float kTauEps = 1e-5f;

// Order-preserving 32-bit key of a float score whose low 7 bits carry a slot
// number (0..127); 0 is never produced for a finite score and marks a pad.
__device__ __forceinline__ uint32_t slot_key(float s, int slot) {
  return (ord_f32(s) & ~127u) | (uint32_t)slot;
}

__device__ __forceinline__ float wave_min_f32(float v) {
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v = fminf(v, xor_shfl_f32(v, m));
  return v;
}
__device__ __forceinline__ float wave_max_f32(float v) {
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v = fmaxf(v, xor_shfl_f32(v, m));
  return v;
}

// Float32 q.k of one key per lane (four partial sums); q in LDS.
template <bool KBF>
__device__ __forceinline__ float lane_dot_f32(const void* keys, size_t key_row, const float* qs) {
  constexpr int D = saki::kHeadDim;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
  for (int d8 = 0; d8 < D; d8 += 8) {
    float f[8];
    if constexpr (KBF) {
      unpack_piece<true>(*reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) +
                                                         key_row * D + d8), f);
    } else {
      const float4* kr = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(keys) +
                                                         key_row * D + d8);
      const float4 a = kr[0], b = kr[1];
      f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
      f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) s[e & 3] = fmaf(qs[d8 + e], f[e], s[e & 3]);
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}

// Float64 q.k of one key per lane (float32 inputs: every product is exact).
template <bool KBF>
__device__ __forceinline__ double lane_dot_f64(const void* keys, size_t key_row, const float* qs) {
  constexpr int D = saki::kHeadDim;
  double acc = 0.0;
#pragma unroll 4
  for (int d8 = 0; d8 < D; d8 += 8) {
    float f[8];
    if constexpr (KBF) {
      unpack_piece<true>(*reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) +
                                                         key_row * D + d8), f);
    } else {
      const float4* kr = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(keys) +
                                                         key_row * D + d8);
      const float4 a = kr[0], b = kr[1];
      f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
      f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fma((double)qs[d8 + e], (double)f[e], acc);
  }
  return acc;
}

// Whether j is in a row's candidate list, kept sorted descending in LDS
// (64 entries; unused slots hold values >= 2^31, which no index equals).
__device__ __forceinline__ bool in_sorted_desc(const uint32_t* a, int j) {
  if (j < 0) return false;
  const uint32_t x = (uint32_t)j;
  int lo = 0;
#pragma unroll
  for (int st = 32; st > 0; st >>= 1)
    if (a[lo + st - 1] > x) lo += st;
  return lo < kWave && a[lo] == x;
}

// Float64 q.k of one key per lane, q read from global memory.
template <bool KBF>
__device__ __forceinline__ double lane_dot_f64_g(const void* keys, size_t key_row,
                                                 const float* __restrict__ qr) {
  constexpr int D = saki::kHeadDim;
  double acc = 0.0;
#pragma unroll 2
  for (int d8 = 0; d8 < D; d8 += 8) {
    float f[8];
    if constexpr (KBF) {
      unpack_piece<true>(*reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) +
                                                         key_row * D + d8), f);
    } else {
      const float4* kr = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(keys) +
                                                         key_row * D + d8);
      const float4 a = kr[0], b = kr[1];
      f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
      f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
    }
    const float4 qa = *reinterpret_cast<const float4*>(qr + d8);
    const float4 qb = *reinterpret_cast<const float4*>(qr + d8 + 4);
    const float qv[8] = {qa.x, qa.y, qa.z, qa.w, qb.x, qb.y, qb.z, qb.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fma((double)qv[e], (double)f[e], acc);
  }
  return acc;
}

constexpr int kGateCap = 64;            // keys one wave collects per row
constexpr int kGateRow = kGateCap + 1;  // row stride; slot kGateCap absorbs overflow writes
constexpr int kBatch = 160;             // keys rescored per wave and batch
constexpr int kGateWaves = 4;           // waves per 16-row work-group

// Float64 partial q.k over dims 32p .. 32p+31 of one key: the four lanes of
// a quad (p = lane & 3) share a key, and quad_sum_f64 completes the sum.
// Every load of the lane is issued before its products.
template <bool KBF>
__device__ __forceinline__ double quad_dot_f64(const void* keys, size_t key_row,
                                               const float* __restrict__ qr, int p) {
  constexpr int D = saki::kHeadDim;
  float f[32], qv[32];
  if constexpr (KBF) {
    const uint4* kr = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) +
                                                     key_row * D + 32 * p);
#pragma unroll
    for (int u = 0; u < 4; ++u) unpack_piece<true>(kr[u], f + 8 * u);
  } else {
    const float4* kr = reinterpret_cast<const float4*>(reinterpret_cast<const float*>(keys) +
                                                       key_row * D + 32 * p);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const float4 v = kr[u];
      f[4 * u] = v.x; f[4 * u + 1] = v.y; f[4 * u + 2] = v.z; f[4 * u + 3] = v.w;
    }
  }
  const float4* q4 = reinterpret_cast<const float4*>(qr + 32 * p);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const float4 v = q4[u];
    qv[4 * u] = v.x; qv[4 * u + 1] = v.y; qv[4 * u + 2] = v.z; qv[4 * u + 3] = v.w;
  }
  double a0 = 0.0, a1 = 0.0;
#pragma unroll
  for (int e = 0; e < 32; e += 2) {
    a0 = fma((double)qv[e], (double)f[e], a0);
    a1 = fma((double)qv[e + 1], (double)f[e + 1], a1);
  }
  return a0 + a1;
}
// The sum over the four lanes of a quad; every lane gets the same bits.
__device__ __forceinline__ double quad_sum_f64(double v) {
  v += __longlong_as_double((long long)xor_shfl_u64((uint64_t)__double_as_longlong(v), 1));
  return v + __longlong_as_double((long long)xor_shfl_u64((uint64_t)__double_as_longlong(v), 2));
}

// Exact top-k and recall hits in one scan.  A row's candidate list S (k
// distinct visible keys) gives the gate tau = min over S of a float32 lower
// bound of q.k; the scan collects C = {j : a3_j + E_j >= tau} with the bf16x3
// upper bound, so C contains the exact top-k T and, since every key of S
// passes, S as well.  Only the keys of C outside S (normally a handful) are
// rescored in float64.  Then, with |S| = k,
//   hits = |T intersect S| = k - |T intersect (C \ S)|,
// and a key o of C \ S is in T iff fewer than k keys of C beat it: the keys
// of S are compared through their float32 intervals (an undecided pair is
// settled in float64) and the others exactly.  With exact_idx or split keys
// the exact order is needed: S's keys in the chunk are rescored as well and
// merged with the others.  A row whose list is invalid (an entry outside
// [0, lim) or a duplicate) takes tau = -inf and treats all of C as others.
//
// A work-group of four waves owns 16 rows: the waves take four rows each for
// the gate and the final count, and every fourth key tile of the scan (all
// 16 rows, one collection list per wave and row, filled without atomics: the
// four lanes of a row append at offsets from a prefix of their counts), so
// that the latency of the per-row work is spread over four times as many
// waves.  A work-group in which one wave collects more than 64 keys for a
// row, or a row has more than 160 others, is flagged for exact_bf16_kernel.
// grid: 1-D xcd grid of ceil(Q / 16) * n_chunks * B * H_q work-groups; the
// flags use the numbering of the two-wave tiers.
template <bool KBF>
__global__ __launch_bounds__(kGateWaves * kWave) __attribute__((amdgpu_waves_per_eu(4))) void exact_gate_kernel(
    const void* __restrict__ keys, const uint8_t* __restrict__ khi,
    const uint8_t* __restrict__ klo, const float* __restrict__ knorm, const float* __restrict__ q,
    const int* __restrict__ q_pos, int H_q, int H_kv, int N_cap, int N_valid, int Q,
    int n_tiles_hi, int n_bh, int row_blocks2, int chunk, int n_chunks, int k,
    const int* __restrict__ approx, int* __restrict__ hits, int* __restrict__ exact_idx,
    KeyF64* __restrict__ part, int* __restrict__ redo) {
  constexpr int D = saki::kHeadDim;
  constexpr size_t TB = (size_t)kTile * D * 2;
  using KD = KeysF64;
  __shared__ int cj[kGateWaves][kMR * kGateRow];  // keys collected by each scanning wave
  __shared__ uint32_t sl[kMR * kWave];   // candidate lists, sorted descending
  __shared__ float ss[kMR * kWave];      // float32 score of sorted entry a
  __shared__ float se[kMR * kWave];      // and its error radius
  __shared__ float tau_s[kMR];           // gates
  __shared__ int bad_s[kMR];             // 1: invalid lists, 2: rows of at most k keys
  __shared__ int ccount[kGateWaves][kMR];
  __shared__ int wg_fallback;
  __shared__ int bj_m[kGateWaves][kBatch];  // per wave: others' key, exact score, row
  __shared__ double bsc_m[kGateWaves][kBatch];
  __shared__ unsigned char brow_m[kGateWaves][kBatch];
  __shared__ int boff_m[kGateWaves][kMR / kGateWaves + 1];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int row_blocks = (Q + kMR - 1) / kMR;
  const long long lb = xcd_logical_block((long long)row_blocks * n_chunks * n_bh);
  if (lb < 0) return;  // uniform over the work-group
  const int rb = (int)(lb % row_blocks), ch = (int)((lb / row_blocks) % n_chunks);
  const size_t bh = (size_t)(lb / ((long long)row_blocks * n_chunks));
  const int b = (int)(bh / H_q), h = (int)(bh % H_q);
  const int gkv = h / (H_q / H_kv);
  const size_t bg = (size_t)b * H_kv + gkv;
  const int row0 = rb * kMR;  // < Q
  const long long flag =
      (((long long)bh * n_chunks + ch) * row_blocks2 + rb / 2) * kMfmaWaves + (rb % 2);
  const int qi = lane % 16, g = lane / 16;
  const int my_row = row0 + qi;
  const bool row_ok = my_row < Q;
  const int my_lim = row_limit(my_row, Q, N_valid, q_pos);
  const int kmax = wave_max_i(my_lim);
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  const int n_rows = min(kMR, Q - row0);
  const bool ordered = exact_idx != nullptr || n_chunks > 1;
  const size_t hoff = bg * n_tiles_hi * TB;
  const float* kn = knorm + bg * n_tiles_hi * kTile;
  const size_t kbase = bg * N_cap;
  int* bj = bj_m[wave];
  double* bsc = bsc_m[wave];
  unsigned char* brow = brow_m[wave];
  int* boff = boff_m[wave];

  // ---- gate, part 1: load, sort and check the candidate lists of rows wave,
  //      wave + 4, ... (the next row's list is loaded before this one is
  //      sorted); the owner wave also sets the row's gate to -inf and its
  //      validity flag (rows past Q count as invalid)
  {
    auto list_entry = [&](int r) -> int {
      return r < n_rows && lane < k ? approx[(bh * Q + row0 + r) * k + lane] : -1;
    };
    int aj_next = list_entry(wave);
#pragma unroll 1
    for (int r = wave; r < kMR; r += kGateWaves) {
      const int aj = aj_next;
      aj_next = list_entry(r + kGateWaves);
      if (lane == 0) tau_s[r] = -INFINITY;
      if (r >= n_rows) {
        if (lane == 0) bad_s[r] = 1;
        continue;
      }
      const int lim_r = __builtin_amdgcn_readlane(my_lim, r);
      bool bad = lane < k && (aj < 0 || aj >= lim_r);
      uint32_t key = lane < k ? (uint32_t)aj : (0x80000000u | (uint32_t)lane);
      wave_sort<KeysU32>(key);
      const uint32_t nxt = (uint32_t)__shfl_down((int)key, 1, kWave);
      const bool dup = lane < kWave - 1 && key == nxt;
      sl[r * kWave + lane] = key;
      // every visible key is in T if its score is a number (finite operands;
      // kbeg = 0, one chunk: the norms of the first tile)
      bool odd = true;
      if (!ordered && lim_r <= k) {
        const float* qr = q + (bh * Q + row0 + r) * saki::kHeadDim;
        odd = !isfinite(qr[lane]) || !isfinite(qr[kWave + lane]) || (lane < lim_r && !isfinite(kn[lane]));
      }
      if (__ballot(odd) == 0) {
        // the list's distinct visible keys count, and the row is done (gate
        // +inf).  As a row without a gate, each of them would be rescored and
        // ranked.
        const int n = __popcll(__ballot(key < (uint32_t)lim_r && !dup));
        if (lane == 0) {
          hits[bh * Q + row0 + r] = n;
          tau_s[r] = INFINITY;
          bad_s[r] = 2;
        }
        continue;
      }
      bad |= dup;
      if (lane == 0) bad_s[r] = __ballot(bad) != 0;  // an invalid list keeps tau = -inf
    }
  }
  if (threadIdx.x == 0) wg_fallback = 0;

  // query norm bound (lanes of row qi, dims 32kk + 8g .. +7); the MFMA
  // operands are formed after the gate
  const float* qrow = q + (bh * Q + (row_ok ? my_row : row0)) * D;  // a valid row
  float qn;
  {
    float sq = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const float4 v0 = *reinterpret_cast<const float4*>(qrow + 32 * kk + 8 * g);
      const float4 v1 = *reinterpret_cast<const float4*>(qrow + 32 * kk + 8 * g + 4);
      sq = fmaf(v0.x, v0.x, sq); sq = fmaf(v0.y, v0.y, sq); sq = fmaf(v0.z, v0.z, sq); sq = fmaf(v0.w, v0.w, sq);
      sq = fmaf(v1.x, v1.x, sq); sq = fmaf(v1.y, v1.y, sq); sq = fmaf(v1.z, v1.z, sq); sq = fmaf(v1.w, v1.w, sq);
    }
    qn = row_ok ? sqrtf(sum_lane_groups(sq)) * (1.f + 1e-5f) : 0.f;
  }
  const float eq = kExactEps3 * qn;
  wave_lds_sync();

  // ---- gate, part 2: tau = min over the list of a float32 lower bound of q.k.
  //      Per row of the wave, eight steps of 8 sorted entries, 8 lanes per
  //      entry (dims 16p .. 16p+15), so each sum is at most 12 roundings deep
  //      (error <= gamma_12 ||q|| ||k||).  A row's entries and validity are
  //      read once; the steps take two key buffers in turn, each refilled
  //      right after use with the step two ahead (the next row's first two
  //      steps at the end of a row).  Pads (k < 64) and the entries of
  //      invalid lists read key 0 and are ignored.
  {
    const int p = lane & 7, slot = lane >> 3;
    const int my_rows_g = n_rows > wave ? (n_rows - wave + kGateWaves - 1) / kGateWaves : 0;
    // row rr of the wave: the key of entry 8u + slot in bit-free form (0 when
    // unused) and a bit mask of the used entries
    auto row_keys = [&](int rr, int (&jv)[8]) -> uint32_t {
      const int r = wave + kGateWaves * rr;
      const bool ok = bad_s[r] == 0;
      uint32_t used = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t kj = sl[r * kWave + 8 * u + slot];
        const bool use = ok && (kj >> 31) == 0;
        jv[u] = use ? (int)kj : 0;
        used |= use ? 1u << u : 0u;
      }
      return used;
    };
    // a key slice stays in its loaded form (four 16-byte words of float32,
    // or two of bf16) until it is used
    auto load_key = [&](uint4* w, float& knv, int j) {
      if constexpr (KBF) {
        const uint4* kr = reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) +
                                                         (kbase + j) * D + 16 * p);
        w[0] = kr[0];
        w[1] = kr[1];
      } else {
        const uint4* kr = reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(keys) +
                                                         (kbase + j) * D + 16 * p);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) w[e4] = kr[e4];
      }
      knv = kn[j];
    };
    // the query slice of the wave's row rr (dims 16p .. 16p+15)
    auto load_q = [&](float* qv, int rr) {
      const float4* qr = reinterpret_cast<const float4*>(
          q + (bh * Q + row0 + wave + kGateWaves * rr) * D + 16 * p);
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const float4 v = qr[e4];
        qv[4 * e4] = v.x; qv[4 * e4 + 1] = v.y; qv[4 * e4 + 2] = v.z; qv[4 * e4 + 3] = v.w;
      }
    };
    // the key of entry 8u + slot of row rr if used, else -1
    auto entry_key = [&](int rr, int u) -> int {
      const int r = wave + kGateWaves * rr;
      const uint32_t kj = sl[r * kWave + 8 * u + slot];
      return bad_s[r] == 0 && (kj >> 31) == 0 ? (int)kj : -1;
    };
    if (my_rows_g > 0) {
      int jv[8];
      float qcur[16], qnext[16];
      uint4 ka[KBF ? 2 : 4], kb[KBF ? 2 : 4];
      float kna, knb;
      uint32_t used = row_keys(0, jv);
      load_q(qcur, 0);
      load_key(ka, kna, jv[0]);
      load_key(kb, knb, jv[1]);
      for (int rr = 0; rr < my_rows_g; ++rr) {
        const int r = wave + kGateWaves * rr;
        const bool more = rr + 1 < my_rows_g;
        // the next row's first two keys (pads and invalid lists read key 0)
        const int n0 = more ? max(entry_key(rr + 1, 0), 0) : 0;
        const int n1 = more ? max(entry_key(rr + 1, 1), 0) : 0;
        const float qr_n = readlane_s(qn, r);
        float lo = INFINITY;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if (u == 4 && more) load_q(qnext, rr + 1);
          const uint4* w = (u & 1) ? kb : ka;
          const float knv = (u & 1) ? knb : kna;
          float f[16];
          if constexpr (KBF) {
            unpack_piece<true>(w[0], f);
            unpack_piece<true>(w[1], f + 8);
          } else {
#pragma unroll
            for (int e4 = 0; e4 < 4; ++e4) {
              f[4 * e4] = __uint_as_float(w[e4].x); f[4 * e4 + 1] = __uint_as_float(w[e4].y);
              f[4 * e4 + 2] = __uint_as_float(w[e4].z); f[4 * e4 + 3] = __uint_as_float(w[e4].w);
            }
          }
          float s0 = 0.f, s1 = 0.f;
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            s0 = fmaf(qcur[e], f[e], s0);
            s1 = fmaf(qcur[e + 1], f[e + 1], s1);
          }
          float sc = s0 + s1;
          sc += xor_shfl_f32(sc, 1);
          sc += xor_shfl_f32(sc, 2);
          sc += xor_shfl_f32(sc, 4);
          const float ea = kTauEps * qr_n * knv;
          const bool use = (used >> u) & 1u;
          if (use && p == 0) {
            ss[r * kWave + 8 * u + slot] = sc;
            se[r * kWave + 8 * u + slot] = ea;
          }
          lo = fminf(lo, use ? sc - ea : INFINITY);
          // refill this buffer with the step two ahead
          if (u + 2 < 8 || more) {
            const int j2 = u + 2 < 8 ? jv[u + 2] : (u == 6 ? n0 : n1);
            if (u & 1) load_key(kb, knb, j2);
            else load_key(ka, kna, j2);
          }
        }
        lo = wave_min_f32(lo);
        if (lane == 0 && bad_s[r] == 0) tau_s[r] = lo;
        if (more) {
          used = row_keys(rr + 1, jv);
#pragma unroll
          for (int e = 0; e < 16; ++e) qcur[e] = qnext[e];
        }
      }
    }
  }
  __syncthreads();

  // query MFMA operands: bf16 hi/lo split of dims 32kk + 8g .. +7
  bf16x8_t qh[4], ql[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    const float4 v0 = *reinterpret_cast<const float4*>(qrow + 32 * kk + 8 * g);
    const float4 v1 = *reinterpret_cast<const float4*>(qrow + 32 * kk + 8 * g + 4);
    const float fv[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
    float fh[8], fl[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float f = row_ok ? fv[e] : 0.f;
      fh[e] = bf16_round(f);
      fl[e] = bf16_round(f - fh[e]);
    }
    qh[kk] = as_bf16x8(pack_bf16x8(fh));
    ql[kk] = as_bf16x8(pack_bf16x8(fl));
  }

  // ---- scan (every fourth tile): collect the keys whose upper bound reaches
  //      the gate into this wave's lists; the four lanes of a row (lane
  //      groups g) append at offsets from a prefix of their counts
  int base = 0;  // this wave's entries for row qi so far (same in the row's four lanes)
  {
    const float my_tau = tau_s[qi];
    int* my_list = cj[wave] + qi * kGateRow;
    // a tile is 16 steps (sub-tile s, k-slice kk): each step's hi and lo
    // pieces come from a four-slot ring, refilled right after use with the
    // step four ahead (past the last tile: a repeat of a valid address)
    uint4 rh[4], rl[4];
    auto load_step = [&](int slot, int t0, int i) {
      const size_t o = hoff + (size_t)(t0 / kTile) * TB + (size_t)(4 * (i & 3) + g) * kTile * 16 +
                       (size_t)(16 * (i >> 2) + qi) * 16;
      rh[slot] = *reinterpret_cast<const uint4*>(khi + o);
      rl[slot] = *reinterpret_cast<const uint4*>(klo + o);
    };
    const int t_first = kbeg + wave * kTile;
    if (t_first < kend) {
#pragma unroll
      for (int i = 0; i < 4; ++i) load_step(i, t_first, i);
    }
    for (int t0 = t_first; t0 < kend; t0 += kGateWaves * kTile) {
      const int tn = t0 + kGateWaves * kTile < kend ? t0 + kGateWaves * kTile : t0;
      uint32_t take = 0;
#pragma unroll
      for (int sub = 0; sub < 4; ++sub) {
        const int kb = t0 + 16 * sub + 4 * g;
        const float4 nv = *reinterpret_cast<const float4*>(kn + kb);  // kb < n_tiles_hi * 64
        f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const int i = 4 * sub + kk;
          const bf16x8_t kh = as_bf16x8(rh[kk]), kl = as_bf16x8(rl[kk]);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, qh[kk], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kl, qh[kk], a, 0, 0, 0);
          a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kh, ql[kk], a, 0, 0, 0);
          if (i + 4 < 16)
            load_step(kk, t0, i + 4);
          else
            load_step(kk, tn, i - 12);
        }
        const float nvs[4] = {nv.x, nv.y, nv.z, nv.w};
#pragma unroll
        for (int v = 0; v < 4; ++v)
          take |= (kb + v < my_lim && fmaf(eq, nvs[v], a[v]) >= my_tau) ? (1u << (4 * sub + v)) : 0u;
      }
      if (__ballot(take != 0) == 0) continue;
      const int c = __popc(take);
      const int c1 = (int)xor_shfl_u32((uint32_t)c, 16);   // count of lane group g ^ 1
      const int c2 = (int)xor_shfl_u32((uint32_t)c, 32);   // g ^ 2
      const int c3 = (int)xor_shfl_u32((uint32_t)c1, 32);  // g ^ 3
      // entries of the groups below g: g=1: g^1; g=2: g^2, g^3; g=3: g^3, g^2, g^1
      int pos = base + (g == 1 ? c1 : g == 2 ? c2 + c3 : g == 3 ? c1 + c2 + c3 : 0);
      base += c + c1 + c2 + c3;
#pragma unroll
      for (int sub = 0; sub < 4; ++sub)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (take & (1u << (4 * sub + v))) {
            my_list[min(pos, kGateCap)] = t0 + 16 * sub + 4 * g + v;
            ++pos;
          }
    }
  }
  if (lane < kMR) ccount[wave][lane] = base;  // lane r < 16 holds row r
  __syncthreads();
  bool fallback = __ballot(ccount[lane / kMR][lane % kMR] > kGateCap) != 0;

  // ---- rows wave, wave + 4, ...: the others C \ S, rescored in batches of whole rows
  int r_done = 0;  // of this wave's rows
  const int my_rows = n_rows > wave ? (n_rows - wave + kGateWaves - 1) / kGateWaves : 0;
  while (!fallback && r_done < my_rows) {
    int nb = 0, r_end = r_done;
    for (; r_end < my_rows; ++r_end) {
      const int r = wave + kGateWaves * r_end;
      const bool rbad = bad_s[r] != 0;
      if (bad_s[r] == 2) {  // counted already
        if (lane == 0) boff[r_end - r_done] = boff[r_end - r_done + 1] = nb;
        continue;
      }
      // others of this row: all of C for an invalid list, else C minus S,
      // appended in one pass (entries past the batch are not written; a row
      // that does not fit is taken back and starts the next batch)
      const int nb0 = nb;
      int n_in_s = 0;
      for (int w = 0; w < kGateWaves; ++w) {
        const int c = ccount[w][r];
        for (int base = 0; base < c; base += kWave) {
          const int e = base + lane;
          const int j = e < c ? cj[w][r * kGateRow + e] : -1;
          const bool is_s = e < c && !rbad && in_sorted_desc(sl + r * kWave, j);
          const bool other = e < c && !is_s;
          const uint64_t m = __ballot(other);
          const int at = nb + prefix_count(m);
          if (other && at < kBatch) {
            bj[at] = j;
            brow[at] = (unsigned char)r;
          }
          nb += __popcll(m);
          n_in_s += __popcll(__ballot(is_s));
        }
      }
      // every key of a valid list passes the gate (a failed check means a bound
      // did not hold: hand the rows over rather than trust the result); a row
      // whose others do not fit one batch is handed over as well
      if ((!rbad && n_chunks == 1 && n_in_s != k) || nb - nb0 > kBatch) {
        fallback = true;
        break;
      }
      if (nb > kBatch) {  // this row starts the next batch
        nb = nb0;
        break;
      }
      if (lane == 0) {
        boff[r_end - r_done] = nb0;
        boff[r_end - r_done + 1] = nb;
      }
    }
    if (fallback) break;
    wave_lds_sync();

    // exact scores of the batch: four lanes per key, 16 keys per pass
    for (int base = 0; base < nb; base += kWave / 4) {
      const int e = base + lane / 4;
      const int ec = e < nb ? e : nb - 1;  // idle quads repeat the last key
      const size_t row = bh * Q + row0 + brow[ec];
      const double sx = quad_sum_f64(quad_dot_f64<KBF>(keys, kbase + bj[ec], q + row * D, lane & 3));
      if (e < nb && (lane & 3) == 0) bsc[e] = sx;
    }
    wave_lds_sync();

    // per row: the exact top-k decided by counting
    for (int rr = r_done; rr < r_end; ++rr) {
      const int r = wave + kGateWaves * rr;
      const size_t row = bh * Q + row0 + r;
      const float* qr = q + row * D;
      const bool rbad = bad_s[r] != 0;
      if (bad_s[r] == 2) continue;
      const int o0 = boff[rr - r_done], o1 = boff[rr - r_done + 1];
      // lane a: sorted list entry a (pads, k < 64, have the top bit set)
      const uint32_t kj = sl[r * kWave + lane];
      const bool real = (kj >> 31) == 0;
      const int aj = real ? (int)kj : -1;
      if (ordered) {
        KeyF64 xs = KD::pad();
        if (!rbad && real && aj >= kbeg && aj < kend)
          xs = KD::make(lane_dot_f64_g<KBF>(keys, kbase + aj, qr), aj);
        wave_sort<KD>(xs);
        for (int base = o0; base < o1; base += kWave) {
          KeyF64 xo = base + lane < o1 ? KD::make(bsc[base + lane], bj[base + lane]) : KD::pad();
          wave_sort<KD>(xo);
          wave_merge<KD>(xs, xo);
        }
        exact_row_out<KD>(xs, row, ch, n_chunks, k, approx, hits, exact_idx, part);
        continue;
      }
      // lane a: S's float32 interval of entry a
      const float sa = !rbad && real ? ss[r * kWave + lane] : 0.f;
      const float ea = !rbad && real ? se[r * kWave + lane] : 0.f;
      const double lo_a = (double)sa - (double)ea, hi_a = (double)sa + (double)ea;
      int in_t = 0, in_ts = 0;
      // others in blocks of 64, one per lane; the key compared with all of
      // them is read from its lane
      for (int base = o0; base < o1; base += kWave) {
        const int e = base + lane;
        const bool live = e < o1;
        const double so_l = live ? bsc[e] : 0.0;
        const int jo_l = live ? bj[e] : 0;
        int cnt = 0;  // keys of C that beat other e
        if (!rbad) {  // keys of S, through their intervals
          const int nbk = min(kWave, o1 - base);
          for (int t = 0; t < nbk; ++t) {
            const double so = readlane_s(so_l, t);
            const int jo = __builtin_amdgcn_readlane(jo_l, t);
            bool beat = real && lo_a > so;
            const bool amb = real && !beat && hi_a >= so;
            if (__ballot(amb) != 0 && amb) {
              const double sx = lane_dot_f64_g<KBF>(keys, kbase + aj, qr);
              beat = sx > so || (sx == so && aj < jo);
            }
            const int cs = __popcll(__ballot(beat));
            cnt += lane == t ? cs : 0;
          }
        }
        for (int base2 = o0; base2 < o1; base2 += kWave) {  // the other others, exactly
          const int e2 = base2 + lane;
          const double s2_l = base2 == base ? so_l : (e2 < o1 ? bsc[e2] : 0.0);
          const int j2_l = base2 == base ? jo_l : (e2 < o1 ? bj[e2] : 0);
          const int n2 = min(kWave, o1 - base2);
          for (int t = 0; t < n2; ++t) {
            const double s2 = readlane_s(s2_l, t);
            const int j2 = __builtin_amdgcn_readlane(j2_l, t);
            cnt += (s2 > so_l || (s2 == so_l && j2 < jo_l)) ? 1 : 0;
          }
        }
        const bool in = live && cnt < k;
        in_t += __popcll(__ballot(in));
        in_ts += __popcll(__ballot(in && rbad && in_sorted_desc(sl + r * kWave, jo_l)));
      }
      if (lane == 0) hits[row] = rbad ? in_ts : k - in_t;
    }
    wave_lds_sync();
    r_done = r_end;
  }
  if (fallback && lane == 0) atomicOr(&wg_fallback, 1);
  __syncthreads();
  if (threadIdx.x == 0) redo[flag] = wg_fallback;
}

// ---------------------------------------------------------------- exact scores, keys read once

// Exact top-k and recall hits where few rows share many keys (saki::once_better
// has the rule).  What bounds it is
// the key read from HBM, so the rows of all query heads of a KV group share
// one read: a wave holds 16 of them as MFMA columns (NB times) and streams
// one chunk of the group's keys.
//   exact_tau_kernel    per row a gate tau <= the exact k-th score, the least
//                       float32 lower bound over its candidate list (-inf for
//                       a list that is not k distinct visible keys)
//   exact_scan_kernel   bf16x3 scores a3 (error at most E = kExactEps3 ||q|| ||k||,
//                       as for exact_gate_kernel): every key with
//                       a3 + E >= tau goes to its (row, chunk) list
//   exact_decide_kernel float64 scores of a row's listed keys, their top-k
// A list that fills up (a poor candidate list, or none) raises its own gate:
// the 64th best listed a3 less the chunk's largest E so far bounds the
// chunk's 64th exact score from below, and only keys that can still reach it
// stay.  A list that stays full (many equal scores) or meets a score that is
// not finite flags its row for exact_stream_kernel.
// 2^20 float32 keys, 8 KV heads, 32 rows: 13.8 ms as one float64 dot product
// per (lane, key), which also read the keys once per query head.
constexpr int kScanCap = 128;        // entries of a (row, chunk) list
constexpr int kTauWaves = 4;         // rows per work-group of exact_tau_kernel
struct ScanEntry {
  float a;  // bf16x3 score
  int j;
};

// grid (ceil(rows / kTauWaves)), block 64 * kTauWaves: one wave per row.
template <bool KBF>
__global__ __launch_bounds__(kTauWaves * kWave) void exact_tau_kernel(
    const void* __restrict__ keys, const float* __restrict__ q, const int* __restrict__ q_pos,
    int H_q, int H_kv, int N_cap, int N_valid, int Q, int k, size_t rows,
    const int* __restrict__ approx, float* __restrict__ tau, int* __restrict__ redo) {
  constexpr int D = saki::kHeadDim;
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const size_t row = (size_t)blockIdx.x * kTauWaves + wave;
  if (row >= rows) return;
  const size_t bh = row / Q;
  const int i = (int)(row % Q);
  const int lim = row_limit(i, Q, N_valid, q_pos);
  const size_t kbase = ((bh / H_q) * H_kv + (bh % H_q) / (H_q / H_kv)) * N_cap;
  const int aj = lane < k ? approx[row * k + lane] : -1;
  bool bad = lane < k && (aj < 0 || aj >= lim);
  uint32_t sorted = lane < k ? (uint32_t)aj : (0x80000000u | (uint32_t)lane);
  wave_sort<KeysU32>(sorted);
  const uint32_t nxt = (uint32_t)__shfl_down((int)sorted, 1, kWave);
  bad |= lane < kWave - 1 && sorted == nxt;
  if (__ballot(bad) != 0) {
    if (lane == 0) {
      tau[row] = -INFINITY;
      redo[row] = 0;
    }
    return;
  }
  // eight steps of 8 entries, 8 lanes per entry (dims 16p .. 16p + 15), so that
  // a float32 sum is at most 12 roundings deep; every load is issued first
  const int p = lane & 7, slot = lane >> 3;
  float qv[16];
  float qs = 0.f;
  {
    const float4* qr = reinterpret_cast<const float4*>(q + row * D + 16 * p);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float4 v = qr[e];
      qv[4 * e] = v.x; qv[4 * e + 1] = v.y; qv[4 * e + 2] = v.z; qv[4 * e + 3] = v.w;
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) qs = fmaf(qv[e], qv[e], qs);
  }
  uint4 w[8][KBF ? 2 : 4];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int e = 8 * u + slot;
    const int j = __shfl(aj, e, kWave);
    const size_t off = (kbase + (e < k ? j : 0)) * D + 16 * p;
#pragma unroll
    for (int x = 0; x < (KBF ? 2 : 4); ++x)
      w[u][x] = KBF ? reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) + off)[x]
                    : reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(keys) + off)[x];
  }
  float lo = INFINITY;
  bool odd = false;  // a bound that is not finite
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    float f[16];
    constexpr int PE = KBF ? 8 : 4;
#pragma unroll
    for (int x = 0; x < (KBF ? 2 : 4); ++x) unpack_piece<KBF>(w[u][x], f + PE * x);
    float s0 = 0.f, s1 = 0.f, n0 = 0.f, n1 = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e += 2) {
      s0 = fmaf(qv[e], f[e], s0);
      s1 = fmaf(qv[e + 1], f[e + 1], s1);
      n0 = fmaf(f[e], f[e], n0);
      n1 = fmaf(f[e + 1], f[e + 1], n1);
    }
    float sc = s0 + s1, nn = n0 + n1, qq = qs;
#pragma unroll
    for (int m = 1; m < 8; m <<= 1) {
      sc += xor_shfl_f32(sc, m);
      nn += xor_shfl_f32(nn, m);
      qq += xor_shfl_f32(qq, m);
    }
    const float b = sc - kTauEps * (1.f + 1e-4f) * sqrtf(qq) * sqrtf(nn);
    const bool use = 8 * u + slot < k;
    lo = use ? fminf(lo, b) : lo;
    odd |= use && !isfinite(b);
  }
  lo = wave_min_f32(lo);
  if (lane == 0) {
    tau[row] = __ballot(odd) != 0 ? -INFINITY : lo;
    redo[row] = 0;
  }
}

// Rows of a KV group: rho = (query head within the group) * Q + i; a wave takes
// rows 16 NB rb .. of them and one chunk of keys.  grid: 1-D, xcd_logical_block
// order over (sequence and KV head, chunk, row block), row blocks fastest (they
// read the same keys), block 64.
template <bool KBF, int NB>
__global__ __launch_bounds__(kWave) void exact_scan_kernel(
    const void* __restrict__ keys, const float* __restrict__ q, const int* __restrict__ q_pos,
    int H_q, int H_kv, int N_cap, int N_valid, int Q, int n_bg, int row_blocks, int chunk,
    int n_chunks, const float* __restrict__ tau, ScanEntry* __restrict__ lists,
    int* __restrict__ counts, int* __restrict__ redo) {
  constexpr int D = saki::kHeadDim;
  const long long lb = xcd_logical_block((long long)row_blocks * n_chunks * n_bg);
  if (lb < 0) return;
  const int rb = (int)(lb % row_blocks), ch = (int)((lb / row_blocks) % n_chunks);
  const size_t bg = (size_t)(lb / ((long long)row_blocks * n_chunks));
  const int G = H_q / H_kv;
  const int lane = lane_id(), qi = lane % 16, g = lane / 16;
  const size_t kbase = bg * N_cap;

  // the wave's rows: query operands (bf16 hi and lo of dims d(kk, g, e), the
  // order the key loads below use), norm bounds, gates
  size_t flat[NB];
  int lim[NB], cnt[NB];
  float eq[NB], thr[NB];
  bf16x8_t qh[NB][4], ql[NB][4];
  int kmax = 0;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int rho = (rb * NB + nb) * kMR + qi;
    const bool ok = rho < G * Q;
    const int hh = ok ? rho / Q : 0, i = ok ? rho % Q : 0;
    flat[nb] = ((bg / H_kv) * H_q + (bg % H_kv) * G + hh) * Q + i;
    lim[nb] = ok ? row_limit(i, Q, N_valid, q_pos) : 0;
    kmax = max(kmax, lim[nb]);
    cnt[nb] = 0;
    thr[nb] = ok ? tau[flat[nb]] : INFINITY;
    const float* qr = q + flat[nb] * D;
    float ss = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const float4 v0 = *reinterpret_cast<const float4*>(qr + 32 * kk + (KBF ? 8 * g : 4 * g));
      const float4 v1 = *reinterpret_cast<const float4*>(qr + 32 * kk + (KBF ? 8 * g + 4 : 16 + 4 * g));
      const float f[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
      uint32_t h[4], l[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = f[2 * e], b = f[2 * e + 1];
        ss = fmaf(a, a, fmaf(b, b, ss));
        h[e] = bf16x2_bits(a, b);
        l[e] = bf16x2_bits(a - __uint_as_float(h[e] << 16), b - __uint_as_float(h[e] & 0xffff0000u));
      }
      qh[nb][kk] = as_bf16x8(uint4{h[0], h[1], h[2], h[3]});
      ql[nb][kk] = as_bf16x8(uint4{l[0], l[1], l[2], l[3]});
    }
    eq[nb] = kExactEps3 * (1.f + 1e-4f) * sqrtf(sum_lane_groups(ss));
  }
  kmax = wave_max_i(kmax);
  const int kbeg = ch * chunk;
  const int kend = min(kbeg + chunk, kmax);
  float emax = 0.f;  // the largest key norm met

  // 16 keys a step: lane (qi, g) loads of key qi the dims 32 kk + 4 g .. + 3 and
  // 32 kk + 16 + 4 g .. + 3 (float32: 64 contiguous bytes of a key per load) or
  // 32 kk + 8 g .. + 7 (bf16), clamped to the chunk's last key
  struct Raw {
    uint4 v[KBF ? 4 : 8];
  };
  auto load = [&](int t0, Raw& r) {
    const size_t row = kbase + min(t0 + qi, kend - 1);
#pragma unroll
    for (int x = 0; x < (KBF ? 4 : 8); ++x)
      r.v[x] = KBF ? *reinterpret_cast<const uint4*>(reinterpret_cast<const uint16_t*>(keys) + row * D +
                                                     32 * x + 8 * g)
                   : *reinterpret_cast<const uint4*>(reinterpret_cast<const float*>(keys) + row * D +
                                                     16 * x + 4 * g);
  };

  // row r's list (of column block nb) is full: raise its gate, keep what can
  // still reach it
  auto squeeze = [&](int nb, int r) {
    const int c = __builtin_amdgcn_readlane(cnt[nb], r);
    const size_t fr = (size_t)readlane_u64((uint64_t)flat[nb], r);
    ScanEntry* le = lists + (fr * n_chunks + ch) * kScanCap;
    const float er = readlane_s(eq[nb], r) * emax * (1.f + 1e-4f);
    __threadfence_block();  // the wave's own entries
    ScanEntry x = lane < c ? le[lane] : ScanEntry{-INFINITY, 0};
    ScanEntry y = kWave + lane < c ? le[kWave + lane] : ScanEntry{-INFINITY, 0};
    const bool odd = (lane < c && !isfinite(x.a)) || (kWave + lane < c && !isfinite(y.a)) || !isfinite(er);
    uint32_t kx = ord_f32(x.a), ky = ord_f32(y.a);
    wave_sort<KeysU32>(kx);
    wave_sort<KeysU32>(ky);
    wave_merge<KeysU32>(kx, ky);
    const float gate = unord_f32(readlane_u32(kx, kWave - 1)) - er;
    const bool tx = lane < c && x.a + er >= gate, ty = kWave + lane < c && y.a + er >= gate;
    const uint64_t mx = __ballot(tx), my = __ballot(ty);
    const int n = __popcll(mx) + __popcll(my);
    const bool full = __ballot(odd) != 0 || n > kScanCap - kMR;
    __threadfence_block();
    if (!full) {
      if (tx) le[prefix_count(mx)] = x;
      if (ty) le[__popcll(mx) + prefix_count(my)] = y;
    }
    if (qi == r) {  // a list that cannot shrink: its row is redone, nothing more is listed
      thr[nb] = full ? INFINITY : fmaxf(thr[nb], gate);
      cnt[nb] = full ? kScanCap + 1 : n;
    }
    __threadfence_block();
  };

  auto step = [&](int t0, const Raw& r) {
    f32x4_t a[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) a[nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      uint4 hv, lv;
      if constexpr (KBF) {
        hv = r.v[kk];
        float f[8];
        unpack_piece<true>(hv, f);
#pragma unroll
        for (int e = 0; e < 8; ++e) ss = fmaf(f[e], f[e], ss);
      } else {
        float f[8];
        unpack_piece<false>(r.v[2 * kk], f);
        unpack_piece<false>(r.v[2 * kk + 1], f + 4);
        uint32_t h[4], l[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = f[2 * e], y = f[2 * e + 1];
          ss = fmaf(x, x, fmaf(y, y, ss));
          h[e] = bf16x2_bits(x, y);
          l[e] = bf16x2_bits(x - __uint_as_float(h[e] << 16), y - __uint_as_float(h[e] & 0xffff0000u));
        }
        hv = uint4{h[0], h[1], h[2], h[3]};
        lv = uint4{l[0], l[1], l[2], l[3]};
      }
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        a[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(hv), qh[nb][kk], a[nb], 0, 0, 0);
        if constexpr (!KBF)
          a[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(lv), qh[nb][kk], a[nb], 0, 0, 0);
        a[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(hv), ql[nb][kk], a[nb], 0, 0, 0);
      }
    }
    // the largest norm of the 16 keys
    float kn = sum_lane_groups(ss);
#pragma unroll
    for (int m = 1; m < 16; m <<= 1) kn = vmax(kn, xor_shfl_f32(kn, m));
    kn = sqrtf(kn);
    emax = vmax(emax, kn);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const float lo = thr[nb] - eq[nb] * kn;
      uint32_t take = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) take |= (a[nb][v] < lo ? 0u : 1u) << v;  // a score that is not a number is taken
      if (__ballot(take != 0) == 0) continue;
      const int j0 = t0 + 4 * g;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (j0 + v >= min(lim[nb], kend)) take &= ~(1u << v);
      auto offsets = [&](int& pos, int& total) {  // of the row's four lanes
        const int c = __popc(take);
        const int c1 = (int)xor_shfl_u32((uint32_t)c, 16), c2 = (int)xor_shfl_u32((uint32_t)c, 32);
        const int c3 = (int)xor_shfl_u32((uint32_t)c1, 32);
        pos = g == 1 ? c1 : g == 2 ? c2 + c3 : g == 3 ? c1 + c2 + c3 : 0;
        total = c + c1 + c2 + c3;
      };
      int pos, total;
      offsets(pos, total);
      const uint64_t over = __ballot(cnt[nb] + total > kScanCap && cnt[nb] <= kScanCap) & 0xffffull;
      if (over) {
        for (uint64_t m = over; m; m &= m - 1) squeeze(nb, __builtin_ctzll(m));
        const float lo2 = thr[nb] - eq[nb] * kn;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (a[nb][v] < lo2) take &= ~(1u << v);
        offsets(pos, total);
      }
      if (cnt[nb] <= kScanCap) {  // not a row to redo
        ScanEntry* le = lists + (flat[nb] * n_chunks + ch) * kScanCap + cnt[nb] + pos;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if ((take >> v) & 1u) *le++ = ScanEntry{a[nb][v], j0 + v};
        cnt[nb] += total;
      }
    }
  };

  // two steps' loads in flight while one is scored
  if (kbeg < kend) {
    Raw r[3];
    load(kbeg, r[0]);
    load(kbeg + 16, r[1]);
    for (int t0 = kbeg; t0 < kend; t0 += 48) {
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const int t = t0 + 16 * d;
        if (t >= kend) break;
        load(t + 32, r[(d + 2) % 3]);
        step(t, r[d]);
      }
    }
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
    if (g == 0 && (rb * NB + nb) * kMR + qi < G * Q) {
      counts[flat[nb] * n_chunks + ch] = min(cnt[nb], kScanCap);
      if (cnt[nb] > kScanCap) redo[flat[nb]] = 1;  // every chunk that writes it writes 1
    }
}

// grid (rows), block 256: the row's listed keys rescored in float64 (four lanes
// per key, 64 keys a pass) and their top-k.  A round takes up to kDecideKeys
// keys, the same number at most from each of up to 256 chunks (with 8 chunks
// and 4 keys from each a round, the rounds' latency made it 35 us).  A row
// flagged for a redo is left.
constexpr int kDecideWaves = 4;
constexpr int kDecideKeys = 1024;

template <bool KBF>
__global__ __launch_bounds__(kDecideWaves * kWave) void exact_decide_kernel(
    const void* __restrict__ keys, const float* __restrict__ q, int H_q, int H_kv, int N_cap, int Q,
    int n_chunks, int k, const ScanEntry* __restrict__ lists, const int* __restrict__ counts,
    const int* __restrict__ redo, const int* __restrict__ approx, int* __restrict__ hits,
    int* __restrict__ exact_idx) {
  constexpr int D = saki::kHeadDim;
  constexpr int NT = kDecideWaves * kWave;
  using KD = KeysF64;
  __shared__ int kj[kDecideKeys];
  __shared__ double ks[kDecideKeys];
  __shared__ KeyF64 wl[kDecideWaves][kWave];
  __shared__ int n_s;
  const size_t row = blockIdx.x;
  if (redo[row] != 0) return;  // the whole work-group
  const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  const size_t bh = row / Q;
  const size_t kbase = ((bh / H_q) * H_kv + (bh % H_q) / (H_q / H_kv)) * N_cap;
  const float* qr = q + row * D;
  KeyF64 best = KD::pad();
  const int per = kDecideKeys / min(n_chunks, NT);
  for (int c0 = 0; c0 < n_chunks; c0 += NT) {
    const int c = c0 + tid;
    int left = c < n_chunks ? counts[row * n_chunks + c] : 0;
    const ScanEntry* le = lists + (row * n_chunks + (c < n_chunks ? c : 0)) * kScanCap;
    for (;;) {
      __syncthreads();
      if (tid == 0) n_s = 0;
      __syncthreads();
      const int take = min(left, per);
      if (take > 0) {
        const int at = atomicAdd(&n_s, take);
        for (int e = 0; e < take; ++e) kj[at + e] = le[e].j;
        le += take;
        left -= take;
      }
      __syncthreads();
      const int n = n_s;  // the same for every thread
      if (n == 0) break;
      for (int b = 0; b < n; b += NT / 4) {
        const int e = b + tid / 4, ec = min(e, n - 1);  // idle quads repeat the last key
        const double sx = quad_sum_f64(quad_dot_f64<KBF>(keys, kbase + kj[ec], qr, tid & 3));
        if (e < n && (tid & 3) == 0) ks[e] = sx;
      }
      __syncthreads();
      for (int b = wave * kWave; b < n; b += NT) {
        const int e = b + lane;
        // scores of -inf and those that are not numbers are never listed
        KeyF64 x = e < n && ks[e] > -(double)INFINITY ? KD::make(ks[e], kj[e]) : KD::pad();
        wave_sort<KD>(x);
        wave_merge<KD>(best, x);
      }
    }
  }
  wl[wave][lane] = best;
  __syncthreads();
  if (wave != 0) return;
  for (int w = 1; w < kDecideWaves; ++w) {
    const KeyF64 b = wl[w][lane];
    if (KD::gt(KD::readlane(b, 0), KD::readlane(best, kWave - 1))) wave_merge<KD>(best, b);
  }
  const int ej = out_index<KD>(best);
  if (exact_idx && lane < k) exact_idx[row * k + lane] = ej;
  const int hsum = row_hits(ej, approx, row, k);
  if (lane == 0) hits[row] = hsum;
}

// ---------------------------------------------------------------- merge of partials

// grid (rows), block 64 * waves (waves <= kMergeWaves): the waves of a row's
// work-group merge interleaved subsets of its sorted partial lists, then
// their lists are merged pairwise in a tree (wave w takes wave w + s's list at
// stride s = 1, 2, 4, ...).  RECALL: the row is an exact list -> exact_idx and
// hits.
// gates / redo: the gate check of score_scan_kernel's chunks (a row whose
// k-th score does not lie above every recorded gate gets redo = 1, else 0);
// only: merge just the rows flagged there.
constexpr int kMergeWaves = 16;

template <class KO, bool RECALL>
__global__ __launch_bounds__(kMergeWaves * kWave) void merge_kernel(
    const typename KO::K* __restrict__ part, size_t rows, int n_chunks, int k,
    int* __restrict__ out_idx, float* __restrict__ out_score,
    const int* __restrict__ approx, int* __restrict__ hits,
    const float* __restrict__ gates = nullptr, int* __restrict__ redo = nullptr,
    const int* __restrict__ only = nullptr) {
  using K = typename KO::K;
  __shared__ K lists[kMergeWaves][kWave];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int waves = blockDim.x / kWave;
  const size_t row = blockIdx.x;
  if (row >= rows) return;
  if (only && only[row] == 0) return;  // the rows a rescan redid, nothing else
  // wave w merges partials w, w + waves, ..., eight at a time; the next
  // eight are loaded before the current ones are merged
  constexpr int kLoads = 8;
  K a = KO::pad();
  K nb[kLoads];
  auto load = [&](int c0) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int c = c0 + u * waves;
      nb[u] = c < n_chunks ? part[(row * n_chunks + c) * kMaxK + lane] : KO::pad();
    }
  };
  if (wave < n_chunks) load(wave);
  for (int c0 = wave; c0 < n_chunks; c0 += kLoads * waves) {
    K b[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) b[u] = nb[u];
    if (c0 + kLoads * waves < n_chunks) load(c0 + kLoads * waves);
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
      // a partial is sorted: skip it when its best cannot enter the list
      if (KO::gt(KO::readlane(b[u], 0), KO::readlane(a, kWave - 1))) wave_merge<KO>(a, b[u]);
  }
  lists[wave][lane] = a;
  __syncthreads();
  for (int st = 1; st < waves; st *= 2) {  // uniform trip count: every wave reaches each barrier
    const bool active = wave % (2 * st) == 0 && wave + st < waves;
    if (active) {
      const K b = lists[wave + st][lane];
      if (KO::gt(KO::readlane(b, 0), KO::readlane(a, kWave - 1))) wave_merge<KO>(a, b);
    }
    __syncthreads();
    if (active) lists[wave][lane] = a;
    __syncthreads();
  }
  if (wave != 0) return;
  const int j = out_index<KO>(a);
  if constexpr (RECALL) {
    if (out_idx && lane < k) out_idx[row * k + lane] = j;
    const int hsum = row_hits(j, approx, row, k);
    if (lane == 0) hits[row] = hsum;
  } else {
    if (lane < k) {
      out_idx[row * k + lane] = j;
      if (out_score) out_score[row * k + lane] = (float)KO::score(a);
    }
    if (gates) {  // score_scan_kernel's chunks that kept only the keys above a gate
      float gmax = -INFINITY;
      for (int c = lane; c < n_chunks; c += kWave) gmax = fmaxf(gmax, gates[row * n_chunks + c]);
      gmax = wave_max_f32(gmax);
      // exact when every recorded gate lies below the k-th score: keys a gate
      // left out score at most the gate
      const float sk = (float)KO::score(KO::readlane(a, k - 1));
      if (lane == 0) redo[row] = (gmax == -INFINITY || sk > gmax) ? 0 : 1;
    }
  }
}

// ---------------------------------------------------------------- calibration moments

// grid: (H_q + H_kv) * nb * (nb + 1) / 2 work-groups, nb = ceil(d / 32), block
// 256.  Work-group (head, block pair bi <= bj) forms the 32 x 32 block (rows
// 32 bi.., columns 32 bj..) of that head's moment on the f64 MFMA (16x16x4: four
// tokens a step) and writes it and its mirror.  Its four waves take a quarter
// of the tokens each, their sums are added in wave order.  An operand is one
// float per lane, loaded in coalesced 64-byte pieces kMomAhead steps ahead, so
// nothing is staged.  Heads below H_q are query heads (uncentred); the rest are
// KV heads, centred by their column means, which every work-group computes for
// its own 64 columns.  As float64 FMAs over tokens staged in LDS, 64 x 64 a
// work-group, 120 of them left more than half of the CUs idle: 77 us for
// 40 heads of 512 tokens.
constexpr int kMomBlk = 32;
constexpr int kMomWaves = 4;
constexpr int kMomAhead = 8;

__global__ __launch_bounds__(kMomWaves * kWave) void moments_kernel(const float* __restrict__ q_cal,
                                                                    const float* __restrict__ k_cal, int H_q,
                                                                    int T, int d, double* __restrict__ Sq,
                                                                    double* __restrict__ Sk,
                                                                    double* __restrict__ mu_out) {
  const int nb = (d + kMomBlk - 1) / kMomBlk;
  const int npairs = nb * (nb + 1) / 2;
  const int head = blockIdx.x / npairs;
  int bi = 0, rem = blockIdx.x % npairs;  // the pair's rank in row-major order of bi <= bj
  while (rem >= nb - bi) {
    rem -= nb - bi;
    ++bi;
  }
  const int bj = bi + rem;
  const bool key = head >= H_q;
  const int hh = key ? head - H_q : head;
  const float* X = (key ? k_cal : q_cal) + (size_t)hh * T * d;
  const int tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  const int qi = lane % 16, g = lane / 16;
  const int i0 = bi * kMomBlk, j0 = bj * kMomBlk;
  constexpr int NC = 2 * kMomBlk;  // columns of both blocks
  constexpr int TP = kMomWaves * kWave / NC;
  __shared__ double mean[NC];
  __shared__ double part[TP][NC];
  __shared__ double red[kMomWaves][16][kWave];
  // column means (KV heads): TP threads per column, every TP-th token each
  if (key) {
    const int c = tid % NC, h = tid / NC;
    const int col = c < kMomBlk ? i0 + c : j0 + c - kMomBlk;
    double m = 0.0;
    if (col < d) {
#pragma unroll 16
      for (int t = h; t < T; t += TP) m += (double)X[(size_t)t * d + col];
    }
    part[h][c] = m;
  }
  __syncthreads();
  if (tid < NC) {
    double m = 0.0;
    if (key) {
#pragma unroll
      for (int h = 0; h < TP; ++h) m += part[h][tid];
      m /= (double)T;
    }
    mean[tid] = m;
  }
  __syncthreads();
  // this lane's columns: i0 + qi, i0 + 16 + qi, j0 + qi, j0 + 16 + qi (the last
  // column for those past d, whose products are not written); tokens t + g of
  // a step, zero past the wave's last
  const int steps = (T + 3) / 4, per = (steps + kMomWaves - 1) / kMomWaves;
  const int s_beg = wave * per, s_end = min(steps, s_beg + per);
  int col[4];
  double mc[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int x = 16 * (c & 1) + qi;
    col[c] = min((c < 2 ? i0 : j0) + x, d - 1);
    mc[c] = mean[(c < 2 ? 0 : kMomBlk) + x];
  }
  f64x4_t acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 2; ++e) acc[a][e] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  float nx[kMomAhead][4];
  auto load = [&](int st, float (&v)[4]) {
    const size_t row = (size_t)min(4 * st + g, T - 1) * d;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = X[row + col[c]];
  };
#pragma unroll
  for (int u = 0; u < kMomAhead; ++u) load(s_beg + u, nx[u]);
  for (int s0 = s_beg; s0 < s_end; s0 += kMomAhead) {
#pragma unroll
    for (int u = 0; u < kMomAhead; ++u) {
      const int st = s0 + u;
      const bool ok = st < s_end && 4 * st + g < T;
      double x[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) x[c] = ok ? (double)nx[u][c] - mc[c] : 0.0;
      load(st + kMomAhead, nx[u]);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int e = 0; e < 2; ++e) acc[a][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[a], x[2 + e], acc[a][e], 0, 0, 0);
    }
  }
  // register v of tile (a, e): row i0 + 16 a + g + 4 v, column j0 + 16 e + qi
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[wave][(2 * a + e) * 4 + v][lane] = acc[a][e][v];
  __syncthreads();
  double* S = key ? Sk + (size_t)hh * d * d : Sq + (size_t)hh * d * d;
#pragma unroll
  for (int u = 0; u < 16 / kMomWaves; ++u) {
    const int x = wave * (16 / kMomWaves) + u;
    double v = red[0][x][lane];
#pragma unroll
    for (int w = 1; w < kMomWaves; ++w) v += red[w][x][lane];
    v /= (double)T;
    const int i = i0 + 16 * (x / 8) + g + 4 * (x % 4), j = j0 + 16 * (x / 4 % 2) + qi;
    if (i < d && j < d) {
      S[(size_t)i * d + j] = v;
      S[(size_t)j * d + i] = v;
    }
  }
  if (key && bi == 0 && tid < kMomBlk && j0 + tid < d) mu_out[(size_t)hh * d + j0 + tid] = mean[kMomBlk + tid];
}

// ---------------------------------------------------------------- reading the winners

__device__ __forceinline__ float wave_sum_f32(float v) {
#pragma unroll
  for (int m = 1; m < kWave; m <<= 1) v += xor_shfl_f32(v, m);
  return v;
}

// theta^(-2l/d) in quarter turns per position.
__device__ __forceinline__ double rope_quarter_turns(int l, float log_theta) {
  constexpr double kTwoOverPi = 0.63661977236758134307553505349006;
  return exp(-(2.0 * l / saki::kHeadDim) * (double)log_theta) * kTwoOverPi;
}
// Sine and cosine of a quarter turns, a in float64: the nearest whole number n
// of them is taken off exactly, the rest (at most pi / 4) goes through the
// Taylor series (T: float to x^9 / x^10, double to x^13 / x^14, each below
// half a float32 step), and n picks the quadrant.
template <class T>
__device__ __forceinline__ void rope_sincos_quarters(double a, float* s, float* c) {
  constexpr double kHalfPi = 1.57079632679489661923132169163975;
  const double n = rint(a);
  const T x = (T)((a - n) * kHalfPi), y = x * x;
  T sp = (T)0, cp = (T)0;
  if constexpr (sizeof(T) == 8) {
    sp = fma(y, (T)(1.0 / 6227020800.0), (T)(-1.0 / 39916800.0));
    sp = fma(y, sp, (T)(1.0 / 362880.0));
    cp = fma(y, (T)(-1.0 / 87178291200.0), (T)(1.0 / 479001600.0));
    cp = fma(y, cp, (T)(-1.0 / 3628800.0));
  } else {
    sp = (T)(1.0 / 362880.0);
    cp = (T)(-1.0 / 3628800.0);
  }
  sp = fma(y, sp, (T)(-1.0 / 5040.0));
  sp = fma(y, sp, (T)(1.0 / 120.0));
  sp = fma(y, sp, (T)(-1.0 / 6.0));
  sp = fma(y * x, sp, x);
  cp = fma(y, cp, (T)(1.0 / 40320.0));
  cp = fma(y, cp, (T)(-1.0 / 720.0));
  cp = fma(y, cp, (T)(1.0 / 24.0));
  cp = fma(y, cp, (T)(-0.5));
  cp = fma(y, cp, (T)1.0);
  const int m = (int)(n - 4.0 * floor(0.25 * n));  // n mod 4
  const float sv = (float)((m & 1) ? cp : sp), cv = (float)((m & 1) ? sp : cp);
  *s = (m & 2) ? -sv : sv;
  *c = ((m + 1) & 2) ? -cv : cv;
}

// grid (Q, B * H_q), block 64 W: one work-group per (sequence, head, query)
// row, k <= 64.  Lane l holds dims l and l + 64 of the query and of each key, so
// that the RoPE pairs (m, m + d/2) stay inside a lane, and a key's score is a
// wave sum of the pairs' products turned by the position difference:
// rope(q, pos) . rope(k, j) depends on pos - j only.  Each wave gathers its
// 64 / W entries' keys (or, for reconstruction, unpacks their codes into LDS
// and forms mu + B_q c) and values in one round of loads, and keeps the softmax
// of its entries relative to its own maximum; the W partial results are then
// rescaled to the row's maximum and added.  Few rows are bound by the chain of
// one wave (W = 16 up to kAttendFewRows rows), many by the work in all (W = 4).
constexpr int kAttendFewRows = 512;
template <int RK, bool KBF, int ST, bool RECON, int W>
__global__ __launch_bounds__(W * kWave) void attend_kernel(
    const void* __restrict__ keys, const float* __restrict__ values,
    const uint8_t* __restrict__ index, int n_tiles, int H_q, int H_kv, int index_heads,
    int N_cap, int N_valid, const float* __restrict__ q, const int* __restrict__ q_pos, int Q,
    const float* __restrict__ Bq, const float* __restrict__ mu,
    const int* __restrict__ top_idx, int k, float log_theta, float* __restrict__ out) {
  constexpr int D = saki::kHeadDim;
  constexpr int HALF = D / 2;
  static_assert(HALF == kWave, "one RoPE pair per lane");
  constexpr int kAttendWaves = W, kAttendBatch = kWave / W;  // list entries per wave: wave w's are consecutive
  constexpr int ES = code_bytes<ST>();
  constexpr int CPP = saki::kChunkBytes / ES;
  constexpr int NP = RK / CPP;
  constexpr size_t TB = (size_t)kTile * RK * ES;
  __shared__ float bq_s[RECON ? D : 1][RECON ? RK + 1 : 1];
  __shared__ float code_s[kAttendWaves][RECON ? kAttendBatch : 1][RECON ? RK : 1];
  __shared__ float part_m[kAttendWaves], part_l[kAttendWaves];
  __shared__ float part_o[kAttendWaves][D];
  const int wave = threadIdx.x / kWave, lane = lane_id();
  const int i = blockIdx.x;
  const size_t bh = blockIdx.y;
  const int h = (int)(bh % H_q);
  const size_t b = bh / H_q;
  const int g = h / (H_q / H_kv);
  const size_t row = bh * Q + i;
  const size_t kbase = ((size_t)b * H_kv + g) * N_cap;
  const size_t cset = b * index_heads + h / (H_q / index_heads);
  const int e0 = wave * kAttendBatch;
  // lane u < kAttendBatch: list entry e0 + u (-1 past k)
  const int my_j = lane < kAttendBatch && e0 + lane < k ? top_idx[row * k + e0 + lane] : -1;
  if constexpr (RECON) {
    for (int e = threadIdx.x; e < D * RK; e += blockDim.x)
      bq_s[e / RK][e % RK] = Bq[(size_t)h * D * RK + e];
  }
  const double turn = rope_quarter_turns(lane, log_theta);
  const int pos = q_pos ? q_pos[i] : N_valid - 1;
  const float qa = q[row * D + lane], qb = q[row * D + lane + HALF];
  int jj[kAttendBatch];
#pragma unroll
  for (int u = 0; u < kAttendBatch; ++u) {
    const int j = __builtin_amdgcn_readlane(my_j, u);
    jj[u] = j < N_valid ? j : -1;  // entries outside [0, N_valid) are skipped
  }
  // keys (or codes) and values of the wave's entries; a skipped entry reads
  // row 0 and gets weight 0
  float k0[kAttendBatch], k1[kAttendBatch], v0[kAttendBatch], v1[kAttendBatch];
#pragma unroll
  for (int u = 0; u < kAttendBatch; ++u) {
    const size_t kr = (kbase + (size_t)max(jj[u], 0)) * D;
    v0[u] = values[kr + lane];
    v1[u] = values[kr + lane + HALF];
    if constexpr (!RECON) {
      k0[u] = load_key_elem<KBF>(keys, kr + lane);
      k1[u] = load_key_elem<KBF>(keys, kr + lane + HALF);
    }
  }
  if constexpr (RECON) {
    for (int t0 = 0; t0 < kAttendBatch * NP; t0 += kWave) {
      // lane t0 + lane unpacks piece p of entry u; the entry is read from
      // its lane by every lane of the wave (all lanes active)
      const int t = t0 + lane;
      const int u = min(t / NP, kAttendBatch - 1), p = t % NP;
      int j = __shfl(my_j, u, kWave);
      j = j >= 0 && j < N_valid ? j : 0;
      if (t < kAttendBatch * NP) {
        const uint4 v = *reinterpret_cast<const uint4*>(
            index + (cset * n_tiles + j / kTile) * TB + (size_t)p * kTile * 16 + (size_t)(j % kTile) * 16);
        float f[CPP];
        unpack_codes<ST>(v, f);
#pragma unroll
        for (int c = 0; c < CPP; ++c) code_s[wave][u][p * CPP + c] = f[c];
      }
    }
    __syncthreads();  // B_q staged by the work-group, codes by the wave
    const float mu0 = mu[(size_t)g * D + lane], mu1 = mu[(size_t)g * D + lane + HALF];
#pragma unroll
    for (int u = 0; u < kAttendBatch; ++u) {
      k0[u] = mu0;
      k1[u] = mu1;
    }
#pragma unroll 2
    for (int m = 0; m < RK; ++m) {  // k_hat = mu + B_q c, one code element of all 16 keys at a time
      const float b0 = bq_s[lane][m], b1 = bq_s[lane + HALF][m];
#pragma unroll
      for (int u = 0; u < kAttendBatch; ++u) {
        const float cv = code_s[wave][u][m];
        k0[u] = fmaf(b0, cv, k0[u]);
        k1[u] = fmaf(b1, cv, k1[u]);
      }
    }
  }
  float my_s = -INFINITY;  // lane u: score of entry e0 + u
#pragma unroll
  for (int u = 0; u < kAttendBatch; ++u) {
    float sn, cs;
    rope_sincos_quarters<float>(((double)pos - (double)max(jj[u], 0)) * turn, &sn, &cs);
    const float re = fmaf(qa, k0[u], qb * k1[u]), im = fmaf(qb, k0[u], -(qa * k1[u]));
    const float sc = wave_sum_f32(fmaf(cs, re, -(sn * im))) * (1.f / 11.313708498984761f);
    if (lane == u && jj[u] >= 0) my_s = sc;
  }
  // this wave's softmax terms relative to its own maximum
  const float mx = wave_max_f32(my_s);
  const float pw = my_s == -INFINITY ? 0.f : expf(my_s - mx);
  const float l = wave_sum_f32(pw);
  float o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int u = 0; u < kAttendBatch; ++u) {
    const float pe = readlane_s(pw, u);
    o0 = fmaf(pe, v0[u], o0);
    o1 = fmaf(pe, v1[u], o1);
  }
  if (lane == 0) {
    part_m[wave] = mx;
    part_l[wave] = l;
  }
  part_o[wave][lane] = o0;
  part_o[wave][lane + HALF] = o1;
  __syncthreads();
  if (wave != 0) return;
  // rescale to the row's maximum and add (an empty row writes zeros)
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kAttendWaves; ++w) M = fmaxf(M, part_m[w]);
  float L = 0.f, a0 = 0.f, a1 = 0.f;
#pragma unroll
  for (int w = 0; w < kAttendWaves; ++w) {
    const float f = part_m[w] == -INFINITY ? 0.f : expf(part_m[w] - M);
    L = fmaf(f, part_l[w], L);
    a0 = fmaf(f, part_o[w][lane], a0);
    a1 = fmaf(f, part_o[w][lane + HALF], a1);
  }
  const float il = L > 0.f ? 1.f / L : 0.f;
  out[row * D + lane] = a0 * il;
  out[row * D + lane + HALF] = a1 * il;
}

// attend_rows_kernel: the same attention for many rows.  A row
// costs one gather of its listed keys and values (64 KB, from L2) and, with a
// wave sum and 64 sines and cosines per key, was bound by the VALU (about 90
// operations per key and wave; 1,147 us for 129,024 rows over 4,096 keys).
//   - One wave per row, all rows of a work-group's range in turn.  Lane (qi, g)
//     works on dims 4 qi .. + 3 and 64 + 4 qi .. + 3 (the RoPE pairs stay inside
//     a lane) of the keys 16 b + 4 g + v, v = 0 .. 3, of step b: 16-byte loads,
//     a score is a sum over 16 lanes (four DPP adds).
//   - rope(q, pos) . rope(k, j) depends on pos - j only: per pair it is
//     cos(t) (q0 k0 + q1 k1) - sin(t) (q1 k0 - q0 k1), t = (pos - j) theta^(-2l/d).
//     For 0 <= pos - j < 64 n_hi, t = t_hi + t_lo with the sines and cosines of
//     both in LDS (64 low and n_hi high rows, float32 values rounded from
//     float64): an angle sum costs four operations.  A step with another
//     difference evaluates its angles (reduced in float64) from the pairs' turns
//     in LDS: formed anew, four exp a lane, they made reconstruction from bf16
//     codes over 131,072 keys (129,024 rows, r = 32) 1,524 us instead of 1,172.
//   - Reconstructed keys are a contraction, mu + B_q c: the codes of 16 listed
//     keys (rows) times the head's B_q (columns, in the order of the dims above,
//     so that a lane receives just its own) on the bf16 MFMA.  B_q waits in LDS
//     as three bf16 terms per element (see build_index_kernel), read once for
//     32 keys; float32 codes are split too (six products, the small ones
//     first).  As r FMAs a key and dim, 19,200 rows took 262 us at r = 32 and
//     96,000 rows 10 ms at r = 128 with float32 codes.
// The work-groups stay for the whole launch (one per CU, the table takes its
// LDS).  With B_q staged per head that pays from kAttendManyRows rows on.  Exact
// keys also need kAttendExactRows of them, as the rows that share a KV head's
// gathers, the table and its reach do.  Against attend_kernel, us, lists spread
// evenly over N float32 keys:
//   rows (H_q x Q, sequences)   N = 1,000      12,000      32,768       131,072
//   2,048 (32 x 1, 64)           23 / 24      27 / 25      30 / 26       30 / 25
//   8,192 (32 x 1, 256)          93 / 92     103 / 100    104 / 96
//   2,048 (32 x 64, 1)           14 / 19      23 / 23      28 / 24       30 / 26
//   3,584 (28 x 128, 1)          15 / 28      28 / 34      38 / 38       42 / 39
//   8,192 (32 x 256, 1)          27 / 58      54 / 65      75 / 77       87 / 85
//   129,024 (32 x 4,032, 1)     333 / 841    750 / 910  1,033 / 1,006  1,282 / 1,147
// so one query a head (and up to 63) stays with attend_kernel, and so do keys
// past kAttendFarKeys, or past the table's reach for fewer than kAttendFarRows
// rows (bf16 keys gain more at 32,768: 16,384 causal rows of 32 heads 3,099 / 3,937).
constexpr int kAttendRowWaves = 16;
constexpr int kRotLo = 64;
constexpr int kRotRows = 256;          // 128 KiB of LDS, fewer beside a large B_q
constexpr int kAttendHeadRows = 64;
constexpr int kAttendManyRows = 1536;
constexpr int kAttendExactRows = 2048;
constexpr int kAttendFarRows = 3584;
constexpr int kAttendFarKeys = 32768;
constexpr int kAttendRowsMaxCap = 1 << 22;  // a head's keys within 32-bit byte offsets

// v of lane N of this lane's row of 16
template <int N>
__device__ __forceinline__ uint32_t row_bcast_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x150 + N, 0xF, 0xF, false);
}
// Sum over the 16 lanes of a row (the same bits in each).
__device__ __forceinline__ float row_sum_f32(float v) {
  v += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x128, 0xF, 0xF, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x124, 0xF, 0xF, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x122, 0xF, 0xF, false));
  v += __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp((int)__float_as_uint(v), 0x121, 0xF, 0xF, false));
  return v;
}
// f(i) for i = 0 .. N - 1 as compile-time constants
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// grid (work-groups resident at once, at most one per 16 rows), block 1024.
// Work-group w (in XCD order, so that the rows of a KV group meet in one L2)
// takes rows [w * per_group, (w + 1) * per_group), its waves one each in turn.
// 16 codes of 16 dims fill half of an MFMA's 32; the other half is zero.
template <int RK>
constexpr int attend_bq_bytes() { return (RK + 31) / 32 * 8 * 3 * kWave * 16; }
template <bool RECON, int RK>
constexpr int attend_rot_rows() {
  return RECON ? std::min(kRotRows, (160 * 1024 - attend_bq_bytes<RK>()) / 512 - 1) : kRotRows;
}
template <int RK, bool KBF, int ST, bool RECON>
__global__ __launch_bounds__(kAttendRowWaves * kWave) void attend_rows_kernel(
    const void* __restrict__ keys, const float* __restrict__ values, const uint8_t* __restrict__ index,
    int n_tiles, int H_q, int H_kv, int index_heads, int N_cap, int N_valid, const float* __restrict__ q,
    const int* __restrict__ q_pos, int Q, const float* __restrict__ Bq, const float* __restrict__ mu,
    const int* __restrict__ top_idx, int k, float log_theta, int n_rows, int per_group, int groups,
    int n_hi, float* __restrict__ out) {
  constexpr int D = saki::kHeadDim;
  constexpr int HALF = D / 2;
  constexpr int ES = code_bytes<ST>();
  constexpr size_t TB = (size_t)kTile * RK * ES;
  constexpr int NK = (RK + 31) / 32;  // MFMA steps of 32 code dims
  __shared__ __align__(16) float rot[attend_rot_rows<RECON, RK>()][D];  // cosines of pairs 0 .. 63, then sines
  // term p of B_q[dim(mb, qi)][32 kk + 8 g .. + 7], dim(mb, qi) = 64 (mb / 4) + 4 qi + mb % 4
  __shared__ uint4 bqs[RECON ? NK : 1][RECON ? 8 : 1][RECON ? 3 : 1][RECON ? kWave : 1];
  __shared__ __align__(16) double turns[HALF];  // quarter turns per position of the pairs
  const long long lg = xcd_logical_block(groups);
  if (lg < 0) return;  // uniform over the work-group
  {
    const int l = threadIdx.x % HALF;
    const double turn = rope_quarter_turns(l, log_theta);
    if (threadIdx.x < HALF) turns[l] = turn;
    for (int e = threadIdx.x / HALF; e < kRotLo + n_hi; e += kAttendRowWaves * kWave / HALF) {
      float sn, cs;
      rope_sincos_quarters<double>((e < kRotLo ? e : (e - kRotLo) * kRotLo) * turn, &sn, &cs);
      rot[e][l] = cs;
      rot[e][HALF + l] = sn;
    }
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
  const int qi = lane % 16, g = lane / 16;
  const int r_end = (int)min((long long)n_rows, (lg + 1) * per_group);
  const int steps = (k + 15) / 16;
  const int my_e = 16 * (qi >> 2) + 4 * g + (qi & 3);  // this lane's list entry
  // with B_q staged, the rows of one head at a time (uniform over the work-group)
  for (int seg = (int)(lg * per_group), seg_end; seg < r_end; seg = seg_end) {
  const int seg_bh = seg / Q;
  seg_end = RECON ? min(r_end, (seg_bh + 1) * Q) : r_end;
  const uint8_t* cb = nullptr;
  float m0[4], m1[4];
  if constexpr (RECON) {
    const int h = seg_bh % H_q, g_kv = h / (H_q / H_kv);
    cb = index + ((size_t)(seg_bh / H_q) * index_heads + h / (H_q / index_heads)) * n_tiles * TB;
    __syncthreads();  // the previous head's reads are done
    for (int e = threadIdx.x; e < NK * 8 * kWave; e += kAttendRowWaves * kWave) {
      const int l = e % kWave, mb = e / kWave % 8, kk = e / kWave / 8;
      const int d = HALF * (mb / 4) + 4 * (l % 16) + mb % 4, c = 32 * kk + 8 * (l / 16);
      float4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
      if (c < RK) {
        const float* src = Bq + ((size_t)h * D + d) * RK + c;
        x = *reinterpret_cast<const float4*>(src);
        y = *reinterpret_cast<const float4*>(src + 4);
      }
      uint32_t t[4][3];
      split3_bf16x2(x.x, x.y, t[0]);
      split3_bf16x2(x.z, x.w, t[1]);
      split3_bf16x2(y.x, y.y, t[2]);
      split3_bf16x2(y.z, y.w, t[3]);
#pragma unroll
      for (int p = 0; p < 3; ++p) bqs[kk][mb][p][l] = uint4{t[0][p], t[1][p], t[2][p], t[3][p]};
    }
    const float4 x = *reinterpret_cast<const float4*>(mu + (size_t)g_kv * D + 4 * qi);
    const float4 y = *reinterpret_cast<const float4*>(mu + (size_t)g_kv * D + HALF + 4 * qi);
    m0[0] = x.x; m0[1] = x.y; m0[2] = x.z; m0[3] = x.w;
    m1[0] = y.x; m1[1] = y.y; m1[2] = y.z; m1[3] = y.w;
    __syncthreads();
  }
  for (int row = seg + wave; row < seg_end; row += kAttendRowWaves) {
    const int bh = RECON ? seg_bh : row / Q, i = row - bh * Q;
    const size_t kv = (size_t)(bh / H_q) * H_kv + bh % H_q / (H_q / H_kv);
    const char* kb = reinterpret_cast<const char*>(keys) + kv * N_cap * D * (KBF ? 2 : 4);
    const char* vb = reinterpret_cast<const char*>(values + kv * N_cap * D);
    int my_j = my_e < k ? top_idx[(size_t)row * k + my_e] : -1;
    if (my_j >= N_valid) my_j = -1;  // entries outside [0, N_valid) are skipped
    const int pos = q_pos ? q_pos[i] : N_valid - 1;
    const float4 q0 = *reinterpret_cast<const float4*>(q + (size_t)row * D + 4 * qi);
    const float4 q1 = *reinterpret_cast<const float4*>(q + (size_t)row * D + HALF + 4 * qi);
    const float qa[4] = {q0.x, q0.y, q0.z, q0.w}, qb[4] = {q1.x, q1.y, q1.z, q1.w};
    // a skipped entry reads row 0 and gets weight 0
    const uint32_t j_c = (uint32_t)max(my_j, 0);
    float my_s = -INFINITY;
    // scores of step b's keys (dims 4 qi + e in k0, 64 + 4 qi + e in k1)
    auto scores = [&](auto bc, const float (&k0)[4][4], const float (&k1)[4][4]) {
      constexpr int b = decltype(bc)::value;
      uint32_t jv[4];
      static_for<4>([&](auto vc) { jv[decltype(vc)::value] = row_bcast_u32<4 * b + decltype(vc)::value>(j_c); });
      float sc[4];
      const uint32_t reach = (uint32_t)(n_hi * kRotLo);
      bool far = false;
#pragma unroll
      for (int v = 0; v < 4; ++v) far |= (uint32_t)(pos - (int)jv[v]) >= reach;
      if (__ballot(far) == 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const uint32_t dp = (uint32_t)(pos - (int)jv[v]);
          const float* lo = rot[dp % kRotLo] + 4 * qi;
          const float* hi = rot[kRotLo + dp / kRotLo] + 4 * qi;
          const float4 cl4 = *reinterpret_cast<const float4*>(lo), sl4 = *reinterpret_cast<const float4*>(lo + HALF);
          const float4 ch4 = *reinterpret_cast<const float4*>(hi), sh4 = *reinterpret_cast<const float4*>(hi + HALF);
          const float cl[4] = {cl4.x, cl4.y, cl4.z, cl4.w}, sl[4] = {sl4.x, sl4.y, sl4.z, sl4.w};
          const float ch[4] = {ch4.x, ch4.y, ch4.z, ch4.w}, sh[4] = {sh4.x, sh4.y, sh4.z, sh4.w};
          float acc = 0.f;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float cs = fmaf(ch[e], cl[e], -(sh[e] * sl[e])), sn = fmaf(sh[e], cl[e], ch[e] * sl[e]);
            acc = fmaf(cs, fmaf(qa[e], k0[v][e], qb[e] * k1[v][e]), acc);
            acc = fmaf(-sn, fmaf(qb[e], k0[v][e], -(qa[e] * k1[v][e])), acc);
          }
          sc[v] = row_sum_f32(acc);
        }
      } else {
        double turn[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) turn[e] = turns[4 * qi + e];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double dp = (double)pos - (double)jv[v];
          float acc = 0.f;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float sn, cs;
            rope_sincos_quarters<float>(dp * turn[e], &sn, &cs);
            acc = fmaf(cs, fmaf(qa[e], k0[v][e], qb[e] * k1[v][e]), acc);
            acc = fmaf(-sn, fmaf(qb[e], k0[v][e], -(qa[e] * k1[v][e])), acc);
          }
          sc[v] = row_sum_f32(acc);
        }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) my_s = qi == 4 * b + v ? sc[v] : my_s;
    };
    if constexpr (!RECON) static_for<4>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if (b >= steps) return;
      float k0[4][4], k1[4][4];
      static_for<4>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        const uint32_t jv = row_bcast_u32<4 * b + v>(j_c);
        if constexpr (KBF) {
          const uint32_t off = jv * (uint32_t)(D * 2) + (uint32_t)(8 * qi);
          const uint2 x = *reinterpret_cast<const uint2*>(kb + off);
          const uint2 y = *reinterpret_cast<const uint2*>(kb + off + D);
          k0[v][0] = __uint_as_float(x.x << 16); k0[v][1] = __uint_as_float(x.x & 0xffff0000u);
          k0[v][2] = __uint_as_float(x.y << 16); k0[v][3] = __uint_as_float(x.y & 0xffff0000u);
          k1[v][0] = __uint_as_float(y.x << 16); k1[v][1] = __uint_as_float(y.x & 0xffff0000u);
          k1[v][2] = __uint_as_float(y.y << 16); k1[v][3] = __uint_as_float(y.y & 0xffff0000u);
        } else {
          const uint32_t off = jv * (uint32_t)(D * 4) + (uint32_t)(16 * qi);
          const float4 x = *reinterpret_cast<const float4*>(kb + off);
          const float4 y = *reinterpret_cast<const float4*>(kb + off + HALF * 4);
          k0[v][0] = x.x; k0[v][1] = x.y; k0[v][2] = x.z; k0[v][3] = x.w;
          k1[v][0] = y.x; k1[v][1] = y.y; k1[v][2] = y.z; k1[v][3] = y.w;
        }
      });
      scores(bc, k0, k1);
    });
    // reconstruction, two steps (32 keys) for each read of B_q
    if constexpr (RECON) static_for<2>([&](auto pc) {
      constexpr int p2 = 2 * decltype(pc)::value;
      if (p2 >= steps) return;
      f32x4_t acc[2][8];
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) acc[s2][mb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      // lane (qi, g): code dims 32 kk + 8 g .. + 7 of list entry 16 b + qi
      const uint8_t* src[2];
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        const uint32_t j = (uint32_t)__shfl((int)j_c, 16 * ((qi >> 2) & 3) + 4 * (p2 + s2) + (qi & 3), kWave);
        src[s2] = cb + (size_t)(j / kTile) * TB + (size_t)(j % kTile) * 16;
      }
#pragma unroll 1
      for (int kk = 0; kk < NK; ++kk) {
        const bool in = 32 * kk + 8 * g < RK;  // RK = 16: lane groups 2 and 3 hold zeros
        const int c = in ? 32 * kk + 8 * g : 0;
        bf16x8_t cv[2][ST == kStF32 ? 3 : 1];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          if constexpr (ST == kStF32) {
            const uint4 x = *reinterpret_cast<const uint4*>(src[s2] + (size_t)(c / 4) * kTile * 16);
            const uint4 y = *reinterpret_cast<const uint4*>(src[s2] + (size_t)(c / 4 + 1) * kTile * 16);
            float f[8];
            unpack_piece<false>(x, f);
            unpack_piece<false>(y, f + 4);
            uint32_t t[4][3];
#pragma unroll
            for (int e = 0; e < 4; ++e) split3_bf16x2(in ? f[2 * e] : 0.f, in ? f[2 * e + 1] : 0.f, t[e]);
#pragma unroll
            for (int p = 0; p < 3; ++p) cv[s2][p] = as_bf16x8(uint4{t[0][p], t[1][p], t[2][p], t[3][p]});
          } else if constexpr (ST == kStBf16) {
            const uint4 x = *reinterpret_cast<const uint4*>(src[s2] + (size_t)(c / 8) * kTile * 16);
            cv[s2][0] = as_bf16x8(in ? x : uint4{0u, 0u, 0u, 0u});
          } else {
            const uint2 x = *reinterpret_cast<const uint2*>(src[s2] + (size_t)(c / 16) * kTile * 16 + c % 16);
            const uint2 w0 = e4m3x4_to_bf16(in ? x.x : 0u), w1 = e4m3x4_to_bf16(in ? x.y : 0u);
            cv[s2][0] = as_bf16x8(uint4{w0.x, w0.y, w1.x, w1.y});
          }
        }
#pragma unroll
        for (int mb = 0; mb < 8; ++mb) {
          const bf16x8_t w1 = as_bf16x8(bqs[kk][mb][0][lane]), w2 = as_bf16x8(bqs[kk][mb][1][lane]),
                         w3 = as_bf16x8(bqs[kk][mb][2][lane]);
#pragma unroll
          for (int s2 = 0; s2 < 2; ++s2) {
            f32x4_t a = acc[s2][mb];
            if constexpr (ST == kStF32) {
              a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][2], w1, a, 0, 0, 0);
              a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][1], w2, a, 0, 0, 0);
            }
            a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][0], w3, a, 0, 0, 0);
            if constexpr (ST == kStF32) a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][1], w1, a, 0, 0, 0);
            a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][0], w2, a, 0, 0, 0);
            acc[s2][mb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cv[s2][0], w1, a, 0, 0, 0);
          }
        }
      }
      static_for<2>([&](auto sc2) {
        constexpr int s2 = decltype(sc2)::value;
        if (p2 + s2 >= steps) return;
        float k0[4][4], k1[4][4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            k0[v][e] = m0[e] + acc[s2][e][v];
            k1[v][e] = m1[e] + acc[s2][4 + e][v];
          }
        scores(std::integral_constant<int, p2 + s2>{}, k0, k1);
      });
    });
    // softmax over the row's entries, one per lane
    my_s = my_j >= 0 ? my_s * (1.f / 11.313708498984761f) : -INFINITY;
    const float mx = wave_max_f32(my_s);
    const float p = my_s == -INFINITY ? 0.f : expf(my_s - mx);
    const float l = wave_sum_f32(p);
    const float il = l > 0.f ? 1.f / l : 0.f;  // a row without entries writes zeros
    float o0[4] = {0.f, 0.f, 0.f, 0.f}, o1[4] = {0.f, 0.f, 0.f, 0.f};
    static_for<4>([&](auto bc) {
      constexpr int b = decltype(bc)::value;
      if (b >= steps) return;
      static_for<4>([&](auto vc) {
        constexpr int v = decltype(vc)::value;
        const uint32_t off = row_bcast_u32<4 * b + v>(j_c) * (uint32_t)(D * 4) + (uint32_t)(16 * qi);
        const float pv = __uint_as_float(row_bcast_u32<4 * b + v>(__float_as_uint(p)));
        const float4 x = *reinterpret_cast<const float4*>(vb + off);
        const float4 y = *reinterpret_cast<const float4*>(vb + off + HALF * 4);
        o0[0] = fmaf(pv, x.x, o0[0]); o0[1] = fmaf(pv, x.y, o0[1]);
        o0[2] = fmaf(pv, x.z, o0[2]); o0[3] = fmaf(pv, x.w, o0[3]);
        o1[0] = fmaf(pv, y.x, o1[0]); o1[1] = fmaf(pv, y.y, o1[1]);
        o1[2] = fmaf(pv, y.z, o1[2]); o1[3] = fmaf(pv, y.w, o1[3]);
      });
    });
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o0[e] = sum_lane_groups(o0[e]) * il;
      o1[e] = sum_lane_groups(o1[e]) * il;
    }
    float* op = out + (size_t)row * D + 4 * qi;
    if (g == 0) *reinterpret_cast<float4*>(op) = float4{o0[0], o0[1], o0[2], o0[3]};
    if (g == 1) *reinterpret_cast<float4*>(op + HALF) = float4{o1[0], o1[1], o1[2], o1[3]};
  }
  }
}

// Work-groups of `kernel` (block `threads`) resident on the whole current
// device at once, or 0 if the runtime cannot tell.  Cached per (kernel,
// block size, device).
template <class K>
int resident_groups(K kernel, int threads, size_t lds = 0) {
  static std::mutex mu;
  static std::map<std::tuple<const void*, int, int>, int> cache;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  const auto key = std::make_tuple(reinterpret_cast<const void*>(kernel), threads, dev);
  {
    std::lock_guard<std::mutex> lock(mu);
    const auto it = cache.find(key);
    if (it != cache.end()) return it->second;
  }
  int cus = 0, per_cu = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  std::lock_guard<std::mutex> lock(mu);
  cache[key] = cus * per_cu;
  return cus * per_cu;
}

template <int RK, bool KBF, int ST, bool RECON>
void launch_attend(const void* keys, const float* values, const uint8_t* index, int B, int H_q,
                   int H_kv, int index_heads, int N_cap, int N_valid, const float* q,
                   const int* q_pos, int Q, const float* Bq, const float* mu, const int* top_idx,
                   int k, float rope_theta, float* out, hipStream_t s) {
  const size_t rows = (size_t)B * H_q * Q;
  {
    // 16-byte loads of keys (or B_q and mu), values, queries and the output; a
    // head's rows within 32-bit byte offsets
    const uintptr_t src = RECON ? reinterpret_cast<uintptr_t>(Bq) | reinterpret_cast<uintptr_t>(mu)
                                : reinterpret_cast<uintptr_t>(keys);
    const bool al = ((src | reinterpret_cast<uintptr_t>(values) | reinterpret_cast<uintptr_t>(q) |
                      reinterpret_cast<uintptr_t>(out)) & 15) == 0;
    const size_t far_keys = rows >= (size_t)kAttendFarRows ? kAttendFarKeys : (kRotRows - kRotLo) * kRotLo;
    const bool many = RECON ? rows >= (size_t)kAttendManyRows
                            : rows >= (size_t)kAttendExactRows && (size_t)N_valid <= far_keys;
    if (al && many && Q >= kAttendHeadRows && rows <= 0x7fffffffu && N_cap <= kAttendRowsMaxCap) {
      const int slots = resident_groups(attend_rows_kernel<RK, KBF, ST, RECON>, kAttendRowWaves * kWave);
      if (slots > 0) {
        const int per = std::max(kAttendRowWaves, (int)((rows + slots - 1) / slots));
        const int groups = (int)((rows + per - 1) / per);
        const int n_hi = std::min(attend_rot_rows<RECON, RK>() - kRotLo, (N_valid + kRotLo - 1) / kRotLo);
        hipLaunchKernelGGL((attend_rows_kernel<RK, KBF, ST, RECON>),
                           dim3((unsigned)((groups + kXcds - 1) / kXcds * kXcds)), dim3(kAttendRowWaves * kWave),
                           0, s, keys, values, index, (int)saki::n_tiles(N_cap), H_q, H_kv, index_heads, N_cap,
                           N_valid, q, q_pos, Q, Bq, mu, top_idx, k, logf(rope_theta), (int)rows, per, groups, n_hi,
                           out);
        return;
      }
    }
  }
  dim3 grid((unsigned)Q, (unsigned)(B * H_q));
  const int nt = (int)saki::n_tiles(N_cap);
  if (rows <= (size_t)kAttendFewRows)
    hipLaunchKernelGGL((attend_kernel<RK, KBF, ST, RECON, 16>), grid, dim3(16 * kWave), 0, s, keys, values, index, nt,
                       H_q, H_kv, index_heads, N_cap, N_valid, q, q_pos, Q, Bq, mu, top_idx, k, logf(rope_theta), out);
  else
    hipLaunchKernelGGL((attend_kernel<RK, KBF, ST, RECON, 4>), grid, dim3(4 * kWave), 0, s, keys, values, index, nt,
                       H_q, H_kv, index_heads, N_cap, N_valid, q, q_pos, Q, Bq, mu, top_idx, k, logf(rope_theta), out);
}

// ---------------------------------------------------------------- dispatch helpers

bool launch_ok() { return hipGetLastError() == hipSuccess; }

// 1-D grid for xcd_logical_block: 8 * ceil(total / 8) work-groups.
dim3 xcd_grid(const saki::Plan& p, int n_bh) {
  const long long total = (long long)p.row_blocks * p.n_chunks * n_bh;
  return dim3((unsigned)(((total + kXcds - 1) / kXcds) * kXcds));
}

template <int RK, bool KBF, int ST>
void launch_build(const void* keys, const float* Bk, const float* mu, int B, int H_q,
                  int H_kv, int N_cap, uint8_t* index, int n_begin, int n_end,
                  hipStream_t s) {
  if (n_end - n_begin <= kAppendKeys) {
    hipLaunchKernelGGL((append_index_kernel<RK, KBF, ST>), dim3(RK / 16, H_q, B), dim3(kWave), 0, s, keys, Bk, mu, H_q,
                       H_kv, N_cap, (int)saki::n_tiles(N_cap), index, n_begin, n_end - n_begin);
    return;
  }
  const int k0 = (n_begin / 16) * 16;
  const int per_head = n_end - n_begin <= kBuildSplitKeys ? 1 : 0;
  const long long units = (long long)(per_head ? H_q : H_kv) * B;
  // slices of at least kBuildKeys keys, about as many work-groups as the
  // device holds at once
  int slices = (n_end - k0 + kBuildKeys - 1) / kBuildKeys;
  if (!per_head) {
    const int slots = resident_groups(build_index_kernel<RK, KBF, ST>, kBuildWaves * kWave);
    if (slots > 0) slices = (int)std::max(1LL, std::min((long long)slices, kBuildRounds * slots / units));
  }
  dim3 grid(slices, per_head ? H_q : H_kv, B);
  hipLaunchKernelGGL((build_index_kernel<RK, KBF, ST>), grid, dim3(kBuildWaves * kWave), 0, s, keys, Bk, mu, H_q,
                     H_kv, N_cap, (int)saki::n_tiles(N_cap), index, n_begin, n_end, per_head);
}

// A split-N streaming launch that fills the GPU exactly once: the plan's
// chunking (which sized the workspace) is coarsened so that the work-groups
// number at most what the device holds at one time (or, given
// max_waves_per_simd, at most that many waves per SIMD), the chunk count
// staying within the plan's.  A work-group takes `chunks_per_group` chunks.
template <class K>
saki::Plan one_round(saki::Plan p, K kernel, int groups_per_chunk, int chunks_per_group,
                     int N_valid, int max_waves_per_simd = 0) {
  if (p.n_chunks <= 1) return p;
  int slots = resident_groups(kernel, kWave * p.waves);
  if (max_waves_per_simd > 0 && slots > 0) {  // at most this many waves on each of a CU's 4 SIMDs
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
      slots = min(slots, cus * 4 * max_waves_per_simd / p.waves);
  }
  if (slots <= 0) return p;
  const int want = max(1, slots / max(1, groups_per_chunk)) * chunks_per_group;
  const size_t n = N_valid > 0 ? (size_t)N_valid : 1;
  size_t chunk = saki::round_up((n + want - 1) / want, kTile);
  const int n_chunks = (int)((n + chunk - 1) / chunk);
  if (n_chunks >= p.n_chunks || chunk > saki::kMaxChunk) return p;
  p.chunk = (int)chunk;
  p.n_chunks = n_chunks;
  return p;
}

// Rows of up to kDecodeOne keys (half as many where a work-group has several
// rows) and kDecodeOneBytes of codes are one chunk: so many take about as long
// as the merge launch that two chunks would need (28 x 2 rows, bf16, r = 32:
// 8,192 keys 17.8 us, 16,384 as one chunk 25.5, cut 19.7; 32 rows, float32, r =
// 128: 8,192 keys 52 and 36).  Longer ones are cut so that the work-groups fill the GPU once, at least
// kDecodeMin keys each, in no more chunks than the plan (which sized the
// workspace) has.  Waves of a work-group (bf16 codes, r = 32):
//   up to one work-group per CU: 16 (fewer lists: 4 rows of each of 32 fp8 code
//     sets over 100,003 keys 43 us, with 8 waves 49), but 8 for short rows,
//     whose waves mostly wait for each other (32 rows over 1,024 keys 9.1 us,
//     with 16 waves 9.8; over 8,192 keys 13.2 and 13.1), and 4 for one row of
//     up to four tiles (64 keys 5.5 us, with 8 waves 5.7, with 16 6.9);
//   more work-groups than CUs: 8, as several small ones overlap their waits (4
//     rows of 512 code sets over 64 keys 13 us, with 16 waves 23; over 4,096
//     keys 38 and 50), and 4 for one row of up to kDecodeShort keys (two rows of
//     each of 1,792 code sets over 64 keys, a work-group each, 17 us, with 8
//     waves 28);
//   chunks of more than kDecodeLong keys: 8 (streaming counts then: 32 rows
//     over 2^20 keys 360 us, with 16 waves 376).
constexpr int kDecodeOne = 16384;
constexpr int kDecodeMin = 4096;
constexpr int kDecodeLong = 32768;
constexpr int kDecodeShort = 4096;              // keys
constexpr size_t kDecodeShortBytes = 256 << 10;  // of codes
constexpr size_t kDecodeOneBytes = 1 << 20;
constexpr int kDecodeCus = 256;
constexpr int kDecodeFew = 1024;
template <int RK, int ST, int R>
void launch_decode(const uint8_t* index, int nt, int B, int H_q, int H_kv, int gq, int N_valid,
                   const float* q, const int* q_pos, int Q, const float* Bq, const float* mu, int k,
                   int* top_idx, float* top_score, uint8_t* ws, const saki::Plan& p0, hipStream_t s) {
  const int n_bi = B * (H_q / gq), row_groups = (gq * Q + R - 1) / R;
  const size_t rows = (size_t)B * H_q * Q, n = N_valid > 0 ? (size_t)N_valid : 1;
  const size_t bytes = n * RK * code_bytes<ST>();
  int waves = kDecodeWaves;
  if ((long long)row_groups * n_bi > kDecodeCus)
    waves = R == 1 && n <= (size_t)kDecodeShort ? 4 : 8;
  else if (n <= (size_t)kDecodeShort && bytes <= kDecodeShortBytes)
    waves = R == 1 && n <= 4 * (size_t)kTile ? 4 : 8;
  size_t want = 1;
  if (n > (size_t)(R == 1 ? kDecodeOne : kDecodeOne / 2) || bytes > kDecodeOneBytes) {
    auto chunks = [&] {
      const long long slots =
          resident_groups(score_decode_kernel<RK, ST, R>, waves * kWave, decode_area<RK, R>(waves));
      return (size_t)std::max(1LL, slots / ((long long)row_groups * n_bi));
    };
    want = chunks();
    if (n / want > (size_t)kDecodeLong && waves > 8) {
      waves = 8;
      want = chunks();
    }
    want = std::min({want, (n + kDecodeMin - 1) / kDecodeMin, (size_t)p0.n_chunks});
  }
  const int tiles = (int)saki::n_tiles((int)n), chunk = (int)((n + want * kTile - 1) / (want * kTile));  // in tiles
  const int n_chunks = (tiles + chunk - 1) / chunk;
  uint64_t* part = n_chunks > 1 ? reinterpret_cast<uint64_t*>(ws + p0.part_off) : nullptr;
  const long long groups = (long long)row_groups * n_chunks * n_bi;
  const size_t lds = decode_area<RK, R>(waves);
  hipLaunchKernelGGL((score_decode_kernel<RK, ST, R>), dim3((unsigned)((groups + kXcds - 1) / kXcds * kXcds)),
                     dim3(waves * kWave), lds, s, index, nt, N_valid, Q, q_pos, q, Bq, mu, H_q, H_kv,
                     gq, n_bi, row_groups, chunk, n_chunks, k, top_idx, top_score, part);
  if (n_chunks > 1)
    hipLaunchKernelGGL((merge_kernel<KeysF32, false>), dim3((unsigned)rows),
                       dim3(kWave * min(kMergeWaves, n_chunks)), 0, s, part, rows, n_chunks, k, top_idx,
                       top_score, nullptr, nullptr);
}

template <int RK, int ST>
void launch_score(const uint8_t* index, int B, int H_q, int H_kv, int index_heads, int N_cap,
                  int N_valid, const float* q, const int* q_pos, int Q, const float* Bq,
                  const float* mu, int k, int* top_idx, float* top_score, uint8_t* ws,
                  const saki::Plan& p0, hipStream_t s) {
  const int gq = H_q / index_heads;
  saki::Plan p = p0;
  if (p.scan) {
    const long long wr = p0.row_blocks, per_chunk = wr * B * H_q;
    // two waves per SIMD: VALU-heavy waves of equal work, none waiting on a third
    p = one_round(p0, score_scan_kernel<RK, ST>, (int)((per_chunk + kScanWaves - 1) / kScanWaves), 1,
                  N_valid, 2);
    const int nt = (int)saki::n_tiles(N_cap);
    auto launch = [&](int chunk, int n_chunks, uint64_t* part, float* gates, const int* only) {
      const long long groups = (per_chunk * n_chunks + kScanWaves - 1) / kScanWaves;
      hipLaunchKernelGGL((score_scan_kernel<RK, ST>), dim3((unsigned)(((groups + kXcds - 1) / kXcds) * kXcds)),
                         dim3(kScanWaves * kWave), 0, s, index, nt, N_valid, Q, q_pos, q, Bq, mu, H_q,
                         H_kv, gq, B * H_q, (int)wr, chunk, n_chunks, k, top_idx, top_score, part,
                         gates, only);
    };
    if (p.n_chunks == 1) {
      launch(p.chunk, 1, nullptr, nullptr, nullptr);
      return;
    }
    // chunks, their merge with the gate check, then the flagged rows over all keys
    uint64_t* part = reinterpret_cast<uint64_t*>(ws + p.part_off);
    float* gates = reinterpret_cast<float*>(ws + p.z_off);
    int* redo = reinterpret_cast<int*>(ws + p.flag_off);
    launch(p.chunk, p.n_chunks, part, gates, nullptr);
    const size_t rows = (size_t)B * H_q * Q;
    // one wave per row: its loads of eight partial lists at a time are in
    // flight together, and few chunks leave little to split further
    hipLaunchKernelGGL((merge_kernel<KeysF32, false>), dim3((unsigned)rows), dim3(kWave), 0, s, part,
                       rows, p.n_chunks, k, top_idx, top_score, nullptr, nullptr, gates, redo);
    // the flagged rows' chunks again without a gate, and their merge
    launch(p.chunk, p.n_chunks, part, gates, redo);
    hipLaunchKernelGGL((merge_kernel<KeysF32, false>), dim3((unsigned)rows), dim3(kWave), 0, s, part,
                       rows, p.n_chunks, k, top_idx, top_score, nullptr, nullptr, nullptr, nullptr,
                       redo);
    return;
  }
  const size_t rows = (size_t)B * H_q * Q;
  const int nt = (int)saki::n_tiles(N_cap);
  if (!p.mfma) {
    // two and three rows over few keys are better work-groups of their own (two
    // rows of each of 28 bf16 code sets over 512 keys 7.3 us, together 9.9; over
    // 1,024 keys 8.9 and 12.8)
    const int n_rho = gq * Q;
    if (n_rho == 1 || (n_rho <= 3 && N_valid <= kDecodeFew))
      launch_decode<RK, ST, 1>(index, nt, B, H_q, H_kv, gq, N_valid, q, q_pos, Q, Bq, mu, k, top_idx, top_score, ws, p0, s);
    else if (n_rho == 2)
      launch_decode<RK, ST, 2>(index, nt, B, H_q, H_kv, gq, N_valid, q, q_pos, Q, Bq, mu, k, top_idx, top_score, ws, p0, s);
    else
      launch_decode<RK, ST, 4>(index, nt, B, H_q, H_kv, gq, N_valid, q, q_pos, Q, Bq, mu, k, top_idx, top_score, ws, p0, s);
    return;
  }
  uint64_t* part = p.n_chunks > 1 ? reinterpret_cast<uint64_t*>(ws + p.part_off) : nullptr;
  uint8_t* zq = ws + p.z_off;
  float* zb = reinterpret_cast<float*>(ws + p.b_off);
  int rows_per = kQsRows;
  while (rows_per > kQsWaves * kMR && (long long)((Q + rows_per - 1) / rows_per) * B * H_q < kQsGroups) rows_per /= 2;
  const int parts = (Q + rows_per - 1) / rows_per;
  const long long qs_groups = (long long)parts * B * H_q;
  hipLaunchKernelGGL((query_sketch_kernel<RK, ST>), dim3((unsigned)(((qs_groups + kXcds - 1) / kXcds) * kXcds)),
                     dim3(kQsWaves * kWave), 0, s, q, Bq, mu, Q, H_q, H_kv, B * H_q, parts, rows_per, zq, zb);
  hipLaunchKernelGGL((score_batch_kernel<RK, ST>), xcd_grid(p, B * H_q), dim3(kBWaves * kWave), 0,
                     s, index, nt, N_valid, Q, q_pos, zq, zb, H_q, gq, B * H_q,
                     p.row_blocks, p.chunk, p.n_chunks, k, top_idx, top_score, part);
  if (p.n_chunks > 1)
    hipLaunchKernelGGL((merge_kernel<KeysF32, false>), dim3((unsigned)rows),
                       dim3(kWave * min(kMergeWaves, p.n_chunks)), 0, s, part, rows, p.n_chunks,
                       k, top_idx, top_score, nullptr, nullptr);
}

// Exact float64 scores, one key per lane: all rows, or those flagged in `only`.
template <bool KBF>
void launch_exact_stream(const void* keys, const float* q, const int* q_pos, int B, int H_q,
                         int H_kv, int N_cap, int N_valid, int Q, int k, const int* approx,
                         int* hits, int* exact_idx, KeyF64* part, const int* only,
                         const saki::Plan& p, hipStream_t s) {
  const size_t rows = (size_t)B * H_q * Q;
  dim3 grid((unsigned)(p.row_blocks * p.n_chunks), B * H_q);
  dim3 block(kWave * p.waves);
  if (p.rows == 4)
    hipLaunchKernelGGL((exact_stream_kernel<KBF, 4>), grid, block, 0, s, keys, q, q_pos, H_q,
                       H_kv, N_cap, N_valid, Q, p.row_blocks, p.chunk, p.n_chunks, k, approx,
                       hits, exact_idx, part, only);
  else
    hipLaunchKernelGGL((exact_stream_kernel<KBF, 1>), grid, block, 0, s, keys, q, q_pos, H_q,
                       H_kv, N_cap, N_valid, Q, p.row_blocks, p.chunk, p.n_chunks, k, approx,
                       hits, exact_idx, part, only);
  if (p.n_chunks > 1)
    hipLaunchKernelGGL((merge_kernel<KeysF64, true>), dim3((unsigned)rows),
                       dim3(kWave * min(kMergeWaves, p.n_chunks)), 0, s, part, rows, p.n_chunks,
                       k, exact_idx, nullptr, approx, hits, nullptr, nullptr, only);
}

// The keys read once for all rows of a KV group: gates, scan, decision, and the
// rows the scan flagged.
template <bool KBF, int NB>
void launch_recall_once(const void* keys, const float* q, const int* q_pos, int B, int H_q,
                        int H_kv, int N_cap, int N_valid, int Q, int k, const int* approx,
                        int* hits, int* exact_idx, uint8_t* ws, const saki::OncePlan& p,
                        hipStream_t s) {
  const size_t rows = (size_t)B * H_q * Q;
  ScanEntry* lists = reinterpret_cast<ScanEntry*>(ws);
  int* counts = reinterpret_cast<int*>(ws + p.count_off);
  float* tau = reinterpret_cast<float*>(ws + p.tau_off);
  int* redo = reinterpret_cast<int*>(ws + p.redo_off);
  // chunks of the plan (which sized the workspace), no more than the GPU holds
  // waves of at once
  int chunk = p.chunk, n_chunks = p.n_chunks;
  const int slots = resident_groups(exact_scan_kernel<KBF, NB>, kWave);
  const int want = slots > 0 ? max(1, slots / max(1, p.row_blocks * B * H_kv)) : n_chunks;
  if (want < n_chunks) {
    chunk = (int)saki::round_up(((size_t)N_valid + want - 1) / want, kTile);
    n_chunks = (N_valid + chunk - 1) / chunk;
  }
  hipLaunchKernelGGL((exact_tau_kernel<KBF>), dim3((unsigned)((rows + kTauWaves - 1) / kTauWaves)),
                     dim3(kTauWaves * kWave), 0, s, keys, q, q_pos, H_q, H_kv, N_cap, N_valid, Q, k,
                     rows, approx, tau, redo);
  const long long total = (long long)p.row_blocks * n_chunks * B * H_kv;
  hipLaunchKernelGGL((exact_scan_kernel<KBF, NB>), dim3((unsigned)((total + kXcds - 1) / kXcds * kXcds)),
                     dim3(kWave), 0, s, keys, q, q_pos, H_q, H_kv, N_cap, N_valid, Q, B * H_kv,
                     p.row_blocks, chunk, n_chunks, (const float*)tau, lists, counts, redo);
  hipLaunchKernelGGL((exact_decide_kernel<KBF>), dim3((unsigned)rows), dim3(kDecideWaves * kWave), 0,
                     s, keys, q, H_q, H_kv, N_cap, Q, n_chunks, k, (const ScanEntry*)lists,
                     (const int*)counts, (const int*)redo, approx, hits, exact_idx);
  launch_exact_stream<KBF>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx, hits,
                           exact_idx, reinterpret_cast<KeyF64*>(ws), redo, p.stream, s);
}

template <bool KBF>
void launch_recall(const void* keys, const float* q, const int* q_pos, int B, int H_q,
                   int H_kv, int N_cap, int N_valid, int Q, int k, const int* approx,
                   int* hits, int* exact_idx, uint8_t* ws, size_t ws_bytes, const saki::Plan& p,
                   hipStream_t s) {
  const saki::OncePlan op = saki::recall_once_plan(B, H_q, H_kv, Q, N_valid);
  // its loads of keys and queries are 16 bytes wide, the other path's elements
  const bool aligned = ((reinterpret_cast<uintptr_t>(keys) | reinterpret_cast<uintptr_t>(q)) & 15) == 0;
  if (op.use && aligned && ws && ws_bytes >= op.ws_bytes) {
    if (op.nb == 2)
      launch_recall_once<KBF, 2>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx, hits,
                                 exact_idx, ws, op, s);
    else
      launch_recall_once<KBF, 1>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx, hits,
                                 exact_idx, ws, op, s);
    return;
  }
  const size_t rows = (size_t)B * H_q * Q;
  KeyF64* part = p.n_chunks > 1 ? reinterpret_cast<KeyF64*>(ws + p.part_off) : nullptr;
  if (!p.mfma) {  // a workspace of the partial lists alone, or none for a single chunk
    launch_exact_stream<KBF>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx, hits,
                             exact_idx, part, nullptr, p, s);
    return;
  }
  dim3 block(kWave * p.waves);
  const int nt_hi = (int)saki::n_tiles(N_valid);
  uint8_t* khi = ws + p.z_off;
  uint8_t* klo = khi + (size_t)B * H_kv * nt_hi * kTile * saki::kHeadDim * 2;
  float* knorm = reinterpret_cast<float*>(ws + p.b_off);
  // three tiers, each running only the waves the previous one flagged
  int* flag1 = reinterpret_cast<int*>(ws + p.flag_off);
  int* flag2 = flag1 + p.flag_count;
  if (nt_hi > 0)
    hipLaunchKernelGGL((keys_hi_kernel<KBF>), dim3(nt_hi, B * H_kv), dim3(256), 0, s, keys, N_cap,
                       N_valid, nt_hi, khi, klo, knorm);
  {
    const long long total = (long long)((Q + kMR - 1) / kMR) * p.n_chunks * B * H_q;
    hipLaunchKernelGGL((exact_gate_kernel<KBF>), dim3((unsigned)(((total + kXcds - 1) / kXcds) * kXcds)),
                       dim3(kGateWaves * kWave), 0, s, keys, khi, klo, knorm, q, q_pos, H_q, H_kv, N_cap,
                       N_valid, Q, nt_hi, B * H_q, p.row_blocks, p.chunk, p.n_chunks, k, approx,
                       hits, exact_idx, part, flag1);
  }
  hipLaunchKernelGGL((exact_bf16_kernel<KBF>), xcd_grid(p, B * H_q), block, 0, s, keys, khi,
                     klo, knorm, q, q_pos, H_q, H_kv, N_cap, N_valid, Q, nt_hi, B * H_q,
                     p.row_blocks, p.chunk, p.n_chunks, k, approx, hits, exact_idx, part,
                     (const int*)flag1, flag2);
  hipLaunchKernelGGL((exact_mfma_kernel<KBF>), xcd_grid(p, B * H_q), block, 0, s, keys, q,
                     q_pos, H_q, H_kv, N_cap, N_valid, Q, p.row_blocks, p.chunk, p.n_chunks, k,
                     approx, hits, exact_idx, part, B * H_q, (const int*)flag2);
  if (p.n_chunks > 1)
    hipLaunchKernelGGL((merge_kernel<KeysF64, true>), dim3((unsigned)rows),
                       dim3(kWave * min(kMergeWaves, p.n_chunks)), 0, s, part, rows, p.n_chunks,
                       k, exact_idx, nullptr, approx, hits);
}

bool dtype_ok(int t) { return t == SAKI_F32 || t == SAKI_BF16; }  // keys
bool sketch_ok(int t) { return t == SAKI_F32 || t == SAKI_BF16 || t == SAKI_FP8; }

// Common size validation of the GPU entry points.
int check_common(int B, int H_q, int H_kv, int N_cap, int N_valid, int d) {
  if (B <= 0 || H_q <= 0 || H_kv <= 0 || H_q % H_kv != 0 || N_cap < 0 || N_valid < 0 ||
      N_valid > N_cap || d <= 0)
    return SAKI_ERR_ARG;
  if (B > 65535 || (long long)B * H_q > 65535) return SAKI_ERR_UNSUPPORTED;
  if (d != saki::kHeadDim) return SAKI_ERR_UNSUPPORTED;
  return SAKI_OK;
}

// Scratch memory of the allocation-free score entry point: a static device
// array, one copy per GPU the library runs on (held until the process
// ends).  In host code `scratch` names a host-side stand-in, never the
// device memory: the device address comes from hipGetSymbolAddress, taken
// once per device with that device current, and only that address is
// passed to kernels.
constexpr size_t kScratchBytes = (size_t)32 << 20;

}  // namespace

static __device__ __align__(256) uint8_t scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch array (*out), or an error.
int scratch_address(void** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return SAKI_ERR_HIP;
  }
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return SAKI_ERR_HIP;
    }
    scratch_ptr[dev] = ptr;
  }
  *out = scratch_ptr[dev];
  return SAKI_OK;
}

// saki_score_topk with ws == NULL meaning the static scratch array (whose
// size the caller passes as ws_bytes).
int score_topk_impl(const void* index, int sketch_dtype, int B, int H_q, int H_kv,
                    int index_heads, int N_cap, int N_valid, int d, int r, const float* q,
                    const int* q_pos, int Q, const float* B_q, const float* mu, int k,
                    int* top_idx, float* top_score, void* ws, size_t ws_bytes, void* stream) {
  int st = check_common(B, H_q, H_kv, N_cap, N_valid, d);
  if (st != SAKI_OK) return st;
  if (Q < 0) return SAKI_ERR_ARG;
  // a code set serves whole query heads and lies within one KV group
  if (index_heads <= 0 || H_q % index_heads != 0 || index_heads % H_kv != 0) return SAKI_ERR_ARG;
  if (!sketch_ok(sketch_dtype) || !saki::rank_supported(r) || k < 1 || k > kMaxK)
    return SAKI_ERR_UNSUPPORTED;
  if (Q == 0) return SAKI_OK;
  if (!index || !q || !B_q || !mu || !top_idx) return SAKI_ERR_ARG;
  const saki::Plan p = saki::score_plan(B, H_q, index_heads, Q, N_valid, r, sketch_dtype);
  if (ws_bytes < p.ws_bytes) return SAKI_ERR_WORKSPACE;
  if (!ws) {  // the static scratch array, resolved only once the sizes fit it
    const int sst = scratch_address(&ws);
    if (sst != SAKI_OK) return sst;
  }
  if ((size_t)p.row_blocks * p.n_chunks > 0x7fffffffu) return SAKI_ERR_UNSUPPORTED;
  // the one-pass kernel's 1-D grid: one wave per (head, row block, chunk)
  if (p.scan && (size_t)B * H_q * p.row_blocks * p.n_chunks * kWave >= 0xffffffffu)
    return SAKI_ERR_UNSUPPORTED;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const uint8_t* ix = reinterpret_cast<const uint8_t*>(index);
  uint8_t* w = reinterpret_cast<uint8_t*>(ws);
#define SAKI_SCORE_ST(RK, ST)                                                                 \
  launch_score<RK, ST>(ix, B, H_q, H_kv, index_heads, N_cap, N_valid, q, q_pos, Q, B_q, mu, k, \
                       top_idx, top_score, w, p, s)
#define SAKI_SCORE(RK)                          \
  do {                                          \
    if (sketch_dtype == SAKI_FP8)               \
      SAKI_SCORE_ST(RK, kStFp8);                \
    else if (sketch_dtype == SAKI_BF16)         \
      SAKI_SCORE_ST(RK, kStBf16);               \
    else                                        \
      SAKI_SCORE_ST(RK, kStF32);                \
  } while (0)
  switch (r) {
    case 16: SAKI_SCORE(16); break;
    case 32: SAKI_SCORE(32); break;
    case 64: SAKI_SCORE(64); break;
    default: SAKI_SCORE(128); break;
  }
#undef SAKI_SCORE
#undef SAKI_SCORE_ST
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

}  // namespace

// ---------------------------------------------------------------- C ABI

extern "C" {

int saki_build_index(const void* keys, int key_dtype, int B, int H_q, int H_kv,
                     int N_cap, int d, int r, const float* B_k, const float* mu,
                     int sketch_dtype, void* index, size_t index_bytes, int n_begin,
                     int n_count, void* stream) {
  int st = check_common(B, H_q, H_kv, N_cap, 0, d);
  if (st != SAKI_OK) return st;
  if (!keys || !B_k || !mu || !index) return SAKI_ERR_ARG;
  if (!dtype_ok(key_dtype) || !sketch_ok(sketch_dtype) || !saki::rank_supported(r))
    return SAKI_ERR_UNSUPPORTED;
  if (n_begin < 0 || n_count < 0 || (long long)n_begin + n_count > N_cap) return SAKI_ERR_ARG;
  if (index_bytes < saki::index_bytes(B, H_q, N_cap, r, sketch_dtype)) return SAKI_ERR_WORKSPACE;
  if (n_count == 0) return SAKI_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* ix = reinterpret_cast<uint8_t*>(index);
  const int n_end = n_begin + n_count;
#define SAKI_BUILD_ST(RK, KB)                                                                \
  do {                                                                                       \
    if (sketch_dtype == SAKI_FP8)                                                            \
      launch_build<RK, KB, kStFp8>(keys, B_k, mu, B, H_q, H_kv, N_cap, ix, n_begin, n_end, s);  \
    else if (sketch_dtype == SAKI_BF16)                                                      \
      launch_build<RK, KB, kStBf16>(keys, B_k, mu, B, H_q, H_kv, N_cap, ix, n_begin, n_end, s); \
    else                                                                                     \
      launch_build<RK, KB, kStF32>(keys, B_k, mu, B, H_q, H_kv, N_cap, ix, n_begin, n_end, s);  \
  } while (0)
#define SAKI_BUILD(RK)                         \
  do {                                         \
    if (key_dtype == SAKI_BF16)                \
      SAKI_BUILD_ST(RK, true);                 \
    else                                       \
      SAKI_BUILD_ST(RK, false);                \
  } while (0)
  switch (r) {
    case 16: SAKI_BUILD(16); break;
    case 32: SAKI_BUILD(32); break;
    case 64: SAKI_BUILD(64); break;
    default: SAKI_BUILD(128); break;
  }
#undef SAKI_BUILD
#undef SAKI_BUILD_ST
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

int saki_index_export(const void* index, int sketch_dtype, int B, int H_q, int N_cap, int r,
                      float* out, void* stream) {
  if (!index || !out || B <= 0 || H_q <= 0 || N_cap < 0) return SAKI_ERR_ARG;
  if ((long long)B * H_q > 65535) return SAKI_ERR_UNSUPPORTED;
  if (!sketch_ok(sketch_dtype) || !saki::rank_supported(r)) return SAKI_ERR_UNSUPPORTED;
  if (N_cap == 0) return SAKI_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  dim3 grid((unsigned)saki::n_tiles(N_cap), B * H_q);
  const uint8_t* ix = reinterpret_cast<const uint8_t*>(index);
  const int nt = (int)saki::n_tiles(N_cap);
#define SAKI_EXPORT(RK)                                                                          \
  do {                                                                                           \
    if (sketch_dtype == SAKI_FP8)                                                                \
      hipLaunchKernelGGL((export_kernel<RK, kStFp8>), grid, dim3(64), 0, s, ix, nt, N_cap, out);   \
    else if (sketch_dtype == SAKI_BF16)                                                          \
      hipLaunchKernelGGL((export_kernel<RK, kStBf16>), grid, dim3(64), 0, s, ix, nt, N_cap, out);  \
    else                                                                                         \
      hipLaunchKernelGGL((export_kernel<RK, kStF32>), grid, dim3(64), 0, s, ix, nt, N_cap, out);   \
  } while (0)
  switch (r) {
    case 16: SAKI_EXPORT(16); break;
    case 32: SAKI_EXPORT(32); break;
    case 64: SAKI_EXPORT(64); break;
    default: SAKI_EXPORT(128); break;
  }
#undef SAKI_EXPORT
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

int saki_score_topk(const void* index, int sketch_dtype, int B, int H_q, int H_kv,
                    int index_heads, int N_cap, int N_valid, int d, int r, const float* q,
                    const int* q_pos, int Q, const float* B_q, const float* mu, int k,
                    int* top_idx, float* top_score, void* ws, size_t ws_bytes, void* stream) {
  if (!ws) return SAKI_ERR_ARG;
  return score_topk_impl(index, sketch_dtype, B, H_q, H_kv, index_heads, N_cap, N_valid, d, r,
                         q, q_pos, Q, B_q, mu, k, top_idx, top_score, ws, ws_bytes, stream);
}

int saki_score_topk_noalloc(const void* index, int sketch_dtype, int B, int H_q, int H_kv,
                            int index_heads, int N_cap, int N_valid, int d, int r,
                            const float* q, const int* q_pos, int Q, const float* B_q,
                            const float* mu, int k, int* top_idx, float* top_score,
                            void* stream) {
  return score_topk_impl(index, sketch_dtype, B, H_q, H_kv, index_heads, N_cap, N_valid, d, r,
                         q, q_pos, Q, B_q, mu, k, top_idx, top_score, nullptr, kScratchBytes,
                         stream);
}

size_t saki_noalloc_scratch_bytes(void) { return kScratchBytes; }

int saki_calibration_moments(const float* q_cal, const float* k_cal, int H_q, int H_kv,
                             int T, int d, double* Sigma_q, double* Sigma_k,
                             double* key_mean, void* stream) {
  if (!q_cal || !k_cal || !Sigma_q || !Sigma_k || !key_mean) return SAKI_ERR_ARG;
  if (H_q <= 0 || H_kv <= 0 || T <= 0 || d <= 0 || d > 4096) return SAKI_ERR_ARG;
  if ((long long)H_q + H_kv > 65535) return SAKI_ERR_UNSUPPORTED;
  const long long nb = (d + kMomBlk - 1) / kMomBlk;
  hipLaunchKernelGGL(moments_kernel, dim3((unsigned)((H_q + H_kv) * (nb * (nb + 1) / 2))), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(stream), q_cal, k_cal, H_q, T, d, Sigma_q,
                     Sigma_k, key_mean);
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

int saki_recall(const void* keys, int key_dtype, const float* q, const int* q_pos, int B,
                int H_q, int H_kv, int N_cap, int N_valid, int Q, int d, int k,
                const int* approx_idx, int* hits, int* exact_idx, void* ws, size_t ws_bytes,
                void* stream) {
  int st = check_common(B, H_q, H_kv, N_cap, N_valid, d);
  if (st != SAKI_OK) return st;
  if (Q < 0) return SAKI_ERR_ARG;
  if (!dtype_ok(key_dtype) || k < 1 || k > kMaxK) return SAKI_ERR_UNSUPPORTED;
  if (Q == 0) return SAKI_OK;
  if (!keys || !q || !approx_idx || !hits) return SAKI_ERR_ARG;
  const saki::Plan p = saki::recall_plan(B, H_q, H_kv, Q, N_valid);
  if (ws_bytes < p.ws_bytes) return SAKI_ERR_WORKSPACE;
  if (p.ws_bytes > 0 && !ws) return SAKI_ERR_ARG;
  if ((size_t)p.row_blocks * p.n_chunks > 0x7fffffffu) return SAKI_ERR_UNSUPPORTED;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  uint8_t* w = reinterpret_cast<uint8_t*>(ws);
  if (key_dtype == SAKI_BF16)
    launch_recall<true>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx_idx, hits,
                        exact_idx, w, ws_bytes, p, s);
  else
    launch_recall<false>(keys, q, q_pos, B, H_q, H_kv, N_cap, N_valid, Q, k, approx_idx, hits,
                         exact_idx, w, ws_bytes, p, s);
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

int saki_attend(const void* keys, int key_dtype, const float* values, const void* index,
                int sketch_dtype, int key_source, int B, int H_q, int H_kv, int index_heads,
                int N_cap, int N_valid, int d, int r, const float* q, const int* q_pos, int Q,
                const float* B_q, const float* mu, const int* top_idx, int k,
                float rope_theta, float* out, void* stream) {
  int st = check_common(B, H_q, H_kv, N_cap, N_valid, d);
  if (st != SAKI_OK) return st;
  if (Q < 0 || k < 1 || !(rope_theta > 0.f) || !std::isfinite(rope_theta)) return SAKI_ERR_ARG;
  if (k > kMaxK) return SAKI_ERR_UNSUPPORTED;
  const bool recon = key_source == SAKI_KEYS_RECONSTRUCTED;
  if (key_source != SAKI_KEYS_EXACT && !recon) return SAKI_ERR_ARG;
  if (Q == 0) return SAKI_OK;
  if (N_valid < 1 || !values || !q || !top_idx || !out) return SAKI_ERR_ARG;
  if (recon) {
    if (!index || !B_q || !mu) return SAKI_ERR_ARG;
    if (index_heads <= 0 || H_q % index_heads != 0 || index_heads % H_kv != 0) return SAKI_ERR_ARG;
    if (!sketch_ok(sketch_dtype) || !saki::rank_supported(r)) return SAKI_ERR_UNSUPPORTED;
  } else {
    if (!keys) return SAKI_ERR_ARG;
    if (!dtype_ok(key_dtype)) return SAKI_ERR_UNSUPPORTED;
  }
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const uint8_t* ix = reinterpret_cast<const uint8_t*>(index);
#define SAKI_ATTEND(RK, KB, ST, RC)                                                              \
  launch_attend<RK, KB, ST, RC>(keys, values, ix, B, H_q, H_kv, index_heads, N_cap, N_valid, q, \
                                q_pos, Q, B_q, mu, top_idx, k, rope_theta, out, s)
#define SAKI_ATTEND_R(RK)                              \
  do {                                                 \
    if (sketch_dtype == SAKI_FP8)                      \
      SAKI_ATTEND(RK, false, kStFp8, true);            \
    else if (sketch_dtype == SAKI_BF16)                \
      SAKI_ATTEND(RK, false, kStBf16, true);           \
    else                                               \
      SAKI_ATTEND(RK, false, kStF32, true);            \
  } while (0)
  if (!recon) {
    if (key_dtype == SAKI_BF16)
      SAKI_ATTEND(32, true, kStF32, false);
    else
      SAKI_ATTEND(32, false, kStF32, false);
  } else {
    switch (r) {
      case 16: SAKI_ATTEND_R(16); break;
      case 32: SAKI_ATTEND_R(32); break;
      case 64: SAKI_ATTEND_R(64); break;
      default: SAKI_ATTEND_R(128); break;
    }
  }
#undef SAKI_ATTEND_R
#undef SAKI_ATTEND
  return launch_ok() ? SAKI_OK : SAKI_ERR_HIP;
}

}  // extern "C"
