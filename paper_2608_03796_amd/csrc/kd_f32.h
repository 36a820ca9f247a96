// The 128x128 tile of fp32 contractions (gfx950): every fp32 operand element
// is split exactly into three bf16 terms and the product is formed from the
// six bf16 MFMAs that matter.
//
// x = hi + mid + lo with hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid:
// both subtractions are exact and 24 bits of mantissa fit in 3 x 8, so the
// three terms are x (mid at most 2^-8 and lo 2^-17 of it). Of the nine
// products the six largest are accumulated in fp32; the three left out (mid
// lo, lo mid, lo lo) are at most 2^-24 of the product together (x = 1.0038986
// squared), as much as the rounding of one fp32 accumulation. Why: the bf16 MFMA does 16 times the
// multiply-adds per cycle of the fp32 one (about 2.5 PFLOP/s against 157
// TFLOP/s dense), so six of them take 3/8 of its time. The relative error of
// the gradients against 64 bits is below the fp32 MFMA's (256 x 256 x 4096:
// 2.2e-7 against 3.3e-7; 1000 x 768 x 30011: 6.3e-7 against 8.1e-7; 2048 x
// 1024 x 32000: 1.0e-6 against 1.1e-6), fewer roundings being made per sum.
// A term cannot be smaller than bf16's smallest step (2^-133), so operands
// below about 1e-33 in magnitude keep fewer than 24 bits.
//
// Non-finite operands give a NaN remainder (inf - inf), hence non-finite
// sums: a tile whose accumulators are not all finite is computed again with
// the fp32 MFMA straight from memory (gemm_f32_plain), which also covers
// magnitudes whose bf16 rounding overflows.
#pragma once

#include "kd_device.h"

namespace kd {

// LDS of one K step (32 elements): per operand three planes of 128 rows x 32
// bf16 (64 bytes a row, four 16-byte slots)
constexpr int kF32Plane = 128 * 64;
constexpr int kF32Op = 3 * kF32Plane;
constexpr int kLdsF32 = 2 * kF32Op;  // 48 KiB

// Slot swizzle: with slot XOR (row / 2) % 4 the fragment reads (16 rows of one
// slot per lane group) and the writes touch each bank equally often.
__device__ __forceinline__ int f32_slot(int row, int oct) {
  return row * 64 + ((oct ^ ((row >> 1) & 3)) << 4);
}

__device__ __forceinline__ float f32_lo16(uint32_t x) { return __builtin_bit_cast(float, x << 16); }
__device__ __forceinline__ float f32_hi16(uint32_t x) {
  return __builtin_bit_cast(float, x & 0xffff0000u);
}

// eight floats -> their hi, mid and lo bf16 terms
__device__ __forceinline__ void split8(const float (&x)[8], u32x4_t& hi, u32x4_t& mid,
                                       u32x4_t& lo) {
  uint32_t h[4], m[4], l[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float x0 = x[2 * p], x1 = x[2 * p + 1];
    h[p] = pack_bf16x2(x0, x1);
    const float r0 = x0 - f32_lo16(h[p]), r1 = x1 - f32_hi16(h[p]);
    m[p] = pack_bf16x2(r0, r1);
    l[p] = pack_bf16x2(r0 - f32_lo16(m[p]), r1 - f32_hi16(m[p]));
  }
  hi = u32x4_t{h[0], h[1], h[2], h[3]};
  mid = u32x4_t{m[0], m[1], m[2], m[3]};
  lo = u32x4_t{l[0], l[1], l[2], l[3]};
}

// Register staging of one operand's K step: 512 pieces of 8 K elements of one
// row (row, octet), two per thread.
//  * K-contiguous: piece u of thread t is row t/4 + 64 u, octet t%4 (two
//    16-byte loads; four lanes read a row's 128 bytes).
//  * K-major: piece u of thread t is column t%128, octet t/128 + 2 u (eight
//    4-byte loads, a wave reading 256 contiguous bytes of a K row each).
template <typename Op>
struct F32Stage;

template <>
struct F32Stage<KcOp> {
  float x[2][8];
  __amdgpu_buffer_rsrc_t r;
  uint32_t off[2];
  __device__ __forceinline__ static int row(int tid, int u) { return (tid >> 2) + 64 * u; }
  __device__ __forceinline__ static int oct(int tid, int) { return tid & 3; }
  __device__ __forceinline__ void init(const KcOp& op, int tid) {
    r = make_rsrc(op.base, op.bytes);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      off[u] = (uint32_t)row(tid, u) * (uint32_t)op.ld + (uint32_t)oct(tid, u) * 32u;
  }
  __device__ __forceinline__ void load(const KcOp&, int ks) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x4_t v = __builtin_bit_cast(
            f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, off[u] + 16u * q, ks * kRowB, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) x[u][4 * q + e] = v[e];
      }
    }
  }
};

template <>
struct F32Stage<KmOp> {
  float x[2][8];
  uint32_t off[2];
  __device__ __forceinline__ static int row(int tid, int) { return tid & 127; }
  __device__ __forceinline__ static int oct(int tid, int u) { return (tid >> 7) + 2 * u; }
  __device__ __forceinline__ void init(const KmOp& op, int tid) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
      off[u] = (uint32_t)(8 * oct(tid, u)) * (uint32_t)op.ld + (uint32_t)row(tid, u) * 4u;
  }
  __device__ __forceinline__ void load(const KmOp& op, int ks) {
    const int64_t step0 = (int64_t)ks * 32 * op.ld;
    int64_t left = op.bytes - step0;
    left = left < 0 ? 0 : (left > 0x7fffffff ? 0x7fffffff : left);
    const __amdgpu_buffer_rsrc_t r = make_rsrc(op.base + step0, (uint32_t)left);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        x[u][e] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(r, off[u] + (uint32_t)(e * op.ld), 0, 0));
  }
};

template <typename Op>
__device__ __forceinline__ void f32_write(const F32Stage<Op>& s, char* lds, int tid) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    u32x4_t hi, mid, lo;
    split8(s.x[u], hi, mid, lo);
    char* d = lds + f32_slot(F32Stage<Op>::row(tid, u), F32Stage<Op>::oct(tid, u));
    *reinterpret_cast<u32x4_t*>(d) = hi;
    *reinterpret_cast<u32x4_t*>(d + kF32Plane) = mid;
    *reinterpret_cast<u32x4_t*>(d + 2 * kF32Plane) = lo;
  }
}

// Four K elements k..k+3 of one row, for the fp32 MFMA
__device__ __forceinline__ u32x4_t f32_frag(const KcOp& op, int row, int k) {
  const __amdgpu_buffer_rsrc_t r = make_rsrc(op.base, op.bytes);
  return __builtin_amdgcn_raw_buffer_load_b128(r, row * op.ld + 4 * k, 0, 0);
}
__device__ __forceinline__ u32x4_t f32_frag(const KmOp& op, int row, int k) {
  u32x4_t v = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t o = (int64_t)(k + e) * op.ld + 4 * row;
    if (o < op.bytes) v[e] = *reinterpret_cast<const uint32_t*>(op.base + o);
  }
  return v;
}

// The tile by fp32 MFMAs with operands read straight from memory: only for
// tiles whose split sums are not all finite (non-finite or huge operands).
template <typename OA, typename OB>
__device__ void gemm_f32_plain(const OA& opa, const OB& opb, int ks_begin, int ks_end,
                               AccTile<128>& acc) {
  typedef Geo<128> G;
  const int lane = threadIdx.x & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc.v[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int k0 = 32 * ks_begin; k0 < 32 * ks_end; k0 += 16) {
    const int k = k0 + 4 * (lane >> 4);
    u32x4_t b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = f32_frag(opb, G::acc_n(wn, j, lane), k);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const u32x4_t a = f32_frag(opa, wm * 64 + 16 * i + (lane & 15), k);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc.v[i][j] = mfma_slot(a, b[j], acc.v[i][j], (float*)nullptr);
    }
  }
}

// acc = A[0:128, k-range] * B[0:128, k-range]^T for fp32 operands (KcOp or
// KmOp as for gemm_tile; 32 K elements per step), 4 waves of 64x64.
//
// The split is done once per workgroup on the way to LDS (176 VALU
// instructions per thread and step against 96 MFMAs per wave; splitting the
// fragments after the LDS reads would do it twice as often), so the operands
// pass through registers: the next step's loads are in flight during the
// current step's MFMAs. One LDS stage of 48 KiB per workgroup: what hides a
// workgroup's split, writes and barriers is the second workgroup on the
// compute unit (three do not fit the registers without spills: 40% slower).
// LDS traffic per step and pair of workgroups is 288 KiB (2304 clocks at 128
// B) against 3072 clocks of MFMA. Measured at 2048 x 1024 x 32000 (dH): 631 us,
// 213 TFLOP/s, against 918 us with fp32 MFMAs in 256x256 tiles; counters: MFMA
// pipes 63% busy at 1.89 GHz, no bank conflicts. Splitting the next step's
// values between the current step's MFMAs was 3% slower; the wave priority
// during the MFMAs gives 1-2%. Ends with a barrier.
template <typename OA, typename OB>
__device__ __forceinline__ void gemm_f32(const OA& opa, const OB& opb, int ks_begin, int ks_end,
                                         char* lds, AccTile<128>& acc) {
  typedef Geo<128> G;
  const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
  const int wm = G::wm(wave), wn = G::wn(wave);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc.v[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  F32Stage<OA> sa;
  F32Stage<OB> sb;
  sa.init(opa, tid);
  sb.init(opb, tid);
  char* const lb = lds + kF32Op;
  int ra[4], rb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    ra[i] = f32_slot(wm * 64 + 16 * i + (lane & 15), lane >> 4);
    rb[i] = f32_slot(wn * 64 + 16 * i + (lane & 15), lane >> 4);
  }
  if (ks_begin < ks_end) {
    sa.load(opa, ks_begin);
    sb.load(opb, ks_begin);
  }
  // products of the terms (0 hi, 1 mid, 2 lo), small ones first
  constexpr int pa[6] = {0, 2, 1, 0, 1, 0}, pb[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll 1
  for (int ks = ks_begin; ks < ks_end; ++ks) {
    f32_write(sa, lds, tid);
    f32_write(sb, lb, tid);
    if (ks + 1 < ks_end) {
      sa.load(opa, ks + 1);
      sb.load(opb, ks + 1);
    }
    __syncthreads();
    __builtin_amdgcn_s_setprio(1);
    u32x4_t b[4][3], a[2][3];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        b[j][p] = *reinterpret_cast<const u32x4_t*>(lb + rb[j] + p * kF32Plane);
#pragma unroll
    for (int p = 0; p < 3; ++p)
      a[0][p] = *reinterpret_cast<const u32x4_t*>(lds + ra[0] + p * kF32Plane);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (i < 3) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
          a[(i + 1) & 1][p] = *reinterpret_cast<const u32x4_t*>(lds + ra[i + 1] + p * kF32Plane);
      }
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          // four independent accumulators in a row, in a snake over the
          // products (fewer operand changes: 1.4% faster)
          const int j = (q & 1) ? 3 - jj : jj;
          acc.v[i][j] = mfma_slot(a[i & 1][pa[q]], b[j][pb[q]], acc.v[i][j], (__bf16*)nullptr);
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();  // every wave has read this step's fragments
  }
  // any sum not finite in the workgroup: all of the tile again in fp32
  float bad = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) bad = __builtin_fmaf(acc.v[i][j][r], 0.f, bad);
  const bool any = __builtin_amdgcn_ballot_w64(!(bad == 0.f)) != 0ull;
  int* flag = reinterpret_cast<int*>(lds);
  if (lane == 0) flag[wave] = any ? 1 : 0;
  __syncthreads();
  const int redo = __builtin_amdgcn_readfirstlane(flag[0] | flag[1] | flag[2] | flag[3]);
  if (redo != 0) gemm_f32_plain(opa, opb, ks_begin, ks_end, acc);
  __syncthreads();
}

}  // namespace kd
