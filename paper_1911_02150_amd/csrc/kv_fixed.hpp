// Correctly rounded K / V rows from integer products: what project_kv.hip and project_kv_rows.hip share (the numbers are
// explained in project_kv.hip).
#pragma once
#include "common.hpp"

namespace mqa {
namespace kv_fixed {

typedef __attribute__((ext_vector_type(4))) int int4v;
typedef __attribute__((ext_vector_type(16))) int int16v;

// Open elements of a tile (of 16384) from which its waves sum all of it in float64 instead.  A wave spends some 8 us on one
// element where the weights are a cache line each (project_kv.hip), the whole tile takes 270 us: us for 32768 rows, d = 1024,
// with one channel of the rows 2^6 times the others and its weights as much smaller (210 open elements a tile) one by one
// 439, all 485; 2^8 times (650) 978 and 481; 2^10 times 2419 and 478; the float64 kernel takes 410, normal deviates 213.
constexpr int kMostOpen = 256;
constexpr int kMaxC = 16384;                   // four products of 2^14 per index in an int32

// what the float64 kernel stores
__device__ __forceinline__ uint32_t to_bf16(double s) { return float_to_bf16_rne((float)s); }

// The scale (a power of two) that takes the largest magnitude `bits` to [2^29, 2^31 - 2^24]: the top digit stays
// an int8 with what the lower ones carry into it.
__device__ __forceinline__ int fixed_exponent(uint32_t bits) {           // x . 2^exponent
  const int e = (int)(bits >> 23);
  if (e == 0) return 127;                                               // (a subnormal, or zero; 30 .. 254 at most below)
  int up = 30 + 127 - e;
  if ((bits & 0x7fffffu) > 0x7d0000u) --up;                             // (2 - 2^-6) 2^30 = 2^31 - 2^24
  return up > 127 ? 127 : up;
}

// Four scaled values -> the words of their four digits, lowest digit first.
struct Digits4 { int word[4]; };
__device__ __forceinline__ Digits4 digits_of(float a, float b, float c, float d) {
  const uint32_t y[4] = {(uint32_t)(int)a + 0x00808080u, (uint32_t)(int)b + 0x00808080u, (uint32_t)(int)c + 0x00808080u, (uint32_t)(int)d + 0x00808080u};
  const uint32_t t0 = __builtin_amdgcn_perm(y[1], y[0], 0x05010400u);           // bytes 0, 0', 1, 1'
  const uint32_t t1 = __builtin_amdgcn_perm(y[1], y[0], 0x07030602u);           // bytes 2, 2', 3, 3'
  const uint32_t t2 = __builtin_amdgcn_perm(y[3], y[2], 0x05010400u);
  const uint32_t t3 = __builtin_amdgcn_perm(y[3], y[2], 0x07030602u);
  Digits4 t;
  t.word[0] = (int)(__builtin_amdgcn_perm(t2, t0, 0x05040100u) ^ 0x80808080u);
  t.word[1] = (int)(__builtin_amdgcn_perm(t2, t0, 0x07060302u) ^ 0x80808080u);
  t.word[2] = (int)(__builtin_amdgcn_perm(t3, t1, 0x05040100u) ^ 0x80808080u);
  t.word[3] = (int)__builtin_amdgcn_perm(t3, t1, 0x07060302u);
  return t;
}

// What a line (row or column) adds to the bounds of its elements, in units of 2^24 of the digit sums (rounded up: 0.2 %
// covers the roundings here and in rounded_sum), and to their exponents.  An element's bound is row.w + col.w + row.r col.r:
//   w: sqrt(C) |d3| + C, for the truncation of the other line's values (|X| <= 2^24 (|d3| + 1)), and half of 0.52 C + 2;
//   r: |(d0, d1, d2)| 2^-4: the dropped products are below 2^-8 (|d2||e0| + |d1||e1| + |d0||e2|) <= 2^-8 |d||e|.
// A line of zeros has w = -inf (its elements are 0 and no bound is needed), one with an infinity w = +inf, one with a NaN a NaN.
struct Line { float w, r; int exponent; };     // exponent: of 2, that an element's sum is multiplied by
__device__ __forceinline__ Line line_of(const int* squares, uint32_t most, int C) {
  Line l;
  l.w = (sqrtf((float)C) * sqrtf((float)squares[3]) + 1.26f * (float)C + 1.f) * 1.002f;
  l.r = sqrtf((float)squares[0] + (float)squares[1] + (float)squares[2]) * (0.0625f * 1.002f);
  l.exponent = 12 - fixed_exponent(most);
  if (most >= 0x7f800000u) l.w = __uint_as_float(most);
  if (most == 0) l.w = -INFINITY;
  return l;
}

// An element's sum from its digit sums (t0: i + j = 3 ... t3: i + j = 6), in units of 2^24 (exact in 64 bits), as the float
// it is rounded to first.
__device__ __forceinline__ float digit_sum(int t0, int t1, int t2, int t3) {
  return (float)fma((double)t3, 0x1p24, fma((double)t2, 0x1p16, fma((double)t1, 0x1p8, (double)t0)));
}

// The element's bf16 from that sum, and whether the bound leaves it open: if a tie (the middle of the low 16 bits) is no
// further off than the bound and the rounding to float (one unit of the last place); just above a power of two the tie below
// is in the next binade: half the spacing, 0x4000 below the power itself.  A sum that leaves the normal floats is open as
// well, and so is 0 (nothing is left of the sum) unless a line is all zeros.
__device__ __forceinline__ uint32_t rounded_sum(float mid, Line row, Line col, bool* is_open) {
  const float bound = fmaf(row.r, col.r, row.w + col.w);
  const int scale = row.exponent + col.exponent;
  const uint32_t bits = __float_as_uint(mid);
  int off = abs((int)(bits & 0xffffu) - 0x8000);
  if ((bits & 0x7f0000u) == 0) off = min(off, (int)(bits & 0xffffu) + 0x3fff);
  const float unit = __uint_as_float((bits & 0x7f800000u) - (23u << 23));      // of the last place (a whole number: 2^0 at least, or 0)
  const int e_out = (int)(bits << 1 >> 24) + scale;
  const bool apart = bound < (float)(off - 1) * unit && e_out >= 2 && e_out <= 253;
  const uint32_t out = bits + ((uint32_t)scale << 23);
  *is_open = mid == 0.f ? !(bound < 0.f) : !apart;
  return mid == 0.f ? 0 : (out + 0x7fffu + (out >> 16 & 1u)) >> 16;
}

// Of an open element: is it NaN (a NaN in a line, or an infinity against a line of zeros)?  It needs no summing then: one row of NaN in
// every 64 of a memory of 64 x 512, d = 1024: 405 -> 123 us with a workspace, 465 -> 174 without.
constexpr uint32_t kNan = 0x7fc0u;
__device__ __forceinline__ bool is_nan(Line row, Line col) {
  const float w = row.w + col.w;
  return w != w;
}

// 32 rows x 64 columns by one wave, in float64 from global memory: register e of lane (i, kk) of a 16 x 16 block is row
// 4 e + kk, column i; step s contracts the indices 4 kk + s of sixteen.  row_at(r), column_at(c): their first elements
// (a column's are `stride` apart); store(r, c, bf16).
template <typename Row, typename Column, typename Store>
__device__ __forceinline__ void float64_tile(int lane, int C, Row&& row_at, Column&& column_at, int stride, Store&& store) {
  typedef __attribute__((ext_vector_type(4))) double double4v;
  const int i = lane & 15, kk = lane >> 4;
  const float* xr[2];
  const float* w[4];
#pragma unroll
  for (int r = 0; r < 2; ++r) xr[r] = row_at(16 * r + i);
#pragma unroll
  for (int j = 0; j < 4; ++j) w[j] = column_at(16 * j + i);
  double4v acc[2][4];
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[r][j] = double4v{0., 0., 0., 0.};
  for (int c0 = 0; c0 < C; c0 += 16) {
    const int c = min(c0 + 4 * kk, C - 4);
    const bool in = c0 + 4 * kk < C;           // (C is a multiple of 8)
    float a[2][4], b[4][4];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const float4 v = *reinterpret_cast<const float4*>(xr[r] + c);
      a[r][0] = in ? v.x : 0.f; a[r][1] = in ? v.y : 0.f; a[r][2] = in ? v.z : 0.f; a[r][3] = in ? v.w : 0.f;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float v = w[j][(size_t)(c + s) * stride];
        b[j][s] = in ? v : 0.f;
      }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[r][j] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)a[r][s], (double)b[j][s], acc[r][j], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 2; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) store(16 * r + 4 * e + kk, 16 * j + i, to_bf16(acc[r][j][e]));
}

}  // namespace kv_fixed
}  // namespace mqa
