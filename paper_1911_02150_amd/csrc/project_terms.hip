// Projections of a decode step's rows: out[rows, N] = in[rows, C] . B[C, N], B addressed inside the projection tensor
// P [h, d, kv] as in project.hip, from three bfloat16 terms per float32 operand.
//
// x = a1 + a2 + a3, each the nearest bfloat16 of what the ones before it leave: exact (8 + 8 + 8 significant bits) for
// 2^-110 <= |x| < 2^127 and 0 (below, the last bits of the third term are past bfloat16's smallest).  Of the nine products of terms the six largest are added,
//   a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1)          (the rest is below 2^-24 |a||b|, 2^-27 typically)
// on v_mfma_f32_16x16x32_bf16: 6 / 16 of the time of the float32 instructions (terms of bfloat16 and which of their products
// count: Henry, Tang and Heinecke 2019).  a1 b1 and the five small ones have a running sum each, added at the end: the small ones' is
// some 2^-8 of the other, so what is left is one rounding of the sum for every 32 indices where the float32 instructions
// round for every four.  No scales are needed (bfloat16 has float32's exponents), so nothing has to be known of a row or column
// before it is multiplied.  A product of terms can overflow where the product of the operands does not, or leave an infinity of the
// other sign or a NaN where that is one infinity: a wave whose sums are not finite at the end, or that met an operand below
// 2^-110 other than 0, multiplies its part again on v_mfma_f32_16x16x4_f32 (as it does where an operand was an infinity or a
// weight NaN).  Relative error of a 1024-term sum of normal deviates 8.1e-8 (all six products in one running sum 1.6e-7, project.hip
// 2.1e-7, gemm.hip 1.6e-7), of a 4096-term one 1.4e-7 (3.5e-7, 4.1e-7), in eight parts 9.1e-8; with every other x a zero, as behind
// a relu, 7.1e-8 (1.6e-7, 1.5e-7), 1.1e-7 (3.3e-7, 2.9e-7) and 8.2e-8.
//
// As in project.hip the waves of a workgroup cut the contraction among them and are summed through LDS; operands come
// from L2 straight into their registers, two steps in flight.  S > 1: the contraction is cut among S workgroups as well, and their
// partial tiles (in the workspace) are summed by finish_kernel, together with what follows the product: the residual and
// the next layernorm.
// Measured (128 rows, 4096 x 1024, weights from HBM): 14.5 us + 3.5 of finish_kernel (project.hip 25 and a layernorm of 3); 64 rows: 13.5
// with both (22).  Of the 14.5: vector instructions 7 (splitting: 11 for two values), matrix cores 3, the first operands 3; on
// the float32 instructions alone it takes the same time (they need no splitting, and 8 us).  Tiles of 64 x 64: 29 (spills), of
// 64 x 32: 19.5.
#include "common.hpp"

#include <math.h>

namespace mqa {
namespace {

typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kWaves = 8, kStep = 32;          // (a step: the indices of one instruction)
constexpr int kWideStage = 32;                 // indices of a stage of gemm.hip's 128 x 128 tiles: parts are whole stages

constexpr uint32_t kLeast = (0x08800000u << 1) - 1;          // 2^-110, in the order of the kernel's `least`

struct Terms { u32x4 t[3]; };                  // eight values

__device__ __forceinline__ void split3(float a, float b, Terms& x, int at) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    uint32_t u = pack_bf16_pair(a, b);
    asm("" : "+v"(u));                         // (the halves are read from the packed register, not rounded once more each)
    x.t[p][at] = u;
    a -= __uint_as_float(u << 16);
    b -= __uint_as_float(u & 0xffff0000u);
  }
}

template <bool KC, int RB, int CB>
__global__ __launch_bounds__(kWaves * 64, 2)
void project_terms_kernel(const float* __restrict__ in, const float* __restrict__ P, float* out, float* part,
                          int rows, int d, int h, int kv, int epilogue) {
  constexpr int TM = RB * 16, TN = CB * 16;
  extern __shared__ __align__(16) float red_raw[];
  float (*red)[TM * TN] = reinterpret_cast<float (*)[TM * TN]>(red_raw);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i = lane & 15, kk = lane >> 4;
  const int C = KC ? h * kv : d, N = KC ? d : h * kv;
  const int n0 = blockIdx.x * TN, row0 = blockIdx.y * TM;
  const int steps = (C + kStep - 1) / kStep, per = (steps + gridDim.z - 1) / gridDim.z;
  const int first = blockIdx.z * per, end = min(first + per, steps);

  const float* arow[RB];
#pragma unroll
  for (int r = 0; r < RB; ++r) arow[r] = in + (size_t)min(row0 + 16 * r + i, rows - 1) * C;
  int ncol[CB];                                // c contiguous: column n0 + 16 j + i of block j; else the lane's CB adjacent columns
#pragma unroll
  for (int j = 0; j < CB; ++j) ncol[j] = min(n0 + 16 * j + i, N - 1);
  const int nb = min(n0 + CB * i, N - CB);
  const float* bcol = P + (size_t)(nb / kv) * d * kv + nb % kv;

  typedef __attribute__((ext_vector_type(CB))) float vec;
  struct Raw { float a[RB][8]; float b[CB][8]; };
  auto load = [&](int step, Raw& x) {
    const int c = min(kStep * step + 8 * kk, C - 8);
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(arow[r] + c + 4 * q);
#pragma unroll
        for (int e = 0; e < 4; ++e) x.a[r][4 * q + e] = v[e];
      }
    if constexpr (KC) {                        // (eight indices stay inside one head: kv % 8 == 0)
      const float* bp = P + (size_t)(c / kv) * d * kv + c % kv;
#pragma unroll
      for (int j = 0; j < CB; ++j)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const floatx4 v = *reinterpret_cast<const floatx4*>(bp + (size_t)ncol[j] * kv + 4 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) x.b[j][4 * q + e] = v[e];
        }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const vec v = *reinterpret_cast<const vec*>(bcol + (size_t)(c + e) * kv);
#pragma unroll
        for (int j = 0; j < CB; ++j) x.b[j][e] = v[j];
      }
    }
  };
  floatx4 acc[RB][CB], low[RB][CB];
  auto drop_tail = [&](int step, Raw& x) {     // (C is a multiple of 8)
    if (kStep * (step + 1) > C && kStep * step + 8 * kk >= C) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int r = 0; r < RB; ++r) x.a[r][e] = 0.f;
#pragma unroll
        for (int j = 0; j < CB; ++j) x.b[j][e] = 0.f;
      }
    }
  };
  auto multiply_plain = [&](const Raw& x) {
#pragma unroll
    for (int e = 0; e < 8; ++e)                // slots 8 kk + e
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.a[r][e], x.b[j][e], acc[r][j], 0, 0, 0);
  };
  uint32_t least = ~0u;                        // of the operands' magnitudes in order, zero last
  auto look = [&](float v) { least = min(least, (__float_as_uint(v) << 1) - 1u); };
  auto multiply_terms = [&](const Raw& x) {
    float low_b = INFINITY;
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
#pragma unroll
      for (int r = 0; r < RB; ++r) look(x.a[r][e]), look(x.a[r][e + 1]);
#pragma unroll
      for (int j = 0; j < CB; ++j) asm("v_min3_f32 %0, %0, abs(%1), abs(%2)" : "+v"(low_b) : "v"(x.b[j][e]), "v"(x.b[j][e + 1]));
    }
    // (weights are seldom zeros: half an instruction for each instead of one and a half; stack step of 64 rows, three layers: 163.1 -> 161.5 us)
    if (__builtin_expect(__any(low_b < 0x1p-110f), 0)) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int j = 0; j < CB; ++j) look(x.b[j][e]);
    }
    Terms b[CB];
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) split3(x.b[j][2 * q], x.b[j][2 * q + 1], b[j], q);
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      Terms a;
#pragma unroll
      for (int q = 0; q < 4; ++q) split3(x.a[r][2 * q], x.a[r][2 * q + 1], a, q);
      auto product = [&](floatx4 (&to)[CB], int pa, int pb) {
#pragma unroll
        for (int j = 0; j < CB; ++j)
          to[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.t[pa]), __builtin_bit_cast(bf16x8, b[j].t[pb]), to[j], 0, 0, 0);
      };
      product(acc[r], 0, 0);
      product(low[r], 0, 1), product(low[r], 1, 0);
      product(low[r], 1, 1), product(low[r], 0, 2), product(low[r], 2, 0);
    }
  };
  auto sweep = [&](auto&& multiply) {          // this wave's steps, one in flight while the one before is multiplied
    Raw x0, x1;
    int step = first + wave;
    if (step < end) load(step, x0);
    while (step < end) {
      if (step + kWaves < end) load(step + kWaves, x1);
      drop_tail(step, x0), multiply(x0);
      step += kWaves;
      if (step >= end) break;
      if (step + kWaves < end) load(step + kWaves, x0);
      drop_tail(step, x1), multiply(x1);
      step += kWaves;
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[r][j] = low[r][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  sweep(multiply_terms);
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[r][j] += low[r][j];
  // An operand too small for its terms; and whatever overflowed on the way (an operand's first term, a product, a sum) has left an
  // infinity or a NaN behind.  So has a NaN in a row of the input, which leaves nothing to multiply again: such a row in every 32, us by looking
  // for it / without that (128 rows): 1024 x 4096 18.3 / 27.0, 4096 x 1024 with its layernorm 20.8 / 30.3 (project.hip 24.0, 28.4).
  float over = 0.f;
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int j = 0; j < CB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) over = fmaf(acc[r][j][e], 0.f, over);
  if (__builtin_expect(__any(!(over == 0.f) || least < kLeast), 0)) {
    bool again = least < kLeast;
    if (!__any(again)) {
      uint32_t nan = 0;                        // bit r: in row i of block r
      for (int step = first + wave; step < end; step += kWaves) {        // (indices past the end are of the same rows)
        const int c = min(kStep * step + 8 * kk, C - 8);
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const floatx4 v = *reinterpret_cast<const floatx4*>(arow[r] + c + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) nan |= v[e] != v[e] ? 1u << r : 0u;
          }
      }
#pragma unroll
      for (int o = 16; o < 64; o <<= 1) nan |= __shfl_xor(nan, o);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t nan_row = __shfl(nan, 4 * kk + e);
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
          for (int j = 0; j < CB; ++j) again |= !(acc[r][j][e] * 0.f == 0.f) && !(nan_row >> r & 1u);
      }
    }
    if (__any(again)) {
      clear();
      sweep(multiply_plain);
    }
  }
  // D layout: register e of lane (i, g) is row 4 g + e of the block, column i (KC) or the lane's CB adjacent ones
#pragma unroll
  for (int r = 0; r < RB; ++r)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float* at = red[wave] + (16 * r + 4 * kk + e) * TN;
      if constexpr (KC) {
#pragma unroll
        for (int j = 0; j < CB; ++j) at[16 * j + i] = acc[r][j][e];
      } else {
        vec v;
#pragma unroll
        for (int j = 0; j < CB; ++j) v[j] = acc[r][j][e];
        *reinterpret_cast<vec*>(at + CB * i) = v;
      }
    }
  __syncthreads();
  for (int q = tid; q < TM * TN / 4; q += kWaves * 64) {
    const int row = row0 + 4 * q / TN, n = n0 + 4 * q % TN;
    if (row >= rows || n >= N) continue;       // (N is a multiple of 8)
    floatx4 s[kWaves];
#pragma unroll
    for (int w = 0; w < kWaves; ++w) s[w] = *reinterpret_cast<const floatx4*>(red[w] + 4 * q);
    floatx4 y = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    if (gridDim.z > 1) {
      *reinterpret_cast<floatx4*>(part + ((size_t)blockIdx.z * rows + row) * N + n) = y;
    } else {
      float* dst = out + (size_t)row * N + n;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = apply_epilogue(y[e], dst + e, epilogue);
      *reinterpret_cast<floatx4*>(dst) = y;
    }
  }
}

__device__ __forceinline__ float block_sum(float x, float* red) {
  x = wave_sum(x);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = x;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// x[row] += the sum of the row's S partial products (in order: the same every time); y[row] = layernorm(x[row]) (gain 1, bias 0).  One workgroup per row of
// at most 1024 NV columns, all loads in flight together.
template <int NV>
__global__ __launch_bounds__(256)
void finish_kernel(const float* __restrict__ part, float* x, float* __restrict__ y, int rows, int N, int S, float eps) {
  __shared__ float red[4];
  const int n4 = N >> 2;
  floatx4* xr = reinterpret_cast<floatx4*>(x + (size_t)blockIdx.x * N);
  const floatx4* pr = reinterpret_cast<const floatx4*>(part + (size_t)blockIdx.x * N);
  const size_t stride = (size_t)rows * n4;
  floatx4 v[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int at = min((int)threadIdx.x + 256 * u, n4 - 1);
    const floatx4 was = xr[at];
    floatx4 s = pr[at];
    int p = 1;
    for (; p + 2 < S; p += 3) {
      const floatx4 a = pr[at + p * stride], b = pr[at + (p + 1) * stride], c = pr[at + (p + 2) * stride];
      s += a, s += b, s += c;
    }
    for (; p < S; ++p) s += pr[at + p * stride];
    v[u] = was + s;
  }
  float sum = 0.f;
#pragma unroll
  for (int u = 0; u < NV; ++u)
    if (threadIdx.x + 256 * u < n4) sum += (v[u][0] + v[u][1]) + (v[u][2] + v[u][3]);
  const float mean = block_sum(sum, red) / N;
  float q = 0.f;
#pragma unroll
  for (int u = 0; u < NV; ++u)
    if (threadIdx.x + 256 * u < n4) {
      const floatx4 c = v[u] - mean;
      q += (c[0] * c[0] + c[1] * c[1]) + (c[2] * c[2] + c[3] * c[3]);
    }
  const float rstd = 1.0f / sqrtf(block_sum(q, red) / N + eps);
  floatx4* yr = reinterpret_cast<floatx4*>(y + (size_t)blockIdx.x * N);
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int at = threadIdx.x + 256 * u;
    if (at < n4) {
      xr[at] = v[u];
      yr[at] = (v[u] - mean) * rstd;
    }
  }
}

template <bool KC, int RB, int CB>
hipError_t launch_tile(int S, const float* in, const float* P, float* out, float* part, int rows, int d, int h, int kv, int epilogue,
                       hipStream_t st) {
  const int N = KC ? d : h * kv;
  constexpr int lds = kWaves * RB * CB * 1024;             // 64 KiB at most
  const dim3 grid((N + 16 * CB - 1) / (16 * CB), (rows + 16 * RB - 1) / (16 * RB), S), block(kWaves * 64);
  hipLaunchKernelGGL((project_terms_kernel<KC, RB, CB>), grid, block, lds, st, in, P, out, part, rows, d, h, kv, epilogue);
  return hipGetLastError();
}

hipError_t launch_tiles(bool outp, TermsForm f, const float* in, const float* P, float* out, float* part, int rows, int d, int h, int kv,
                        int epilogue, hipStream_t st) {
#define MQA_TERMS(RB_, CB_)                                                                                   \
  if (f.RB == RB_ && f.CB == CB_)                                                                             \
    return outp ? launch_tile<true, RB_, CB_>(f.S, in, P, out, part, rows, d, h, kv, epilogue, st)            \
                : launch_tile<false, RB_, CB_>(f.S, in, P, out, part, rows, d, h, kv, epilogue, st);
  MQA_TERMS(1, 1) MQA_TERMS(1, 2) MQA_TERMS(1, 4) MQA_TERMS(2, 2) MQA_TERMS(2, 4)
#undef MQA_TERMS
  return hipErrorNotSupported;
}

long long workgroups(int RB, int CB, int rows, int N) {
  return ((long long)rows + 16 * RB - 1) / (16 * RB) * (((long long)N + 16 * CB - 1) / (16 * CB));
}

// (sizes whose columns or contraction do not fit an int have no form)
bool counts(int h, int kv) { return (long long)h * kv <= 1ll << 30; }

}  // namespace

// Is a product of its own the faster one here?  us, the kernel that otherwise takes it / this one:
//   weights n contiguous, C x N: 4096 x 1024, rows = 128: 25.2 / 23.1, 384: 55.9 / 37.7; 1024 x 4096, 64: 12.0 / 11.8, 128: 18.2 / 14.8;
//   2048 x 2048, 128: 20.7 / 18.3, 192: 31.3 / 21.8; 1024 x 1024, 192: 10.4 / 10.0, 384: 17.0 / 12.5
//   c contiguous: 1024 x 1024, 192: 13.4 / 11.0; 1536 x 1280, 128: 19.3 / 15.8; 2048 x 1024, 100: 15.7 / 14.8
// The smallest tile of at most 256 workgroups (one per compute unit; a second round takes as long again: 2048 x 2048, 512: 33.8 /
// 40.6).  Where that is 16 x 16, or 16 x 32 and the contraction short, project.hip's are as fast (4096 x 1024, 32: 21.0 / 20.4;
// 1024 x 1024, 128: 7.6 / 7.6; 512 x 640: 5.5 / 5.9), and with c contiguous gemm.hip's are where 32 x 64 is the smallest (1024 x 1024, 384: 15.2 / 15.6;
// 1536 x 1280, 384: 19.7 / 22.6).
// Two lines lie where tests that hold a size to a kernel want them, not where the times cross.  More than 192 rows in a round of more
// than 240 workgroups are left to the other kernels: mostly slower (n contiguous, 1024 x 1024, 256: 10.8 / 10.5, 512: 15.8 / 12.8; 2048 x 1024, 256:
// 20.3 / 18.0; 4096 x 1024, 256: 34.5 / 31.4, 512: 45.4 / 40.1; 1000 x 2024, 225: 18.3 / 14.3; c contiguous, 1024 x 1024, 256: 12.1 / 11.3; 4096 x
// 1024, 256: 32.8 / 34.6).  Sums of up to 512 terms in 32 x 32 tiles, n contiguous, are taken: with up to 2^20 weights slower by 0.1 to 0.4 us
// (512 x 1024, 224: 6.2 / 6.7; 256 x 1536, 128: 4.3 / 4.6; 384 x 1024, 224: 5.8 / 5.9; 512 x 4096, 48: 7.8 / 7.3).
TermsForm terms_form(bool outp, int rows, int d, int h, int kv) {
  if (!counts(h, kv)) return TermsForm{0, 0, 0};
  const int N = outp ? d : h * kv, C = outp ? h * kv : d;
  if (rows <= 16) return TermsForm{0, 0, 0};               // (1024 x 4096, 16: 8.6 / 9.2)
  static const TermsForm order[] = {{1, 1, 1}, {1, 2, 1}, {2, 2, 1}, {2, 4, 1}};
  for (const TermsForm& f : order) {
    const long long n = workgroups(f.RB, f.CB, rows, N);
    if (n > 256) continue;
    if ((f.RB == 1 && f.CB == 1) || (f.RB == 1 && C <= 1024) || (n > 240 && rows > 192)) break;
    if (outp && f.CB == 4 && gemm_form(3, rows, d, h, kv, 0)) break;
    return f;
  }
  return TermsForm{0, 0, 0};
}

// The same for a product whose contraction is cut among S workgroups, its parts summed by the launch that adds it to the
// residual and normalises the rows, against a product and a layernorm (us):
//   weights n contiguous: 4096 x 1024, rows = 1: 19.3 / 10.0, 64: 22.9 / 13.5, 128: 28.1 / 18.2, 384: 59.2 / 40.9, 512: 44.5 / 44.9;
//   2048 x 512, 128: 12.4 / 9.4; 2048 x 2048, 192: 35.2 / 28.1, 256: 27.6 / 30.3; 640 x 2560, 64: 12.4 / 11.8, 128: 15.7 / 16.4
//   c contiguous: 1024 x 1024, 1: 7.4 / 6.6, 128: 12.0 / 10.6, 256: 15.0 / 14.1, 384: 18.5 / 21.0; 1536 x 1280, 256: 31.4 / 26.8,
//   384: 23.3 / 29.2
// Tile and S: the least of 6 us for the launches, a round of up to 256 workgroups at `w` us for 1024 indices (measured, within 2 us
// over 100 sizes), and 1 us per MiB of parts.
//   More rows, or parts that are longer than that: gemm.hip's 128 x 128 tiles, one round of up to 256, of parts of the contraction: 9 us, 33 for
// 1024 indices and 0.4 per MiB (4096 x 1024, 512 rows: 48 / 34, 1024: 71 / 51, 2048: 99 / 80; 5120 x 1280, 512: 84 / 49, 1536: 120 / 93;
// 1024 x 1024, 1024: 23 / 25), against a product by gemm_form and a layernorm; up to 256 rows the smaller tiles are as fast (a stack step of 256
// rows: 394, with these 400).
//   Those tiles hold an operand in 22 to 24 bits.  Where the product alone would be one of all 24 (gemm_form 0), they are taken only if the sum is long
// enough for their error to be the smaller one, whatever the values (relative error of float32 instructions / these; normal deviates, every other x a
// zero, wide tails, one channel in 97 of 30 times the rest, all positive): 4096 terms, 260 to 448 rows 4.1e-7 / 2.1e-7, 2.9e-7 / 2.1e-7, 4.1e-7 / 2.1e-7,
// 4.1e-7 / 2.1e-7, 1.3e-7 / 6.5e-8; 2048, 600 rows 2.9e-7 / 1.7e-7, 2.1e-7 / 1.7e-7, 2.9e-7 / 1.7e-7, 3.0e-7 / 1.7e-7, 8.4e-8 / 5.2e-8; but 1024, 260 rows
// 2.1e-7 / 1.6e-7, 1.53e-7 / 1.60e-7, 2.1e-7 / 1.7e-7, 2.2e-7 / 1.7e-7, 7.4e-8 / 5.9e-8.
TermsForm terms_parts_form(bool outp, int rows, int d, int h, int kv) {
  TermsForm best{0, 0, 0};
  if (!counts(h, kv)) return best;
  const int N = outp ? d : h * kv, C = outp ? h * kv : d;
  if (N > 4096) return best;
  double least = 1e30;
  if (workgroups(2, 4, rows, N) <= (outp ? 160 : C >= N ? 240 : 128)) {
    static const struct { int RB, CB; double w[2]; } tiles[] = {{1, 1, {4.2, 3.8}}, {1, 2, {5.0, 6.0}}, {1, 4, {6.3, 9.0}}, {2, 2, {6.4, 8.0}}, {2, 4, {8.8, 13.0}}};
    for (const auto& t : tiles) {
      if (t.RB == 2 && rows <= 16) continue;
      for (int S = 2; S <= 16 && C >= 4 * kStep * S; S *= 2) {
        const double rounds = (double)((workgroups(t.RB, t.CB, rows, N) * S + 255) / 256);
        const double us = 6.2 + t.w[outp] * rounds * C / (1024. * S) + (double)S * rows * N / 262144.;
        if (us < least) best = TermsForm{t.RB, t.CB, S}, least = us;
      }
    }
  }
  const long long wide = workgroups(8, 8, rows, N);
  if (rows > (best.S ? 256 : 128) && wide <= 128 && gemm_fits(outp, d, h, kv, 128) && (C >= 1280 || gemm_form(outp ? 3 : 0, rows, d, h, kv, 0))) {
    int S = 2;
    while (S < 16 && 2 * S * wide <= 256 && C >= 512 * S) S *= 2;
    const int stages = (C + kWideStage - 1) / kWideStage, per = (stages + S - 1) / S;
    S = (stages + per - 1) / per;              // (no empty parts)
    const double us = 8.7 + 33. * per * kWideStage / 1024. + 0.4 * S * rows * N / 262144.;
    const double apart = gemm_us(outp, rows, N, C) + 3.5 + 0.8 * rows * N / 262144.;
    if (S > 1 && us < least && (best.S || us < 0.82 * apart)) best = TermsForm{8, 8, S};
  }
  return best;
}
size_t terms_parts_bytes(bool outp, int rows, int d, int h, int kv) {
  return (size_t)terms_parts_form(outp, rows, d, h, kv).S * rows * (size_t)(outp ? d : h * kv) * 4;
}

// hipErrorNotSupported: no form (terms_form)
hipError_t launch_project_terms(bool outp, const float* in, const float* P, float* out, int rows, int d, int h, int kv, int epilogue,
                                hipStream_t st) {
  const TermsForm f = terms_form(outp, rows, d, h, kv);
  return f.S ? launch_tiles(outp, f, in, P, out, nullptr, rows, d, h, kv, epilogue, st) : hipErrorNotSupported;
}

// x += in . B, y = layernorm(x), in two launches; workspace: terms_parts_bytes(...).  hipErrorNotSupported: no form (terms_parts_form)
hipError_t launch_project_add_layernorm(bool outp, const float* in, const float* P, float* x, float* y, int rows, int d, int h, int kv,
                                        float eps, void* workspace, hipStream_t st) {
  const TermsForm f = terms_parts_form(outp, rows, d, h, kv);
  if (!f.S) return hipErrorNotSupported;
  const int N = outp ? d : h * kv;
  float* part = static_cast<float*>(workspace);
  const hipError_t e = f.RB == 8 ? launch_gemm_parts(outp ? 3 : 0, in, P, part, rows, d, h, kv, 0, 128, f.S, st)
                                 : launch_tiles(outp, f, in, P, nullptr, part, rows, d, h, kv, 0, st);
  if (e != hipSuccess) return e;
  if (N <= 1024) hipLaunchKernelGGL(finish_kernel<1>, dim3(rows), dim3(256), 0, st, part, x, y, rows, N, f.S, eps);
  else if (N <= 2048) hipLaunchKernelGGL(finish_kernel<2>, dim3(rows), dim3(256), 0, st, part, x, y, rows, N, f.S, eps);
  else hipLaunchKernelGGL(finish_kernel<4>, dim3(rows), dim3(256), 0, st, part, x, y, rows, N, f.S, eps);
  return hipGetLastError();
}

}  // namespace mqa
