// Products of the decoder stack whose operands are laid out beforehand.
//
// A packed matrix [lines][C] (C a multiple of 32) holds x 2^s as two fp16 terms, hi + lo, each the nearest fp16 of what is
// left (22 to 24 significant bits, gemm.hip's operands): for every 32 indices a plane of hi and one of lo, in each line after line 64 bytes.
// What a product wants of 16 neighbouring lines is then 1 KiB in one piece, and what makes a row writes 64 bytes at a time.
//
// Packed are the weights, once (a line is a column of the product, scaled by the power of two that takes its largest value to
// [2^14, 2^15)), and the activations that the stack makes itself, whose range is known before they are: a layernorm's row has a norm of at most
// sqrt(d), so one scale holds it whatever comes; so has relu(layernorm . W1), each column of which is at most d times the
// largest value of its column of W1: it keeps that column's scale, which the rows of W2 have been divided by.  So a product
// is nothing but loads and fp16 instructions:
//   a.b = ah bh + (ah bl + al bh)                           (al bl is below 2^-22 |a||b|, 2^-25 typically)
// Weights that two terms do not hold (a column with more than a few values below 2^-17 of its largest next to one another, a NaN, an infinity) are
// told by the pack (`verdict`) and multiplied by gemm.hip, which looks at its operands at run time.
//
// What bounds it: the matrix cores and the power they draw.  Against gemm.hip, which splits both operands on the way to LDS (us, TFLOP/s of
// the float32 product): 16384 x 1024 x 4096: 417 -> 337 (408), 16384 x 4096 x 1024: 393 -> 315 (436: 1.31 PFLOP/s of fp16 products; a
// library product of 8192^3 reaches 1.35), 3000 x 1024 x 1024: 33.7 -> 27.7, 600 x 4096 x 1024: 57 -> 28 (in four parts), 1 x 1024 x
// 32768: 26.4 -> 24, 128 x 1024 x 32768: 43 -> 36.5.  Of that: no splitting in the way 417 -> 376; v_mfma_f32_16x16x32 in the place of
// 32x32x16 376 -> 368 (less power: 402 -> 330 at 4096 x 1024); LDS reads without bank conflicts 368 -> 337.  One wave per SIMD with
// 128 x 128 sums: 401.
#include "common.hpp"

#include <math.h>
#include <type_traits>

namespace mqa {
namespace {

typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(8))) _Float16 halfx8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

__device__ __forceinline__ void load_lds16(const unsigned char* src, unsigned char* dst) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src, (__attribute__((address_space(3))) void*)dst, 16, 0, 0);
}
template <int N> __device__ __forceinline__ void wait_and_meet() {      // at most N loads still on their way; nothing read from LDS any more
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// Eight values -> the 16 bytes of a line's planes, `plane` bytes apart.
__device__ __forceinline__ void store_packed8(unsigned char* at, size_t plane, const float (&v)[8]) {
  uint32_t hi[4], lo[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const Split2 s = split2(v[2 * p], v[2 * p + 1]);
    hi[p] = s.hi; lo[p] = s.lo;
  }
  *reinterpret_cast<uint4*>(at) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
  *reinterpret_cast<uint4*>(at + plane) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}

struct PackedProduct {
  const unsigned char* x;      // packed [C / 32][2][rows][64]
  const unsigned char* w;      // packed [C / 32][2][N][64]
  const float* col_scale;      // [N] what takes a finished sum of a column back
  float scale;                 // ... and what all of them have in common
  void* out;                   // float32 [parts][rows][N] or packed [N / 32][2][rows][64]
  int rows, N, blocks;         // blocks: of 32 indices
  int epilogue;                // 0 store, 1 relu, 2 add to what out holds, 3 relu into a packed matrix
  int tiles_m, tiles_n, per;   // per: blocks of a part of the contraction
};

// Eight sums of neighbouring columns of one row; ADD: to what is there, read beforehand
__device__ __forceinline__ float* place8(const PackedProduct& p, int row, int n, int part) {
  return static_cast<float*>(p.out) + ((size_t)part * p.rows + row) * p.N + n;
}
template <bool ADD>
__device__ __forceinline__ void finish8(const PackedProduct& p, int row, int n, int part, float (&v)[8], floatx4 was0, floatx4 was1) {
  if (!ADD && p.epilogue == 3) {       // (the columns keep the scale of their weights)
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f) * p.scale;
    store_packed8(static_cast<unsigned char*>(p.out) + ((size_t)(n >> 5) * 2 * p.rows + row) * 64 + (n >> 3 & 3) * 16, (size_t)p.rows * 64, v);
    return;
  }
  const floatx4 c0 = *reinterpret_cast<const floatx4*>(p.col_scale + n), c1 = *reinterpret_cast<const floatx4*>(p.col_scale + n + 4);
  floatx4 y0, y1;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    y0[e] = v[e] * c0[e] * p.scale;
    y1[e] = v[4 + e] * c1[e] * p.scale;
    if (ADD) {
      y0[e] += was0[e];
      y1[e] += was1[e];
    } else if (p.epilogue == 1) {
      y0[e] = fmaxf(y0[e], 0.f);
      y1[e] = fmaxf(y1[e], 0.f);
    }
  }
  float* dst = place8(p, row, n, part);
  *reinterpret_cast<floatx4*>(dst) = y0;
  *reinterpret_cast<floatx4*>(dst + 4) = y1;
}

// Tile of TM rows x TN columns, 8 waves: WN x WM of them in each of KG groups; a stage is KG blocks, group kg works on block kg; NB
// stages in LDS, NB - 1 of them on their way (straight from memory to LDS).  Weights are the instruction's row operand, so that a
// lane's sums are neighbouring columns of one row.  LOW: the small products have a running sum of their own, added at the end
// (1024 terms: error 1.7e-7 instead of 2.7e-7); without, they are added first (3.57e-7, last 3.64e-7).
template <int TN, int TM, int WN, int WM, int KG, int NB, bool LOW>
struct PackedTile {
  static constexpr int NX = KG * 2 * TM / 16, NW = KG * 2 * TN / 16;      // KiB of a stage, one instruction of a wave each
  static constexpr int LJ = (NX + NW) / 8;
  static constexpr int STAGE = (NX + NW) * 1024;
  static constexpr int PART = KG > 1 ? KG * TN * TM * 4 : 0;
  static constexpr int LDS = NB * STAGE > PART ? NB * STAGE : PART;
  static_assert(WN * WM * KG == 8 && (NX + NW) % 8 == 0 && LDS <= 160 * 1024, "8 waves, every one with as many loads");
};
template <int TN, int TM, int WN, int WM, int KG, int NB, bool LOW>
__global__ __launch_bounds__(512, 2)
void packed_tile_kernel(PackedProduct p) {
  typedef PackedTile<TN, TM, WN, WM, KG, NB, LOW> L;
  constexpr int RN = TN / WN / 16, RM = TM / WM / 16, LJ = L::LJ;
  extern __shared__ __align__(16) unsigned char smem[];
  // tiles: every XCD takes a contiguous run, column-major inside groups of 8 tile rows, as in gemm.hip
  const int per_xcd = gridDim.x >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= p.tiles_m * p.tiles_n) return;
  const int band = tile / (8 * p.tiles_n), in_band = tile - band * 8 * p.tiles_n;
  const int band_rows = min(8, p.tiles_m - band * 8);
  const int row0 = (band * 8 + in_band % band_rows) * TM, n0 = (in_band / band_rows) * TN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, kk = lane >> 4;
  const int kg = wave / (WN * WM), wn = wave / WM % WN, wm = wave % WM;
  const int first = blockIdx.y * p.per, blocks = min(p.per, p.blocks - first), nst = (blocks + KG - 1) / KG;

  // Staging: an instruction brings 16 lines of a plane; the four 16-byte pieces of line r are in the order piece ^ f(r / 4 & 3),
  // f = 0, 2, 3, 1, so that 16 lanes that read one piece of 16 lines, or two neighbouring pieces of eight each, meet 16
  // different groups of banks.  Lines past the end are the last one again (their sums are not stored).
  uint32_t off[LJ];
#pragma unroll
  for (int j = 0; j < LJ; ++j) {
    const int at = j * 8 + wave;               // which KiB of the stage: x's (group, plane, 16 lines), then the weights'
    const int r = (at < L::NX ? at : at - L::NX) * 16 + (lane >> 2), q = r >> 2 & 3, piece = (lane & 3) ^ (((q << 1) ^ (q >> 1) * 3) & 3);
    off[j] = (uint32_t)(at < L::NX ? min(row0 + r % TM, p.rows - 1) : min(n0 + r % TN, p.N - 1)) * 64u + piece * 16;
  }
  auto load_stage = [&](int st) {
    unsigned char* to = smem + (st % NB) * L::STAGE + wave * 1024;
#pragma unroll
    for (int j = 0; j < LJ; ++j) {
      const int at = j * 8 + wave, unit = at < L::NX ? at * 16 / TM : (at - L::NX) * 16 / TN;      // (group, plane)
      const int b = first + min(st * KG + (unit >> 1), blocks - 1);
      const unsigned char* base = at < L::NX ? p.x + ((size_t)b * 2 + (unit & 1)) * p.rows * 64 : p.w + ((size_t)b * 2 + (unit & 1)) * p.N * 64;
      load_lds16(base + off[j], to + j * 8192);
    }
  };
  floatx4 acc[RN][RM], low[LOW ? RN : 1][LOW ? RM : 1];
#pragma unroll
  for (int a = 0; a < RN; ++a)
#pragma unroll
    for (int b = 0; b < RM; ++b) {
      acc[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (LOW) low[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  const int turn = (((i >> 2) << 1) ^ (i >> 3) * 3) & 3;
  const int x0 = (kg * 2 * TM + wm * RM * 16 + i) * 64 + (kk ^ turn) * 16;
  const int w0 = L::NX * 1024 + (kg * 2 * TN + wn * RN * 16 + i) * 64 + (kk ^ turn) * 16;

#pragma unroll
  for (int s = 0; s < NB - 1; ++s)
    if (s < nst) load_stage(s);
  for (int st = 0; st < nst; ++st) {
    // stage st is there (those behind it may be on their way), and its predecessor's place is free
    if (nst - 1 - st >= NB - 2) wait_and_meet<LJ * (NB - 2)>();
    else wait_and_meet<0>();
    if (st + NB - 1 < nst) load_stage(st + NB - 1);
    if (KG > 1 && st * KG + kg >= blocks) continue;        // (the same for the whole wave; the barriers are above)
    const unsigned char* at = smem + (st % NB) * L::STAGE;
    halfx8 x[2][RM], w[2][RN];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int b = 0; b < RM; ++b) x[t][b] = *reinterpret_cast<const halfx8*>(at + x0 + t * (TM * 64) + b * 1024);
#pragma unroll
      for (int a = 0; a < RN; ++a) w[t][a] = *reinterpret_cast<const halfx8*>(at + w0 + t * (TN * 64) + a * 1024);
    }
    auto product = [&](auto small, int tw, int tx) {
#pragma unroll
      for (int a = 0; a < RN; ++a)
#pragma unroll
        for (int b = 0; b < RM; ++b) {
          floatx4& to = LOW && decltype(small)::value ? low[LOW ? a : 0][LOW ? b : 0] : acc[a][b];
          to = __builtin_amdgcn_mfma_f32_16x16x32_f16(w[tw][a], x[tx][b], to, 0, 0, 0);
        }
    };
    if constexpr (LOW) product(std::false_type{}, 0, 0);
    product(std::true_type{}, 0, 1);
    product(std::true_type{}, 1, 0);
    if constexpr (!LOW) product(std::false_type{}, 0, 0);
  }
  if constexpr (LOW)
#pragma unroll
    for (int a = 0; a < RN; ++a)
#pragma unroll
      for (int b = 0; b < RM; ++b) acc[a][b] += low[a][b];

  // Register e of lane (i, kk): column 4 kk + e, row i of the block.  Two blocks of columns change rows of lanes so that a lane
  // has eight neighbouring columns of one.  KG > 1: the groups' sums meet in LDS, each group finishes a share.
  constexpr int PAIRS = RN / 2 * RM, SHARE = (PAIRS + KG - 1) / KG;
  static_assert(RN % 2 == 0, "blocks of columns in pairs");
  const floatx4* part = reinterpret_cast<const floatx4*>(smem) + (wave % (WN * WM)) * (RN * RM * 64) + lane;
  if constexpr (KG > 1) {
    __syncthreads();
    floatx4* mine = reinterpret_cast<floatx4*>(smem) + wave * (RN * RM * 64) + lane;
#pragma unroll
    for (int a = 0; a < RN; ++a)
#pragma unroll
      for (int b = 0; b < RM; ++b) mine[(a * RM + b) * 64] = acc[a][b];
    __syncthreads();
  }
  auto finish = [&](auto add) {
    constexpr bool ADD = decltype(add)::value;
    // What a sum is added to: the loads of eight blocks in flight together.  One by one, each behind the last one's stores: 16384 x 4096 x 1024
    // in a stack 324 us, so 297; x 1024 x 1024 131, so 98 (without the adding 85)
    constexpr int BATCH = ADD && SHARE > 8 ? 8 : SHARE;
#pragma unroll
    for (int k0 = 0; k0 < SHARE; k0 += BATCH) {
      floatx4 was[ADD ? BATCH : 1][2];
      auto place = [&](int k, int& row, int& n) {
        const int at = kg * SHARE + k, a = at / RM * 2, b = at % RM;
        row = row0 + wm * RM * 16 + b * 16 + i, n = n0 + wn * RN * 16 + a * 16 + 16 * (kk & 1) + 8 * (kk >> 1);
        return !(PAIRS % KG && at >= PAIRS) && row < p.rows && n < p.N;
      };
      int row, n;
      if constexpr (ADD)
#pragma unroll
        for (int k = 0; k < BATCH; ++k)
          if (k0 + k < SHARE && place(k0 + k, row, n)) {
            const floatx4* from = reinterpret_cast<const floatx4*>(place8(p, row, n, blockIdx.y));
            was[k][0] = from[0];
            was[k][1] = from[1];
          }
#pragma unroll
      for (int k = k0; k < k0 + BATCH && k < SHARE; ++k) {
        floatx4 lo, hi;
        float v[8];
        const int at = kg * SHARE + k, a = at / RM * 2, b = at % RM;
        if (PAIRS % KG && at >= PAIRS) break;
        if constexpr (KG == 1) {
          lo = acc[k / RM * 2][k % RM];
          hi = acc[k / RM * 2 + 1][k % RM];
        } else {
          lo = hi = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < KG; ++q) {
            const floatx4* from = part + q * (WN * WM * RN * RM * 64) + (a * RM + b) * 64;
            lo += from[0];
            hi += from[RM * 64];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(lo[e]), __float_as_uint(hi[e]), false, false);
          v[e] = __uint_as_float(s[0]);
          v[4 + e] = __uint_as_float(s[1]);
        }
        if (place(k, row, n)) finish8<ADD>(p, row, n, blockIdx.y, v, was[ADD ? k - k0 : 0][0], was[ADD ? k - k0 : 0][1]);
      }
    }
  };
  if (p.epilogue == 2) finish(std::true_type{});
  else finish(std::false_type{});
}

template <int TN, int TM, int WN, int WM, int KG, int NB, bool LOW>
hipError_t launch_tile(PackedProduct p, int S, hipStream_t st) {
  typedef PackedTile<TN, TM, WN, WM, KG, NB, LOW> L;
  auto kern = packed_tile_kernel<TN, TM, WN, WM, KG, NB, LOW>;
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  p.tiles_m = (p.rows + TM - 1) / TM, p.tiles_n = (p.N + TN - 1) / TN;
  p.per = (p.blocks + S - 1) / S;
  const long long tiles = (long long)p.tiles_m * p.tiles_n;
  hipLaunchKernelGGL(kern, dim3((unsigned)((tiles + 7) / 8 * 8), S), dim3(512), L::LDS, st, p);
  return hipGetLastError();
}

// ---- Weights: 32 columns x 256 indices per workgroup; the largest value of each column, then (WRITE) its scale and the terms.
constexpr float kSmall = 0.125f;               // scaled values from here on are held to 2^-22 of themselves
constexpr int kFew = 6;                        // ... of 256 neighbouring ones of a column that may be smaller

__global__ __launch_bounds__(256)
void clear_kernel(float* a, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) a[i] = 0.f;
}

// most: [N] bits of the columns' largest values on the way in, 1 / scale on the way out of `finish_scales_kernel`
template <bool KC, bool WRITE>
__global__ __launch_bounds__(256)
void pack_weights_kernel(const float* __restrict__ P, const float* __restrict__ row_scale, unsigned char* __restrict__ packed,
                         uint32_t* most, int32_t* __restrict__ verdict, int d, int h, int kv) {
  __shared__ uint32_t tally[32];               // largest values, or counts of small ones
  const int C = KC ? h * kv : d, N = KC ? d : h * kv;
  if (threadIdx.x < 32) tally[threadIdx.x] = 0;
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (int u = 0; u < 4; ++u) {                // neighbouring lanes where the weights are contiguous
    const int j = KC ? (threadIdx.x >> 5) + 8 * u : threadIdx.x & 31, o = blockIdx.y * 32 + (KC ? threadIdx.x & 31 : (threadIdx.x >> 5) + 8 * u);
    const int n = blockIdx.x * 32 + j, c = 8 * o;
    if (n >= N || c >= C) continue;            // (C is a multiple of 32, and eight indices stay inside one head: kv % 8 == 0)
    const float* at = KC ? P + (size_t)(c / kv) * d * kv + (size_t)n * kv + c % kv : P + (size_t)(n / kv) * d * kv + (size_t)c * kv + n % kv;
    float v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = at[KC ? e : (size_t)e * kv] * (row_scale ? row_scale[c + e] : 1.f);
    if constexpr (!WRITE) {
      float peak = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        bad |= !(fabsf(v[e]) < 0x1p100f);      // (a NaN, too)
        peak = fmaxf(peak, fabsf(v[e]));
      }
      bad |= peak > 0.f && peak < 0x1p-100f;   // (so small that the scale is not there)
      atomicMax(&tally[j], __float_as_uint(peak));
    } else {
      const float m = __uint_as_float(most[n]), scale = split_scale(m > 0.f ? m : 1.f, 14);
      int few = 0;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] *= scale;
        few += v[e] != 0.f && fabsf(v[e]) < kSmall ? 1 : 0;
      }
      if (few) atomicAdd(&tally[j], (uint32_t)few);
      store_packed8(packed + ((size_t)(o >> 2) * 2 * N + n) * 64 + (o & 3) * 16, (size_t)N * 64, v);
    }
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    const int n = blockIdx.x * 32 + threadIdx.x;
    if constexpr (WRITE) bad = tally[threadIdx.x] > kFew;
    else if (n < N) atomicMax(&most[n], tally[threadIdx.x]);
  }
  if (bad) *verdict = 1;                       // (whoever finds it writes the same)
}
__global__ __launch_bounds__(256)
void finish_scales_kernel(float* most, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) most[i] = 1.f / split_scale(most[i] > 0.f ? most[i] : 1.f, 14);
}

}  // namespace

// Tiles, what a round of 256 of them takes for 1024 indices (us; measured, many rows and all parts in one round), and the relative
// error of a sum of 1024 normal deviates (x 1e-7; it grows with the root of the length).
struct PackedForm { int TN, TM; double us, error; };
static const PackedForm kForms[] = {{256, 256, 70, 3.57}, {256, 128, 42, 2.19}, {128, 128, 23.5, 1.68}, {128, 64, 15, 1.68}, {64, 64, 8.2, 1.38}, {128, 32, 9, 1.38}};
constexpr int kPackedForms = 6;

bool packed_fits(int rows, int N, int C) {
  return rows > 0 && N > 0 && C > 0 && C % 32 == 0 && N % 8 == 0 && C <= 1 << 24 && rows <= 1 << 25 && N <= 1 << 25;      // (32-bit offsets inside a plane)
}

// The form and the parts of the contraction (1: none) that take the least time here, by
//   4 us + rounds of 256 tiles x `us` x C / 1024 / parts + 0.4 us per MiB of parts (what a launch that reads the row anyway spends on them),
// among those whose error is no larger than `error` (x 1e-7 for 1024 terms of a chain, `length` of them in it); -1: none.
int packed_form(int rows, int N, int C, bool parts, double error, int length) {
  int best = -1;
  double least = 1e30;
  for (int f = 0; f < kPackedForms; ++f)
    for (int S = 1; S <= (parts ? 8 : 1) && (S == 1 || C >= 256 * S); S *= 2) {
      const int blocks = C / 32, per = (blocks + S - 1) / S;
      if (S > 1 && (blocks + per - 1) / per != S) continue;             // (no empty parts)
      const double len = 32. * per > 512. ? 32. * per : 512., len0 = length > 512 ? length : 512.;
      if (kForms[f].error * sqrt(len) > error * sqrt(len0)) continue;
      const double tiles = (double)((N + kForms[f].TN - 1) / kForms[f].TN) * ((rows + kForms[f].TM - 1) / kForms[f].TM) * S;
      const double us = 4. + ceil(tiles / 256.) * kForms[f].us * 32. * per / 1024. + (S > 1 ? 0.4 * S * rows * (double)N / 262144. : 0.);
      if (us < least) least = us, best = 16 * f + S;
    }
  return best;
}

// The form of a stack's product of packed operands, 16 x its number + parts; 0 where it stays with the kernels that read the float32 weights:
// a product of few rows that is one of three exact terms there (project_terms.hip), whose error two terms do not reach, and
// sizes without a form.  residual: x += product, layernorm follows (mqa_project_add_layernorm's sizes).
int packed_plan(int mode, int rows, int d, int h, int kv, int residual) {
  const bool outp = mode == 3;
  if ((long long)h * kv > 1 << 24) return 0;
  const int N = outp ? d : h * kv, C = outp ? h * kv : d;
  if (!packed_fits(rows, N, C) || C < 64 || (residual && N > 4096)) return 0;
  int edge = 0, length = C;
  if (residual) {
    const TermsForm f = terms_parts_form(outp, rows, d, h, kv);
    if (f.S && f.RB != 8) return 0;
    if (f.S) edge = 128, length = (C + f.S - 1) / f.S;
  }
  if (!edge) {
    if (terms_form(outp, rows, d, h, kv).S) return 0;
    edge = gemm_form(mode, rows, d, h, kv, 0);
  }
  const double error = edge == 256 ? 3.62 : edge == 128 ? 2.65 : edge == 64 ? 2.0 : edge == 32 ? 1.6 : 2.07;      // (of 1024 terms: gemm.hip, project.hip)
  if (!edge && (double)N * C < 8e6) return 0;  // (few rows: 16 x 1024 x 4096 6.3 there, 7.5 here; 1 x 1024 x 32768 26.4 / 24)
  const int form = packed_form(rows, N, C, residual, error, length);
  return form < 0 ? 0 : form;
}

hipError_t launch_packed_product(const void* x, const void* w, float scale, void* out, int rows, int N, int C, int epilogue, int form,
                                 hipStream_t st) {
  const unsigned char* wp = static_cast<const unsigned char*>(w);
  const PackedProduct p{static_cast<const unsigned char*>(x), wp, reinterpret_cast<const float*>(wp + packed_bytes(N, C)), scale, out, rows, N, C / 32, epilogue, 0, 0, 0};
  const int S = form & 15;
  switch (form >> 4) {
    case 0: return launch_tile<256, 256, 4, 2, 1, 2, false>(p, S, st);
    case 1: return launch_tile<256, 128, 4, 2, 1, 3, true>(p, S, st);
    case 2: return launch_tile<128, 128, 2, 2, 2, 2, true>(p, S, st);
    case 3: return launch_tile<128, 64, 2, 2, 2, 3, true>(p, S, st);
    case 4: return launch_tile<64, 64, 2, 1, 4, 2, true>(p, S, st);
    case 5: return launch_tile<128, 32, 2, 1, 4, 2, true>(p, S, st);
  }
  return hipErrorNotSupported;
}

hipError_t launch_pack_weights(bool outp, const float* P, const float* row_scale, void* packed, int32_t* verdict, int d, int h, int kv, hipStream_t st) {
  const int N = outp ? d : h * kv, C = outp ? h * kv : d;
  unsigned char* to = static_cast<unsigned char*>(packed);
  float* scales = reinterpret_cast<float*>(to + packed_bytes(N, C));
  uint32_t* most = reinterpret_cast<uint32_t*>(scales);
  const dim3 grid((N + 31) / 32, (C + 255) / 256), lines((N + 255) / 256), block(256);
  hipLaunchKernelGGL(clear_kernel, lines, block, 0, st, scales, N);
  if (outp) {
    hipLaunchKernelGGL((pack_weights_kernel<true, false>), grid, block, 0, st, P, row_scale, to, most, verdict, d, h, kv);
    hipLaunchKernelGGL((pack_weights_kernel<true, true>), grid, block, 0, st, P, row_scale, to, most, verdict, d, h, kv);
  } else {
    hipLaunchKernelGGL((pack_weights_kernel<false, false>), grid, block, 0, st, P, row_scale, to, most, verdict, d, h, kv);
    hipLaunchKernelGGL((pack_weights_kernel<false, true>), grid, block, 0, st, P, row_scale, to, most, verdict, d, h, kv);
  }
  hipLaunchKernelGGL(finish_scales_kernel, lines, block, 0, st, scales, N);
  return hipGetLastError();
}

// log2 of what a packed layernorm row of N columns is scaled by: sqrt(N) comes to 2^15 at most
int packed_layernorm_exponent(int N) {
  int s = 15;
  while (s > 0 && ldexp(1., 2 * (15 - s)) < N) --s;
  return s;
}

}  // namespace mqa
