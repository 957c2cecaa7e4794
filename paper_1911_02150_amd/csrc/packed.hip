// The feed-forward of a stack's long prompts, x += relu(layernorm(x) . W1) . W2, from operands that are laid out on the way.
//
// A packed matrix [lines][C] (C a multiple of 32) holds x 2^s as two fp16 terms, hi + lo, each the nearest fp16 of what is
// left (22 to 24 significant bits, gemm.hip's operands): for every 32 indices a plane of hi and one of lo, in each line after line 64 bytes.
// What a product wants of 16 neighbouring lines is then 1 KiB in one piece, and what makes a row writes 64 bytes at a time.
//
// Packed are, in every call, the weights (a line is a column of the product, scaled by the power of two that takes its largest value to
// [2^14, 2^15)) and the activations between, whose range is known before they are: a layernorm's row has a norm of at most
// sqrt(d), so one scale holds it whatever comes; relu(layernorm . W1), each column of which is at most d times the
// largest value of its column of W1, keeps that column's scale, which the rows of W2 have been divided by, to an eighth of that (of normal deviates it
// reaches 2^-5 of it).  So a product is nothing but loads and fp16 instructions:
//   a.b = ah bh + (ah bl + al bh)                           (al bl is below 2^-22 |a||b|, 2^-25 typically)
// What two terms do not hold is looked for where it is packed, and told on the device.  Weights: a column with more than a few values below 2^-17 of its
// largest next to one another, a NaN, an infinity: the whole call.  Rows, by gemm.hip's measure (`row_holds`), or a hidden value past fp16's range: the
// 256 rows around them.  Their packed products return at once, and the launches behind, which return at once otherwise, are
// gemm.hip's on the float32 values.  Nothing is kept from one call for the next, and nothing is asked of the device.
//
// What bounds it: the matrix cores and the power they draw.  Against gemm.hip, which splits both operands on the way to LDS (us, TFLOP/s of
// the float32 product): 16384 x 1024 x 4096: 417 -> 337 (408), 16384 x 4096 x 1024: 393 -> 315 (436: 1.31 PFLOP/s of fp16 products; a
// library product of 8192^3 reaches 1.35).  Of that: no splitting in the way 417 -> 376; v_mfma_f32_16x16x32 in the place of
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
  const int32_t* flag;         // not 0: this product is not to be
  int32_t* bad;                // [rows / 256] not 0: of these rows it is not
  uint32_t* tallies;           // [tally_tiles][rows] of the hidden values in one tile: octets (eight neighbouring columns) with a value that the terms hold
  int tally_tiles;             // in few bits, with any but zeros << 8, and with one far above << 16
  const unsigned char* x;      // packed [C / 32][2][rows][64]
  const unsigned char* w;      // packed [C / 32][2][N][64]
  const uint32_t* most;        // [N] bits of the largest value of each column of the weights, as scaled for packing
  float scale;                 // of the finished sums
  void* out;                   // float32 [rows][N], added to, or packed [N / 32][2][rows][64]
  int rows, N, blocks;         // blocks: of 32 indices
  int tiles_m, tiles_n;
};

__device__ __forceinline__ float column_scale(uint32_t most) { return split_scale(most ? __uint_as_float(most) : 1.f, 14); }

// Eight sums of neighbouring columns of one row.  ADD: to what is there, read beforehand; else relu, packed (the columns keep the scale of their weights),
// and counted
template <bool ADD>
__device__ __forceinline__ void finish8(const PackedProduct& p, int row, int n, float (&v)[8], floatx4 was0, floatx4 was1, uint32_t& tally) {
  if constexpr (!ADD) {
    float most = 0.f;
    bool small = false;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      v[e] = fmaxf(v[e], 0.f) * p.scale;
      most = fmaxf(most, v[e]);
      small |= v[e] != 0.f && v[e] < kFull;
    }
    tally += (small ? 1u : 0u) + (most > 0.f ? 1u << 8 : 0u) + (most >= kFarAbove ? 1u << 16 : 0u);
    if (__builtin_expect(!(most < 65504.f), 0)) p.bad[row >> 8] = 1;
    store_packed8(static_cast<unsigned char*>(p.out) + ((size_t)(n >> 5) * 2 * p.rows + row) * 64 + (n >> 3 & 3) * 16, (size_t)p.rows * 64, v);
  } else {
    const u32x4 m0 = *reinterpret_cast<const u32x4*>(p.most + n), m1 = *reinterpret_cast<const u32x4*>(p.most + n + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      was0[e] += v[e] * (1.f / column_scale(m0[e])) * p.scale;
      was1[e] += v[4 + e] * (1.f / column_scale(m1[e])) * p.scale;
    }
    floatx4* dst = reinterpret_cast<floatx4*>(static_cast<float*>(p.out) + (size_t)row * p.N + n);
    dst[0] = was0;
    dst[1] = was1;
  }
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
  static constexpr int STATE = NB * STAGE > PART ? NB * STAGE : PART;
  static constexpr int LDS = STATE + 4 * TM;                             // (behind it the rows' tallies)
  static_assert(WN * WM * KG == 8 && (NX + NW) % 8 == 0 && LDS <= 160 * 1024, "8 waves, every one with as many loads");
};
template <int TN, int TM, int WN, int WM, int KG, int NB, bool LOW, bool ADD>
__global__ __launch_bounds__(512, 2)
void packed_tile_kernel(PackedProduct p) {
  if (*p.flag) return;
  typedef PackedTile<TN, TM, WN, WM, KG, NB, LOW> L;
  constexpr int RN = TN / WN / 16, RM = TM / WM / 16, LJ = L::LJ;
  extern __shared__ __align__(16) unsigned char smem[];
  // tiles: every XCD takes a contiguous run, column-major inside groups of 8 tile rows, as in gemm.hip
  const int per_xcd = gridDim.x >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= p.tiles_m * p.tiles_n) return;
  const int band = tile / (8 * p.tiles_n), in_band = tile - band * 8 * p.tiles_n;
  const int band_rows = min(8, p.tiles_m - band * 8);
  const int tile_n = in_band / band_rows, row0 = (band * 8 + in_band % band_rows) * TM, n0 = tile_n * TN;

  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t* const tally = reinterpret_cast<uint32_t*>(smem + L::STATE);
  if constexpr (ADD) {
    // do the terms hold the hidden values of these 256 rows?  (every tile of theirs comes to the same)
    const int block = row0 >> 8, r = block * 256 + (tid & 255);
    int small = 0, octets = 0, far = 0;
    if (r < p.rows)
      for (int t = tid >> 8; t < p.tally_tiles; t += 2) {
        const uint32_t w = p.tallies[(size_t)t * p.rows + r];
        small += w & 255, octets += w >> 8 & 255, far += w >> 16;
      }
    int (*half)[256] = reinterpret_cast<int (*)[256]>(smem);
    if (tid >= 256) half[0][tid & 255] = small, half[1][tid & 255] = octets, half[2][tid & 255] = far;
    __syncthreads();
    bool bad = p.bad[block] != 0;
    if (tid < 256) bad |= !row_holds(small + half[0][tid], octets + half[1][tid], far + half[2][tid]);
    if (__syncthreads_or(bad)) {
      if (tid == 0) p.bad[block] = 1;
      return;
    }
  } else if (tid < TM) {
    tally[tid] = 0;                            // (barriers between this and its use: below)
  }
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, kk = lane >> 4;
  const int kg = wave / (WN * WM), wn = wave / WM % WN, wm = wave % WM;
  const int blocks = p.blocks, nst = (blocks + KG - 1) / KG;

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
      const int b = min(st * KG + (unit >> 1), blocks - 1);
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
  // What a sum is added to: the loads of eight blocks in flight together.  One by one, each behind the last one's stores: 16384 x 4096 x 1024
  // in a stack 324 us, so 297; x 1024 x 1024 131, so 98 (without the adding 85)
  constexpr int BATCH = ADD && SHARE > 8 ? 8 : SHARE;
  static_assert(SHARE % RM == 0 && PAIRS % KG == 0, "block k of a share is of rows k % RM");
  uint32_t counts[RM] = {};
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
          const floatx4* from = reinterpret_cast<const floatx4*>(static_cast<const float*>(p.out) + (size_t)row * p.N + n);
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
      if (place(k, row, n)) finish8<ADD>(p, row, n, v, was[ADD ? k - k0 : 0][0], was[ADD ? k - k0 : 0][1], counts[k % RM]);
    }
  }
  if constexpr (!ADD) {
#pragma unroll
    for (int b = 0; b < RM; ++b) atomicAdd(&tally[wm * RM * 16 + b * 16 + i], counts[b]);
    __syncthreads();
    if (tid < TM && row0 + tid < p.rows) p.tallies[(size_t)tile_n * p.rows + row0 + tid] = tally[tid];
  }
}

template <int TN, int TM, int WN, int WM, int KG, int NB, bool LOW, bool ADD>
hipError_t launch_tile(PackedProduct p, hipStream_t st) {
  typedef PackedTile<TN, TM, WN, WM, KG, NB, LOW> L;
  auto kern = packed_tile_kernel<TN, TM, WN, WM, KG, NB, LOW, ADD>;
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, L::LDS);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  p.tiles_m = (p.rows + TM - 1) / TM, p.tiles_n = (p.N + TN - 1) / TN;
  const long long tiles = (long long)p.tiles_m * p.tiles_n;
  hipLaunchKernelGGL(kern, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(512), L::LDS, st, p);
  return hipGetLastError();
}

template <bool ADD>
hipError_t launch_product(const PackedProduct& p, int form, hipStream_t st) {
  switch (form) {
    case 0: return launch_tile<256, 256, 4, 2, 1, 2, false, ADD>(p, st);
    case 1: return launch_tile<256, 128, 4, 2, 1, 3, true, ADD>(p, st);
    case 2: return launch_tile<128, 128, 2, 2, 2, 2, true, ADD>(p, st);
  }
  return hipErrorNotSupported;
}

// ---- Weights [C][N]: 32 columns x 256 indices per workgroup, four columns x eight indices per thread, all loads in flight together (in single
// words 14 us for 1024 x 4096, so 6); first the largest value of each column, then (WRITE) the terms.
constexpr float kSmall = 0.125f;               // scaled values from here on are held to 2^-22 of themselves
constexpr int kFew = 6;                        // ... of 256 neighbouring ones of a column that may be smaller

__global__ __launch_bounds__(256)
void clear_kernel(uint32_t* a, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) a[i] = 0;
}

struct PackWeights {
  const float* P;
  const uint32_t* before;      // NULL, or the largest values of the columns of the weights before these, whose scales the rows are divided by
  unsigned char* packed;
  uint32_t* most;
  int C, N, tiles_n;           // (C and N are multiples of 32)
};

template <bool WRITE>
__device__ __forceinline__ void pack_tile(const PackWeights& p, int tile, int32_t* flag, uint32_t* tally) {
  const int n0 = tile % p.tiles_n * 32, o = tile / p.tiles_n * 32 + (threadIdx.x >> 3), q = threadIdx.x & 7, n = n0 + 4 * q, c = 8 * o;
  if (threadIdx.x < 32) tally[threadIdx.x] = 0;      // largest values, or counts of small ones
  __syncthreads();
  bool bad = false;
  if (c < p.C) {
    floatx4 v[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = *reinterpret_cast<const floatx4*>(p.P + (size_t)(c + e) * p.N + n);
    if (p.before) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= 1.f / column_scale(p.before[c + e]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (!WRITE) {
        float peak = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          bad |= !(fabsf(v[e][j]) < 0x1p100f);      // (a NaN, too)
          peak = fmaxf(peak, fabsf(v[e][j]));
        }
        bad |= peak > 0.f && peak < 0x1p-100f;      // (so small that the scale is not there)
        atomicMax(&tally[4 * q + j], __float_as_uint(peak));
      } else {
        const float scale = column_scale(p.most[n + j]);
        float t[8];
        int few = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          t[e] = v[e][j] * scale;
          few += t[e] != 0.f && fabsf(t[e]) < kSmall ? 1 : 0;
        }
        if (few) atomicAdd(&tally[4 * q + j], (uint32_t)few);
        store_packed8(p.packed + ((size_t)(o >> 2) * 2 * p.N + n + j) * 64 + (o & 3) * 16, (size_t)p.N * 64, t);
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < 32) {
    if constexpr (WRITE) bad = tally[threadIdx.x] > kFew;
    else atomicMax(&p.most[n0 + threadIdx.x], tally[threadIdx.x]);
  }
  if (bad) *flag = 1;                          // (whoever finds it writes the same)
}

// `first` tiles: the largest values of `look`; then the terms of `write`
__global__ __launch_bounds__(256)
void pack_kernel(PackWeights look, PackWeights write, int first, int32_t* flag) {
  __shared__ uint32_t tally[32];
  __shared__ int done;
  if (threadIdx.x == 0) done = *flag;          // (other workgroups of this launch may set it: one look for all waves of this one)
  __syncthreads();
  if (done) return;
  if ((int)blockIdx.x < first) pack_tile<false>(look, blockIdx.x, flag, tally);
  else pack_tile<true>(write, blockIdx.x - first, flag, tally);
}

// Tiles, what a round of 256 of them takes for 1024 indices (us; measured), and the relative error of a sum of 1024 normal deviates
// (x 1e-7; it grows with the root of the length).
struct PackedForm { int TN, TM; double us, error; };
const PackedForm kForms[] = {{256, 256, 70, 3.57}, {256, 128, 42, 2.19}, {128, 128, 23.5, 1.68}};

// The form that takes the least time, rounds of 256 tiles x `us` x C / 1024, among those whose error is no larger than gemm.hip's
// in tiles of this edge; -1: none.
int packed_form(int rows, int N, int C, int edge) {
  const double error = edge == 256 ? 3.62 : edge == 128 ? 2.65 : 0.;
  int best = -1;
  double least = 0.;
  for (int f = 0; f < 3; ++f) {
    if (kForms[f].error > error) continue;
    const double tiles = (double)((N + kForms[f].TN - 1) / kForms[f].TN) * ((rows + kForms[f].TM - 1) / kForms[f].TM);
    const double us = ceil(tiles / 256.) * kForms[f].us;
    if (best < 0 || us < least) least = us, best = f;
  }
  return best;
}

// log2 of what a packed layernorm row of N columns is scaled by: sqrt(N) comes to 2^15 at most
int layernorm_exponent(int N) {
  int s = 15;
  while (s > 0 && ldexp(1., 2 * (15 - s)) < N) --s;
  return s;
}

// A call's workspace, in bytes from its beginning: the flag, the columns' largest values and the blocks of rows (cleared by every call), the packed weights,
// then the packed (or, where those are not to be used, the float32) layernorm and hidden rows, and the tallies of these.
struct Places {
  size_t most1, most2, bad, w1, w2, rows, hidden, tallies, bytes;
  Places(int rows_, int d, int ff) {
    most1 = 16, most2 = most1 + 4 * (size_t)ff, bad = most2 + 4 * (size_t)d, w1 = bad + ((size_t)rows_ + 1023) / 1024 * 16;
    w2 = w1 + 4 * (size_t)d * ff, rows = w2 + 4 * (size_t)d * ff, hidden = rows + 4 * (size_t)rows_ * d;
    tallies = hidden + 4 * (size_t)rows_ * ff, bytes = tallies + 4 * (size_t)((ff + 127) / 128) * rows_;
  }
};

}  // namespace

FeedForwardPlan feed_forward_plan(int rows, int d, int ff) {
  FeedForwardPlan f{};
  if (rows <= 0 || d <= 0 || ff <= 0 || (d & 31) || (ff & 31) || d > 4096 || ff > 1 << 20 || rows > 1 << 25) return f;      // (32-bit offsets inside a plane)
  f.edge1 = gemm_edge(rows, ff, d), f.edge2 = gemm_edge(rows, d, ff);
  f.form1 = packed_form(rows, ff, d, f.edge1), f.form2 = packed_form(rows, d, ff, f.edge2);
  if (f.form1 < 0 || f.form2 < 0) return f;
  f.bytes = Places(rows, d, ff).bytes;
  // The weights cost as much for few rows as for many: 30 us for 2 x 1024 x 4096, and the launches that do nothing 15.  us, the three calls / this, values
  // that two terms hold | do not: 16384 x 1024 x 4096 849 / 692 | 841 / 894, 6000 432 / 340 | 431 / 475, 4000 243 / 215, 2500 199 / 195; 16384 x 512 x 2048
  // 273 / 221, 8192 141 / 132; 6000 x 768 x 3072 333 / 273; 8192 x 1280 x 2048 314 / 287, 4000 x 1280 x 5120 511 / 418, 2500 258 / 247.
  f.faster = rows >= 4096 && (double)rows * d * ff >= 12e9 ? 1 : 0;
  return f;
}

// x += relu(layernorm(x) . W1) . W2 from a workspace of the plan's size
hipError_t launch_feed_forward(const FeedForwardPlan& f, const float* W1, const float* W2, float* x, int rows, int d, int ff, float eps, void* workspace,
                               hipStream_t st) {
  unsigned char* const ws = static_cast<unsigned char*>(workspace);
  const Places at(rows, d, ff);
  int32_t *flag = reinterpret_cast<int32_t*>(ws), *bad = reinterpret_cast<int32_t*>(ws + at.bad);
  uint32_t* tallies = reinterpret_cast<uint32_t*>(ws + at.tallies);
  uint32_t *most1 = reinterpret_cast<uint32_t*>(ws + at.most1), *most2 = reinterpret_cast<uint32_t*>(ws + at.most2);
  const int ints = (int)(at.w1 / 4);
  hipLaunchKernelGGL(clear_kernel, dim3((ints + 255) / 256), dim3(256), 0, st, reinterpret_cast<uint32_t*>(ws), ints);
  const PackWeights one{W1, nullptr, ws + at.w1, most1, d, ff, ff / 32}, two{W2, most1, ws + at.w2, most2, ff, d, d / 32};
  const int tiles1 = ff / 32 * ((d + 255) / 256), tiles2 = d / 32 * ((ff + 255) / 256);
  hipLaunchKernelGGL(pack_kernel, dim3(tiles1), dim3(256), 0, st, one, one, tiles1, flag);
  hipLaunchKernelGGL(pack_kernel, dim3(tiles2 + tiles1), dim3(256), 0, st, two, one, tiles2, flag);
  hipLaunchKernelGGL(pack_kernel, dim3(tiles2), dim3(256), 0, st, two, two, 0, flag);
  const int s = layernorm_exponent(d);
  hipError_t e = launch_layernorm_packed(flag, bad, x, ws + at.rows, ldexpf(1.f, s), rows, d, eps, st);
  if (e != hipSuccess) return e;
  // |hx 2^s . W1| <= sqrt(d) 2^s sqrt(d) 2^15 (the columns' largest values are below 2^15), and sqrt(d) 2^s <= 2^15: the hidden rows come to 2^18 at
  // most, and to 2^15 if they are not nearly parallel to a column of W1
  const int tiles = (ff + kForms[f.form1].TN - 1) / kForms[f.form1].TN;
  PackedProduct p{flag, bad, tallies, tiles, ws + at.rows, ws + at.w1, most1, ldexpf(1.f, s - 27), ws + at.hidden, rows, ff, d / 32, 0, 0};
  e = launch_product<false>(p, f.form1, st);
  if (e != hipSuccess) return e;
  p = PackedProduct{flag, bad, tallies, tiles, ws + at.hidden, ws + at.w2, most2, ldexpf(1.f, 27 - 2 * s), x, rows, d, ff / 32, 0, 0};
  e = launch_product<true>(p, f.form2, st);
  if (e != hipSuccess) return e;
  float *hx = reinterpret_cast<float*>(ws + at.rows), *u = reinterpret_cast<float*>(ws + at.hidden);
  e = launch_layernorm_if(flag, bad, x, hx, rows, d, eps, st);
  if (e == hipSuccess) e = launch_gemm_if(flag, bad, f.edge1, hx, W1, u, rows, d, ff, 1, st);
  if (e == hipSuccess) e = launch_gemm_if(flag, bad, f.edge2, u, W2, x, rows, ff, d, 2, st);
  return e;
}

}  // namespace mqa
