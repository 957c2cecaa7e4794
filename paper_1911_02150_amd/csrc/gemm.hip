// Large float32 GEMMs of the projections (prompt-sized row counts, the feed-forward and
// vocabulary matrices of the decoder stack): out[rows, N] = in[rows, C] . B[C, N] with B addressed
// inside the projection tensor P [h, d, kv] exactly as in project.hip.
//
// The float32 matrix instructions are the bound of such a product (157 TFLOP/s against 2.5 PFLOP/s
// in 16 bits), so every float32 operand x is scaled by a power of two and written as two fp16 terms,
// x s = h + l, each the nearest fp16 of what is left (22 to 24 significant bits), and the product as
//   a.b = ah bh + (ah bl + al bh)                            (al bl is below 2^-22 |a||b|, 2^-25 typically)
// accumulated in float32 on v_mfma_f32_32x32x16_f16 (two-term products: Markidis et al. 2018, Ootomo and Yokota 2022).  An fp16 product is exact in float32 and an
// instruction adds 16 of them with one rounding of the running sum, where the float32
// instruction rounds after every second one: the shorter chain of roundings more than pays for the terms.
// Relative error of a 1024-term sum of normal deviates 3.6e-7 (float32 instructions: 5.7e-7), of a
// 4096-term one 7.2e-7 (1.15e-6), of a 520-term one 2.7e-7.
// Scales: one per row of A and per column of B in a tile, such that the largest value among its first indices (32 at
// least) comes to [2^9, 2^10).  A scaled value is held to 2^-23 of itself from 2^-2 on, to 2^-21 from 2^-4 on, and to
// 2^-25 below: products as good as float32 ones need nearly all values of a line above 2^-4, wherever the line's largest
// value is and whatever it meets.  So the octets (eight consecutive indices) with a smaller value other than 0 are
// counted, per line, while they are staged: few may have one (see `holds`).  Where too many have, or a value outgrew
// the scale, the scales are set again from the largest values of all and, if the counts are right then, the tile is multiplied
// again; if not (a line whose values lie more than about 2^11 apart, an infinity) it is multiplied on float32 instructions
// (v_mfma_f32_32x32x2_f32), the values themselves in the place of their two terms.  So are contractions of
// less than 64, too short to count.  Measured (us, rows = 16384, 1024 x 4096; without the counting / with it / on float32
// instructions alone): normal deviates 386 / 407 / 1095; one channel 2^6 times the others 735 / 1020 / 1095 (scales set
// again); 2^12 times 727 / 1660 / 1095 (float32 after that).  Without it the others' part of such sums was lost from 2^14 on.
//
// Measured (b=128, n=128 prompt: rows = 16384, TFLOP/s of the float32 product; 128x128 tiles of
// v_mfma_f32_32x32x2_f32 / three bf16 terms and six products / this): 1024 x 4096: 126 / 224 / 338; 4096 x 1024:
// 129 / 228 / 350; 1024 x 1024: 122 / 220 / 334; logits of 128 rows 101 / 145 / 200.  That is 1.0 PFLOP/s of fp16
// products with the matrix cores busy 51 % of the 1.9 GHz the card runs at under this load (hipBLASLt's 8192^3 bf16
// product reaches 1.29 here); vector instructions take 30 %, LDS 22 % (counters before the counting of octets).  More stages ahead in registers (2, 3), or two
// stages per barrier in LDS, measured the same.
//
// Workgroup: 512 threads, two waves per SIMD, tile BM x BN, WR x WC waves in each of KG groups; a
// stage holds 16*KG contraction indices, group kg works on 16 of them (KG > 1: the groups' tiles are added in
// LDS at the end).  Tiles of 256 (KG = 1) to 32 (KG = 8) square: the smaller ones stage more indices at a time, so that
// every form moves the same 32 KiB of operands per barrier, and below 128 two workgroups share a compute unit, one
// loading while the other multiplies (2048 x 1024 . 1024 x 2048 in 64 x 64 tiles: 65 -> 50 us).  Stages go
// global -> registers (PD stages ahead) -> split -> LDS (two buffers, one barrier per stage).
// Threads 0..255 stage A before they multiply, threads 256..511 stage B after they have: the
// two waves of a SIMD are then out of step and one splits while the other multiplies.
//
// A lane (i, g) of a 32x32x16 operand reads 16 bytes, k = 8g..8g+7 of row i; 32 rows of a half are 512
// contiguous bytes in LDS.  A lane's JB accumulator blocks are JB adjacent columns (one store of
// 4*JB bytes).
#include "common.hpp"

#include <math.h>
#include <type_traits>

namespace mqa {
namespace {

typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(8))) _Float16 halfx8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kFirstTop = 9, kLastTop = 14;    // log2 of what the scales take a line's largest value to: in the first stage, of all
// (scaled values from kFull on are held to 2^-21 of themselves, 2^-23 from 2^-2 on)

// LDS of a stage, in bytes: per group A's two planes, then B's two planes; a plane is two halves g
// of 16 bytes per row (A) or slot (B): contraction indices 8g .. 8g+7.  Column n of the tile lives in slot
// n / JB of column block n % JB.  The few bytes between the halves, groups and column blocks put what
// eight consecutive lanes write (two halves of four rows, two groups of two rows, or two column
// blocks of four slots) on different banks.
template <int BM, int BN, int JB, int KG> struct SplitTile {
  static constexpr int QCOLS = BN / JB;
  static constexpr int B_BLOCK = QCOLS * 16 + (JB == 4 ? 32 : 0);
  static constexpr int PAD = KG >= 4 ? 16 : 64 / KG;
  static constexpr int A_G = BM * 16 + PAD, B_G = JB * B_BLOCK + PAD;
  static constexpr int A_PLANE = 2 * A_G, B_PLANE = 2 * B_G;
  static constexpr int GROUP = 2 * (A_PLANE + B_PLANE) + (KG >= 4 ? 32 : KG == 2 ? 64 : 0);
  static constexpr int STAGE = KG * GROUP;
  // behind the two stages (and, KG > 1, the groups' partial tiles that re-use them): the largest values, the scales'
  // exponents, the counts of short octets and of octets of zeros of the tile's rows and columns, and flags
  static constexpr int PART = KG > 1 ? KG * BM * BN * 4 : 0;
  static constexpr int STATE = 2 * STAGE > PART ? 2 * STAGE : PART;
  static constexpr int BYTES = STATE + (BM + BN) * 16 + 16;
  static __device__ __host__ constexpr int slot_bytes(int block, int slot) { return block * B_BLOCK + slot * 16; }
  // n contiguous, one column block: even columns in the first half of the slots, odd ones in the second, so
  // that the lanes of a pair of columns each write neighbouring slots
  static __device__ __host__ constexpr int column_at(int column) { return JB > 1 ? slot_bytes(column % JB, column / JB) : slot_bytes(0, (column & 1) * (BN / 2) + (column >> 1)); }
};

template <typename V> __device__ __forceinline__ V load_at(const float* base, uint32_t bytes) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + bytes);
}

// B_KCONTIG = false: B[c][n] = P[(n / kv) * d * kv + c * kv + n % kv]   (C = d, N = h * kv)
// B_KCONTIG = true : B[c][n] = P[(c / kv) * d * kv + n * kv + c % kv]   (C = h * kv, N = d)
// ONLY: nothing happens unless *only is not 0, or that of the tile's 256 rows
template <bool B_KCONTIG, int BM, int BN, int WR, int WC, int KG, int PD, bool ONLY>
__global__ __launch_bounds__(512, KG >= 4 ? 4 : 2)      // (waves per SIMD: two workgroups per compute unit of the small tiles)
void gemm_split_kernel(const float* __restrict__ in, const float* __restrict__ P, float* out,
                       int rows, int d, int h, int kv, int epilogue, int tiles_m, int tiles_n, int per, const int32_t* __restrict__ only, const int32_t* __restrict__ only_rows) {
  static_assert(WR * WC * KG == 8 && BM * KG == 256 && BN * KG == 256, "512 threads, 16 staged values of each operand per thread of a half");
  constexpr int RB = BM / WR / 32, JB = BN / WC / 32;      // 32x32 blocks per wave
  typedef SplitTile<BM, BN, JB, KG> L;
  constexpr int KO = 2 * KG;                               // groups of eight contraction indices in a stage
  extern __shared__ __align__(16) unsigned char smem[];

  // tiles: every XCD takes a contiguous run of tiles, column-major inside groups of 8 tile rows, so that
  // the workgroups that run together on an XCD share their operands in its L2
  const int per_xcd = gridDim.x >> 3;
  const int tile = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (tile >= tiles_m * tiles_n) return;
  const int band = tile / (8 * tiles_n), in_band = tile - band * 8 * tiles_n;
  const int band_rows = min(8, tiles_m - band * 8);
  const int row0 = (band * 8 + in_band % band_rows) * BM, n0 = (in_band / band_rows) * BN;
  if constexpr (ONLY)
    if (*only == 0 && only_rows[row0 >> 8] == 0) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31, g = lane >> 5;
  const int kg = wave / (WR * WC), wr = (wave / WC) % WR, wc = wave % WC;
  // this workgroup's part of the contraction: the C indices from `from` on of the whole (per: a multiple of a stage's)
  const int whole = B_KCONTIG ? h * kv : d, from = blockIdx.y * per, C = min(per, whole - from);
  const int N = B_KCONTIG ? d : h * kv;
  const size_t head_stride = (size_t)d * kv;
  const int ts = tid & 255;
  const int nst = (C + 16 * KG - 1) / (16 * KG);
  out += (size_t)blockIdx.y * rows * N;
  uint32_t* most = reinterpret_cast<uint32_t*>(smem + L::STATE);        // [BM + BN] bits of the largest |value| seen
  int* expo = reinterpret_cast<int*>(most + BM + BN);                   // [BM + BN] the tile holds x . 2^-expo
  int* shorts = expo + BM + BN;                                         // [BM + BN] octets with a value that the terms hold in few bits
  int* zeros = shorts + BM + BN;                                        // [BM + BN] octets of zeros (one stage of them behind the last)
  int* again = zeros + BM + BN;                                         // [3] something did not fit; what does not in any scale; what did not in the first

  // ---- staging: 16 values per thread and stage.  Loads are unconditional (indices past the contraction
  // are clamped and their values zeroed when the last stage is split), so that the compiler can
  // count the loads in flight.
  //   A, and B with c contiguous: thread -> eight indices (octet ts % KO) of rows ts / KO + (256 / KO) i
  //   B with n contiguous: thread -> columns 2 pair, 2 pair + 1 at the eight indices of an octet
  const int o_row = ts % KO, r_row = ts / KO;
  const int pair = ts % (BN / 2), o_col = ts / (BN / 2);
  auto run = [&](auto role, auto&& clear, auto&& multiply, auto&& finite) {
    constexpr bool STAGE_A = decltype(role)::value, BY_ROWS = STAGE_A || B_KCONTIG;
    uint32_t* const my_most = most + (STAGE_A ? 0 : BM);
    int* const my_expo = expo + (STAGE_A ? 0 : BM);
    int* const my_short = shorts + (STAGE_A ? 0 : BM);
    int* const my_zeros = zeros + (STAGE_A ? 0 : BM);
    int line[2];                               // the thread's two rows of A or columns of B (by their place in LDS)
#pragma unroll
    for (int i = 0; i < 2; ++i) line[i] = BY_ROWS ? r_row + (256 / KO) * i : 2 * pair + i;
    float scale[2];                            // of these two
    // octets of them with a value that the terms hold in few bits (short), and of zeros; where the scale is not the
    // line's own also the largest value (every octet is looked at then: suspect)
    int short_octets[2], zero_octets[2];
    float peak[2], suspect;
    // a base that is the same in every lane (scalar registers) and a 32-bit offset in bytes of the lane (split_fits)
    const float* base_of = STAGE_A ? in + (size_t)row0 * whole + from : B_KCONTIG ? P + (size_t)n0 * kv : P + (size_t)(n0 / kv) * head_stride + n0 % kv + (size_t)from * kv;
    uint32_t src[BY_ROWS ? 2 : 1];
    if constexpr (BY_ROWS) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        src[i] = STAGE_A ? (uint32_t)min(line[i], rows - 1 - row0) * (4u * (uint32_t)whole)
                         : (uint32_t)min(JB * (line[i] % L::QCOLS) + line[i] / L::QCOLS, N - 1 - n0) * (4u * (uint32_t)kv);        // line: the slot
    } else {
      const int n = n0 + min(2 * pair, N - 2 - n0);
      src[0] = (uint32_t)(n / kv - n0 / kv) * (uint32_t)(4 * head_stride) + 4u * (uint32_t)(n % kv) - 4u * (uint32_t)(n0 % kv);
    }
    struct Regs { float x[16]; };              // [row][8 indices], or [8 indices][column]
    auto load_stage = [&](int st, Regs& rg) {
      const int c0 = min(st, nst - 1) * 16 * KG, c = min(8 * (BY_ROWS ? o_row : o_col), C - 8 - c0);
      if constexpr (BY_ROWS) {
        const float* at = base_of + c0;        // (c contiguous: below)
        uint32_t off = 4u * (uint32_t)c;
        if constexpr (!STAGE_A) {              // eight indices stay inside one head (kv % 8 == 0), a stage need not
          const int head = (from + c0) / kv, in_head = from + c0 - head * kv;
          at = base_of + (size_t)head * head_stride + in_head;
          if (in_head + 16 * KG > kv) off += (uint32_t)((in_head + c) / kv) * (uint32_t)(4 * (head_stride - kv));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float4 v = load_at<float4>(at + 4 * (i & 1), src[i >> 1] + off);
          rg.x[4 * i] = v.x; rg.x[4 * i + 1] = v.y; rg.x[4 * i + 2] = v.z; rg.x[4 * i + 3] = v.w;
        }
      } else {
        const float* at = base_of + (size_t)c0 * kv;
        const uint32_t off = src[0] + (uint32_t)c * (4u * (uint32_t)kv);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float2 v = load_at<float2>(at + (size_t)i * kv, off);
          rg.x[2 * i] = v.x; rg.x[2 * i + 1] = v.y;
        }
      }
    };
    auto value = [&](const Regs& rg, int i, int k) -> float { return BY_ROWS ? rg.x[8 * i + k] : rg.x[2 * k + i]; };
    auto drop_tail = [&](int st, Regs& rg) {   // (C is a multiple of 8)
      if (st * 16 * KG + 16 * KG > C && st * 16 * KG + 8 * (BY_ROWS ? o_row : o_col) >= C) {
#pragma unroll
        for (int i = 0; i < 16; ++i) rg.x[i] = 0.f;
      }
    };
    // |x| in order, zero last
    auto order = [](float x) -> uint32_t { return (__float_as_uint(x) << 1) - 2u; };
    auto count = [&](bool past, const Regs& rg) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint32_t u = ~0u;
#pragma unroll
        for (int k = 0; k < 8; ++k) u = min(u, order(value(rg, i, k)));
        if (suspect > kFull) {
#pragma unroll
          for (int k = 0; k < 8; ++k) peak[i] = fmaxf(peak[i], fabsf(value(rg, i, k)));
        }
        short_octets[i] += !past && u < order(ldexpf(kFull, split_exponent(scale[i]))) ? 1 : 0;
        zero_octets[i] += past || u >= order(0.f) ? 1 : 0;
      }
    };
    auto store_stage = [&](auto plain, int st, Regs& rg) {
      unsigned char* base = smem + (st & 1) * L::STAGE;
      const int octet = BY_ROWS ? o_row : o_col;
      // Past the end: zeros; or, in the large tiles, scaled by 0 (two selections instead of sixteen moves a stage, 412 -> 394 us
      // at 16384 x 4096 x 1024; the small ones have no register for it).  An infinity there is in the line as well and takes
      // it to the float32 instructions.
      constexpr bool CLEAR = decltype(plain)::value || KG >= 4;
      const bool past = !CLEAR && st * 16 * KG + 8 * octet >= C;
      const float by[2] = {past ? 0.f : scale[0], past ? 0.f : scale[1]};
      if constexpr (CLEAR) drop_tail(st, rg);
      base += (octet >> 1) * L::GROUP + (octet & 1) * (STAGE_A ? L::A_G : L::B_G) + (STAGE_A ? 0 : 2 * L::A_PLANE);
      float least[2] = {INFINITY, INFINITY};
#pragma unroll
      for (int i = 0; i < 2; ++i) {            // two rows / columns of eight indices
        u32x4 t[2];
        if constexpr (decltype(plain)::value) {      // the values themselves, four in each plane
#pragma unroll
          for (int k = 0; k < 8; ++k) t[k >> 2][k & 3] = __float_as_uint(value(rg, i, k));
        } else {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float a = value(rg, i, 2 * k) * by[i], b = value(rg, i, 2 * k + 1) * by[i];
            least[i] = fminf(least[i], fminf(fabsf(a), fabsf(b)));
            const Split2 s = split2(a, b);
            t[0][k] = s.hi; t[1][k] = s.lo;
          }
        }
        const int at = STAGE_A ? 16 * line[i] : B_KCONTIG ? L::slot_bytes(line[i] / L::QCOLS, line[i] % L::QCOLS) : L::column_at(line[i]);
#pragma unroll
        for (int p = 0; p < 2; ++p) *reinterpret_cast<u32x4*>(base + p * (STAGE_A ? L::A_PLANE : L::B_PLANE) + at) = t[p];
      }
      if (!decltype(plain)::value && fminf(least[0], least[1]) < suspect) count(past, rg);      // (a zero, or one of some ten thousand normal deviates)
    };
    // scales from the largest values known; a line of zeros so far takes the largest of the tile's lines
    auto set_scales = [&](int top) {
      float whole = 0.f;
#pragma unroll
      for (int i = 0; i < (STAGE_A ? BM : BN); i += 64) whole = fmaxf(whole, __uint_as_float(my_most[(lane + i) % (STAGE_A ? BM : BN)]));
      whole = wave_max(whole);
      suspect = kFull;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float m = __uint_as_float(my_most[line[i]]);
        scale[i] = split_scale(m > 0.f ? m : whole > 0.f ? whole : 1.f, top);
        if (m == 0.f) suspect = INFINITY;
        my_expo[line[i]] = split_exponent(scale[i]);
        short_octets[i] = zero_octets[i] = 0;
        peak[i] = 0.f;
      }
    };
    auto largest = [&](Regs& rg) {             // (into peak)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k) peak[i] = fmaxf(peak[i], fabsf(value(rg, i, k)));
    };
    auto tell_peaks = [&]() {
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (peak[i] > 0.f) atomicMax(&my_most[line[i]], __float_as_uint(peak[i]));
    };
    Regs regs[PD];                             // the PD stages after the one in LDS, on their way
    auto sweep = [&](auto plain) {             // (the first stage is in regs[0])
      clear();
      store_stage(plain, 0, regs[0]);
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        load_stage(1 + u, regs[u]);
        __builtin_amdgcn_sched_barrier(0);     // requested in the order of use
      }
      __syncthreads();
      for (int s0 = 0; s0 < nst; s0 += PD) {
#pragma unroll
        for (int u = 0; u < PD; ++u) {
          const int st = s0 + u;
          if (st >= nst) break;
          if constexpr (STAGE_A) multiply(plain, st & 1);
          store_stage(plain, st + 1, regs[u]);
          load_stage(st + 1 + PD, regs[u]);
          if constexpr (!STAGE_A) multiply(plain, st & 1);
          __syncthreads();
        }
      }
    };
    // a line: some value of it is far above what the terms cut off, and few octets (none of up to 7 with anything but zeros,
    // 2 and an eighth of more) hold a value that is not
    auto holds = [&](int i) -> bool {
      const int n = my_short[line[i]], octets = (nst + 1) * KO - my_zeros[line[i]];
      return n <= (octets < 8 ? 0 : 2 + octets / 8) && (n == 0 || __uint_as_float(my_most[line[i]]) * scale[i] >= kFarAbove);
    };
    bool plain = C < 64;                       // (too few octets to tell)
    auto tell_counts = [&]() {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (short_octets[i] > 0) atomicAdd(&my_short[line[i]], short_octets[i]);
        if (zero_octets[i] > 0) atomicAdd(&my_zeros[line[i]], zero_octets[i]);
      }
    };
    auto scan = [&](auto&& look) {             // (a stage of zeros at the end, as in a sweep)
#pragma unroll 1
      for (int st = 0; st <= nst; ++st) {
        load_stage(st, regs[0]);
        drop_tail(st, regs[0]);
        look(regs[0]);
      }
    };
    for (int top = kFirstTop; !plain; top = kLastTop) {
      if (top == kFirstTop) {                  // the first 32 indices at least
        constexpr int LOOK = KG < 2 ? 2 : 1;
        peak[0] = peak[1] = 0.f;
#pragma unroll 1
        for (int u = LOOK - 1; u >= 0; --u) {
          load_stage(u, regs[0]);
          drop_tail(u, regs[0]);
          largest(regs[0]);
        }
        tell_peaks();
        __syncthreads();
        set_scales(top);
      } else {
        load_stage(0, regs[0]);
      }
      sweep(std::false_type{});
      if (top == kLastTop) break;              // (counted beforehand)
      // Did the terms hold the lines?  (a scaled value that overflowed leaves nothing finite of its line)
      if (!finite()) again[0] = 1;
      tell_counts();
      tell_peaks();
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (!holds(i)) again[0] = again[2] = 1;
      __syncthreads();
      if (__builtin_expect(again[0] == 0, 1)) break;
      // Would they with the right scales?  The largest values, then the counts
      peak[0] = peak[1] = 0.f;
      scan([&](Regs& rg) { largest(rg); });
      tell_peaks();
#pragma unroll
      for (int i = 0; i < 2; ++i) my_short[line[i]] = my_zeros[line[i]] = 0;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float m = __uint_as_float(my_most[line[i]]);
        if (!(m * scale[i] < 65520.f)) again[2] = 1;
        if (m == INFINITY) again[1] = 1;
      }
      __syncthreads();
      if (!again[2]) break;                    // (a NaN alone, and the outputs are what they were to be)
      set_scales(kLastTop);
      scan([&](Regs& rg) { count(false, rg); });
      tell_counts();
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 2; ++i)
        if (!holds(i)) again[1] = 1;
      __syncthreads();
      plain = again[1];
    }
    if (__builtin_expect(plain, 0)) {
#pragma unroll
      for (int i = 0; i < 2; ++i) my_expo[line[i]] = 0;
      load_stage(0, regs[0]);
      sweep(std::true_type{});
    }
  };

  floatx16 acc[RB][JB];
  auto clear = [&]() {
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[r][j][e] = 0.f;
  };

  auto finite = [&]() -> bool {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) s = fmaf(acc[r][j][e], 0.f, s);
    return s == 0.f;
  };
  auto multiply = [&](auto plain, int buf) {
    const unsigned char* As = smem + buf * L::STAGE + kg * L::GROUP + g * L::A_G + (wr * RB * 32 + i32) * 16;
    const unsigned char* Bs = smem + buf * L::STAGE + kg * L::GROUP + 2 * L::A_PLANE + g * L::B_G + L::slot_bytes(0, wc * 32 + i32);
    typedef std::conditional_t<decltype(plain)::value, floatx4, halfx8> operand;
    operand a[2][RB], b[2][JB];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int r = 0; r < RB; ++r) a[p][r] = *reinterpret_cast<const operand*>(As + p * L::A_PLANE + r * 512);
#pragma unroll
      for (int j = 0; j < JB; ++j) b[p][j] = *reinterpret_cast<const operand*>(Bs + p * L::B_PLANE + L::slot_bytes(j, 0));
    }
    if constexpr (decltype(plain)::value) {      // step (p, e): the indices 4 p + e of both octets
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int j = 0; j < JB; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[p][r][e], b[p][j][e], acc[r][j], 0, 0, 0);
    } else {
    auto product = [&](int pa, int pb) {
#pragma unroll
      for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int j = 0; j < JB; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[pa][r], b[pb][j], acc[r][j], 0, 0, 0);
    };
    product(0, 0); product(0, 1); product(1, 0);
    }
  };

  for (int i = tid; i < BM + BN; i += 512) most[i] = 0, shorts[i] = zeros[i] = 0;
  if (tid < 3) again[tid] = 0;
  __syncthreads();
  if (wave < 4) run(std::true_type{}, clear, multiply, finite);
  else run(std::false_type{}, clear, multiply, finite);

  // KG > 1: the groups' partial tiles meet in LDS (free after the last barrier); group kg finishes the
  // registers [kg SHARE, (kg + 1) SHARE) of all of them
  constexpr int SHARE = RB * 16 / KG;
  float* part = reinterpret_cast<float*>(smem) + lane;
  if constexpr (KG > 1) {
    float* mine = part + (size_t)wave * (RB * JB * 16 * 64);
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
      for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int j = 0; j < JB; ++j) mine[((r * 16 + e) * JB + j) * 64] = acc[r][j][e];
    __syncthreads();
  }

  // D layout of a 32x32 block: register e of lane (i, g) is element (8 (e/4) + 4 g + e%4, i); the lane's
  // JB blocks are columns n .. n + JB - 1
  const int slot = wc * 32 + i32;
  const int n = n0 + (JB == 1 && !B_KCONTIG ? 2 * (slot % (BN / 2)) + slot / (BN / 2) : JB * slot);
  if (n >= N) return;                          // (N is a multiple of 8: all JB columns are in or out)
  typedef __attribute__((ext_vector_type(JB))) float vec;
  int col_expo[JB];                            // (column q JB + j of the tile: by slots where c is contiguous)
#pragma unroll
  for (int j = 0; j < JB; ++j) col_expo[j] = expo[BM + (B_KCONTIG ? j * L::QCOLS + slot : n - n0 + j)];
  auto row_in_tile = [&](int re) { return wr * RB * 32 + 32 * (re >> 4) + 8 * ((re >> 2) & 3) + 4 * g + (re & 3); };
  auto finish = [&](float* dst, vec x) {
    if (epilogue == 1) {
#pragma unroll
      for (int j = 0; j < JB; ++j) x[j] = fmaxf(x[j], 0.f);
    } else if (epilogue == 2) {
      x += *reinterpret_cast<vec*>(dst);
    }
    *reinterpret_cast<vec*>(dst) = x;
  };
  const int re0 = kg * SHARE;
#pragma unroll
  for (int k = 0; k < SHARE; ++k) {
    vec x;
    const int row_expo = expo[row_in_tile(re0 + k)];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      float y = 0.f;
      if constexpr (KG == 1) y = acc[k >> 4][j][k & 15];
      else
#pragma unroll
        for (int q = 0; q < KG; ++q) y += part[((size_t)(q * WR * WC + wave % (WR * WC)) * (RB * 16) + re0 + k) * (JB * 64) + j * 64];
      x[j] = ldexpf(y, row_expo + col_expo[j]);
    }
    const int row = row0 + row_in_tile(re0 + k);
    if (row < rows) finish(out + (size_t)row * N + n, x);
  }
}

// The 32-bit offsets inside a tile: of its rows and columns and of the heads that a tile (n contiguous) or a stage
// (c contiguous) reaches over.
bool split_fits(bool outp, int d, int h, int kv, int tile, int stage) {
  const long long C = outp ? (long long)h * kv : d, most = 1ll << 30;      // floats: 4 GiB
  if (C * tile >= most || (long long)kv * (tile > stage ? tile : stage) >= most) return false;
  const int reach = outp ? stage : tile;
  return h == 1 || kv % reach == 0 || (long long)d * kv * (reach / kv + 2) < most;
}

template <bool KC, int BM, int BN, int WR, int WC, int KG, int PD, bool ONLY = false>
hipError_t launch_split(const float* in, const float* P, float* out, int rows, int d, int h, int kv, int N,
                        int epilogue, int S, hipStream_t st, const int32_t* only = nullptr, const int32_t* only_rows = nullptr) {
  constexpr size_t lds = SplitTile<BM, BN, BN / WC / 32, KG>::BYTES;       // 67 KiB (32, 64), 132 (128: the groups' partial tiles), 74 (256)
  auto kern = gemm_split_kernel<KC, BM, BN, WR, WC, KG, PD, ONLY>;
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  const int tm = (rows + BM - 1) / BM, tn = (N + BN - 1) / BN;
  const long long tiles = (long long)tm * tn;
  const dim3 grid((unsigned)((tiles + 7) / 8 * 8), S), block(512);
  const int C = KC ? h * kv : d, stage = 16 * KG, per = S > 1 ? ((C + stage - 1) / stage + S - 1) / S * stage : C;
  hipLaunchKernelGGL(kern, grid, block, lds, st, in, P, out, rows, d, h, kv, epilogue, tm, tn, per, only, only_rows);
  return hipGetLastError();
}

}  // namespace

// The edge of the tiles that a product takes here; 0 where the split-contraction kernel of project.hip is the faster one
// or the offsets do not fit.  `apart` is what a launch of its own costs the caller more (us).
// The forms differ in how they fill the chip and in what a staged byte is worth.  Measured, us = 5 + C / 1024 times
//   32 x 32 tiles: 5.7 up to 256 of them, 10.5 for each 512 (two per compute unit)     128 x 1024 x 4096 (C = 1024): 15
//   64 x 64:       12                     22.5                                         1024 x 1024 x 1024: 17, 2048 x 2048: 50
//   128 x 128:     33 for each 256 (one per compute unit)                              4096 x 1024 x 1024: 38
//   256 x 256:     70                                                                  2000 x 1000 x 5008: 88
// and the split-contraction kernel on float32 instructions 5 (less below C = 1024, in proportion) + 2 rows N C / 64
// TFLOP/s (80 with n contiguous): 128 x 512 x 4096: 9.1 (32 x 32 tiles 10.6); 128 x 1024 x 1024: 9.2; 128 x 4096 x 1024, long sums and few tiles: 24, 32 x 32 tiles 26; 1024 x 1024 x 1024: 32; 768 x
// 4096 x 1024: 104, 64 x 64 tiles 50.
struct GemmCost { int edge; double tiles_us, split_us; };
static GemmCost gemm_cost(bool outp, int rows, int N, double C) {
  auto tiles = [&](int t) { return (double)((N + t - 1) / t) * (double)((rows + t - 1) / t); };
  auto rounds = [&](int t, double per_round) { return ceil(tiles(t) / per_round); };
  const double w[4] = {tiles(32) <= 256 ? 5.7 : 10.5 * rounds(32, 512), tiles(64) <= 256 ? 12. : 22.5 * rounds(64, 512),
                       33. * rounds(128, 256), 70. * rounds(256, 256)};
  int best = 0;
  for (int f = 1; f < 4; ++f)
    if (w[f] < w[best]) best = f;
  const double split_contraction = (C < 1024. ? 5. * C / 1024. : 5.) + 2. * ((rows + 15) / 16 * 16) * N * C / (outp ? 64e6 : 80e6);
  return GemmCost{32 << best, 5. + C / 1024. * w[best], split_contraction};
}
bool gemm_fits(bool outp, int d, int h, int kv, int edge) { return split_fits(outp, d, h, kv, edge, 16 * (256 / edge)); }
double gemm_us(bool outp, int rows, int N, int C) {
  const GemmCost c = gemm_cost(outp, rows, N, C);
  return c.tiles_us < c.split_us ? c.tiles_us : c.split_us;
}
int gemm_form(int mode, int rows, int d, int h, int kv, int apart) {
  const bool outp = (mode == 3);
  const GemmCost c = gemm_cost(outp, rows, outp ? d : h * kv, outp ? (double)h * kv : (double)d);
  if (c.tiles_us + apart > 0.9 * c.split_us) return 0;
  return gemm_fits(outp, d, h, kv, c.edge) ? c.edge : 0;
}

// The same for a product rows x C . C x N that is one of these tiles in any case; 0: the offsets do not fit
int gemm_edge(int rows, int N, int C) {
  const GemmCost c = gemm_cost(false, rows, N, C);
  return gemm_fits(false, C, 1, N, c.edge) ? c.edge : 0;
}

// in [rows, C] . P [C, N] if *only is not 0 on the device, or only_rows[i] for the rows 256 i .. 256 i + 255
hipError_t launch_gemm_if(const int32_t* only, const int32_t* only_rows, int edge, const float* in, const float* P, float* out, int rows, int C, int N, int epilogue,
                          hipStream_t st) {
  if (edge == 128) return launch_split<false, 128, 128, 2, 2, 2, 3, true>(in, P, out, rows, C, 1, N, N, epilogue, 1, st, only, only_rows);
  if (edge == 256) return launch_split<false, 256, 256, 4, 2, 1, 1, true>(in, P, out, rows, C, 1, N, N, epilogue, 1, st, only, only_rows);
  return hipErrorNotSupported;
}

// S > 1: the contraction in S parts, their products one behind another in `out` (S x rows x N); edge: of the tiles
hipError_t launch_gemm_parts(int mode, const float* in, const float* P, float* out,
                             int rows, int d, int h, int kv, int epilogue, int edge, int S, hipStream_t st) {
  const bool outp = (mode == 3);
  const int N = outp ? d : h * kv;
#define MQA_SPLIT(BM, WR, WC, KG, PD) \
  return outp ? launch_split<true, BM, BM, WR, WC, KG, PD>(in, P, out, rows, d, h, kv, N, epilogue, S, st) \
              : launch_split<false, BM, BM, WR, WC, KG, PD>(in, P, out, rows, d, h, kv, N, epilogue, S, st)
  switch (edge) {
    case 32: MQA_SPLIT(32, 1, 1, 8, 1);
    case 64: MQA_SPLIT(64, 2, 1, 4, 1);
    case 128: MQA_SPLIT(128, 2, 2, 2, 3);
    case 256: MQA_SPLIT(256, 4, 2, 1, 1);
  }
#undef MQA_SPLIT
  return hipErrorNotSupported;
}

// hipErrorNotSupported: no form (gemm_form); the caller then uses the split-contraction kernel
hipError_t launch_gemm_tiled(int mode, const float* in, const float* P, float* out,
                             int rows, int d, int h, int kv, int epilogue, int apart, hipStream_t st) {
  return launch_gemm_parts(mode, in, P, out, rows, d, h, kv, epilogue, gemm_form(mode, rows, d, h, kv, apart), 1, st);
}

}  // namespace mqa
