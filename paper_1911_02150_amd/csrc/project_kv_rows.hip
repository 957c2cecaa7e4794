// New K / V rows of many positions at once (a memory, a prompt) into a bf16 cache, for callers that hand over a workspace:
// the numbers of project_kv.hip (fixed point in four base-256 digits, the ten largest digit products exact in integers, a
// bound on the rest, float64 for what the bound leaves open; see there for the bounds), with the weights prepared once
// per call instead of once per tile of rows.
//   prepare_kernel   every column of P_k and P_v: its largest magnitude, its digits in the order in which a wave's matrix
//                    operands want them, what it adds to the bounds, and the column itself with its elements side by side
//   kv_rows_kernel   tiles of 64 rows x 128 columns of K and V side by side
// In project_kv.hip's tiles of 128 x 128 half of the values that are converted and scanned are weights that every other
// tile of rows converts again, and an open element costs a cache line per weight.  Here a wave loads the weights' digits
// straight into its operand registers (1 KiB at a time, from L2; no two waves of a workgroup need the same), only the
// rows go through LDS (64 indices to a barrier), and a workgroup is four waves, so that two share a compute unit and one
// multiplies while the other looks for its rows' largest magnitudes or rounds its sums.
// Measured (32768 rows, d = 1024, 256 columns): 110.7 us with the preparation's 7 (project_kv.hip 180, the float64 kernel 410).
// Of a tile's 60 us, two side by side: first pass 8, products 38, sums and rounding 8, open elements 4.  Bound by no single
// unit (a third of the cycles each in the matrix cores and in vector instructions): the card holds 1.6 to 2.0 GHz in the products (22 us of them at that
// clock without the conversions).  v_mfma_i32_16x16x64_i8 draws less of it than 32x32x32, us before / so: 113.5 /
// 110.7, 16384 rows 66.9 / 62.4, 12800 rows of 2048 indices 110.5 / 103.5, 8192 rows x 2048 columns 221 / 205.  Without effect: tiles of 64 x 256 with eight waves (half the conversions, nothing beside them: 120), raised
// priority of every second workgroup, weights two steps ahead or from L1, sums in 64-bit integers.
#include "kv_fixed.hpp"

namespace mqa {
namespace {

using namespace kv_fixed;

constexpr int kRows = 64, kColumns = 128;      // of a tile
constexpr int kGroups = 512;                   // two workgroups per compute unit

// Open elements of a tile (of 8192, those that need no summing aside) from which its waves sum all of it in float64.  One element costs
// half a wave some 4 us of latency (more from 1024 indices on), all of them 0.26 us for each index.  us, with one channel of the rows 2^6 / 2^7 /
// 2^8 / 2^9 times the others and its weights as much smaller, by this limit against all in float64: 32768 rows, d = 1024: 160 / 180 / 216 / 400
// against 406; 19200 rows, d = 200: 52 / 65 / 81 / 81 against 82; one row with an infinity (128 open) in every 1024: 169 against 401 and 81 against 82.
__device__ __forceinline__ int most_open(int C) { return min(3 * C / 8, 512); }

// Workspace: digits [column block of 32][step of 32 indices][digit][lane][16 bytes], columns [N][C] floats, lines [columns
// padded] (of 16 bytes).
struct KvPrepared {
  int C, steps, N, padded;             // steps: of 32 indices, an even number; padded: columns, a multiple of 128
  __host__ __device__ size_t digits() const { return 0; }
  __host__ __device__ size_t columns() const { return (size_t)padded * steps * 128; }
  __host__ __device__ size_t lines() const { return columns() + (((size_t)N * C * 4 + 15) & ~(size_t)15); }
  __host__ __device__ size_t bytes() const { return lines() + (size_t)padded * 16; }
};
KvPrepared prepared_of(int d, int h_kv, int k, int v) {
  KvPrepared w;
  w.C = d;
  w.steps = (d + 63) / 64 * 2;
  w.N = h_kv * (k + v);
  w.padded = (w.N + kColumns - 1) / kColumns * kColumns;
  return w;
}

struct KvRowsParams {
  const float* x;                // [rows, C]
  const float* P[2];             // [h_kv, C, kv[which]]
  uint16_t* dst[2];              // caches [seq, h_kv, cap, kv[which]]
  const int32_t* lens_in;        // append: rows already there; else valid rows per sequence, or null
  int32_t* lens_out;
  unsigned char* ws;
  KvPrepared w;
  int rows, h_kv, cap, n;        // row r is row r % n of sequence r / n
  int kv[2];
  int append, tiles_m, tiles_n;
};

// Four columns (k and v are multiples of 16: of one head) by 256 threads; a thread takes sixteen indices of a column at a
// time.  Bound by latency (64 workgroups for k = v = 128).
__global__ __launch_bounds__(256)
void prepare_kernel(KvRowsParams p) {
  __shared__ uint32_t most[4];
  __shared__ int norm[4][4];
  const KvPrepared w = p.w;
  const int tid = threadIdx.x, j = tid & 3, C = w.C;
  const int n = blockIdx.x * 4 + j;
  if (tid < 4) most[tid] = 0;
  if (tid < 16) norm[tid >> 2][tid & 3] = 0;
  const bool real = n < w.N;                   // (else padding: digits of zero)
  const int which = n >= p.h_kv * p.kv[0] ? 1 : 0, kv = p.kv[which];
  const int in_part = which ? n - p.h_kv * p.kv[0] : n;
  const float* src = real ? p.P[which] + (size_t)(in_part / kv) * C * kv + in_part % kv : p.P[0];
  const size_t stride = real ? kv : 0;
  float x[16];
  auto load = [&](int c0) {                    // (C is a multiple of 8)
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = src[(size_t)min(c0 + i, C - 1) * stride];
  };
  uint32_t m = 0;
  const int groups = 2 * w.steps;              // of sixteen indices
  for (int s = tid >> 2; s < groups; s += 64) {
    load(16 * s);                              // (indices past the end repeat the last)
#pragma unroll
    for (int i = 0; i < 16; ++i) m = max(m, __float_as_uint(x[i]) & 0x7fffffffu);
  }
  if (!real) m = 0;
  __syncthreads();
  atomicMax(&most[j], m);
  __syncthreads();
  const uint32_t top = most[j];
  const float scale = real ? __uint_as_float((uint32_t)(fixed_exponent(top) + 127) << 23) : 0.f;
  int sq[4] = {0, 0, 0, 0};
  float* column = reinterpret_cast<float*>(p.ws + w.columns()) + (size_t)n * C;
  for (int s = tid >> 2; s < groups; s += 64) {
    if (groups > 64) load(16 * s);             // (else still in the registers)
    int4v d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float by = 16 * s + 4 * q < C ? scale : 0.f;
      const Digits4 t = digits_of(x[4 * q] * by, x[4 * q + 1] * by, x[4 * q + 2] * by, x[4 * q + 3] * by);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        d[e][q] = t.word[e];
        sq[e] = __builtin_amdgcn_sdot4(t.word[e], t.word[e], sq[e], false);
      }
      if (real && 16 * s + 4 * q < C) *reinterpret_cast<float4*>(column + 16 * s + 4 * q) = make_float4(x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]);
    }
    // lane (i, g) of a step: column i of the block, indices 16 g ..
    unsigned char* at = p.ws + w.digits() + ((size_t)(n >> 5) * w.steps + (s >> 1)) * 4096 + ((s & 1) * 32 + (n & 31)) * 16;
#pragma unroll
    for (int e = 0; e < 4; ++e) *reinterpret_cast<int4v*>(at + e * 1024) = d[e];
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) atomicAdd(&norm[j][e], sq[e]);
  __syncthreads();
  if (tid < 4) *reinterpret_cast<Line*>(p.ws + w.lines() + (size_t)n * 16) = line_of(norm[j], top, C);
}

// LDS, in bytes.  A digit of the rows is two halves of sixteen indices; what eight lanes write (the halves and steps of two
// rows) lies on different banks.
struct KvTile {
  static constexpr int HALF = kRows * 16 + 64, DIGIT = 2 * HALF, STEP = 4 * DIGIT + 128;
  static constexpr int STAGE = 2 * STEP;                // 64 indices
  static constexpr int SUM_ROW = 4 * kColumns + 16, SUMS = kRows * SUM_ROW;      // a tile's sums, its finished rows and a list of elements
  static constexpr int ROW = 2 * kColumns + 16, OUT = kRows * ROW, LIST = 2 * kRows * kColumns;
  static constexpr int BODY = 2 * STAGE > SUMS + OUT + LIST ? 2 * STAGE : SUMS + OUT + LIST;
  static constexpr int BYTES = BODY + (kRows + kColumns) * 16 + 16;      // and the tile's lines (16 bytes each), and a count
};

__global__ __launch_bounds__(256, 2)
void kv_rows_kernel(KvRowsParams p) {
  typedef KvTile T;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char* const lines = smem + T::BODY;           // rows, then columns
  auto line_at = [&](int i) -> Line& { return *reinterpret_cast<Line*>(lines + 16 * i); };
  int* count = reinterpret_cast<int*>(lines + (kRows + kColumns) * 16);

  const KvPrepared w = p.w;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, i32 = lane & 31, g = lane >> 4;
  const int C = w.C, rows = p.rows;
  const int nst = w.steps / 2;

  // staging: a thread holds sixteen indices (two octets) of a row
  const int line = tid >> 2, part = tid & 3;
  struct Regs { float x[16]; };
  auto load_stage = [&](const float* src, int st, Regs& rg) {          // (indices past the end are clamped, and dropped before use)
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const float* at = src + min(64 * st + 16 * part + 8 * o, C - 8);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float4 v = *reinterpret_cast<const float4*>(at + 4 * i);
        rg.x[8 * o + 4 * i] = v.x; rg.x[8 * o + 4 * i + 1] = v.y; rg.x[8 * o + 4 * i + 2] = v.z; rg.x[8 * o + 4 * i + 3] = v.w;
      }
    }
  };
  auto largest = [&](uint32_t m, const Regs& rg) {
#pragma unroll
    for (int i = 0; i < 16; ++i) m = max(m, __float_as_uint(rg.x[i]) & 0x7fffffffu);
    return m;
  };
  auto of_row = [&](auto v, auto&& join) {
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) v = join(v, __shfl_xor(v, o));
    return v;
  };

  // column tiles of a row tile are neighbours on one XCD
  const int tiles = p.tiles_m * p.tiles_n, per_xcd = (tiles + 7) >> 3;
  auto tile_at = [&](int turn) -> int {        // the turn'th tile of this workgroup, or -1
    const int at = blockIdx.x + turn * gridDim.x;
    const int t = (at & 7) * per_xcd + (at >> 3);
    return at < 8 * per_xcd && t < tiles ? t : -1;
  };
  auto row_of = [&](int tile) { return p.x + (size_t)min(tile / p.tiles_n * kRows + line, rows - 1) * C; };

  for (int turn = 0;; ++turn) {
    const int tile = tile_at(turn);
    if (tile < 0) break;
    const int tile_m = tile / p.tiles_n, tile_n = tile - tile_m * p.tiles_n;
    const int row0 = tile_m * kRows, n0 = tile_n * kColumns;
    const float* src = row_of(tile);
    uint32_t row_most = 0;                     // of this thread's row
    {
      constexpr int AHEAD = 4;
      Regs rg[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) load_stage(src, u, rg[u]);
      for (int s0 = 0; s0 < nst; s0 += AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
          row_most = largest(row_most, rg[u]);
          load_stage(src, s0 + u + AHEAD, rg[u]);
        }
    }
    row_most = of_row(row_most, [](uint32_t a, uint32_t b) { return max(a, b); });
    if (tid == 0) *count = 0;
    if (tid < kColumns) *reinterpret_cast<int4v*>(lines + (kRows + tid) * 16) = *reinterpret_cast<const int4v*>(p.ws + w.lines() + (size_t)(n0 + tid) * 16);
    const float scale = __uint_as_float((uint32_t)(fixed_exponent(row_most) + 127) << 23);

    int sq[4] = {0, 0, 0, 0};
    auto store_stage = [&](int st, const Regs& rg) {
      unsigned char* dst = smem + (st & 1) * T::STAGE + (part >> 1) * T::STEP + (part & 1) * T::HALF + line * 16;
      int4v d[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float by = 64 * st + 16 * part + 8 * (k >> 1) < C ? scale : 0.f;       // (C is a multiple of 8)
        const float* x = rg.x + 4 * k;
        const Digits4 t = digits_of(x[0] * by, x[1] * by, x[2] * by, x[3] * by);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          d[q][k] = t.word[q];
          sq[q] = __builtin_amdgcn_sdot4(t.word[q], t.word[q], sq[q], false);
        }
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<int4v*>(dst + q * T::DIGIT) = d[q];
    };

    int4v acc[4][4][2];                        // sums of the digit products with i + j = 3 + t, per row block and column block of 16
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[t][r][c] = int4v{0, 0, 0, 0};
    const __amdgpu_buffer_rsrc_t weights = __builtin_amdgcn_make_buffer_rsrc(
        p.ws + w.digits() + (size_t)((n0 >> 5) + wave) * w.steps * 4096, 0, (uint32_t)w.steps * 4096u, 0x00020000u);
    // lane (i16, g) of a stage: column i16 of a block, indices 16 g ..
    const uint32_t in_stage = (uint32_t)((g >> 1) * 4096 + ((g & 1) * 32 + i16) * 16);
    auto weights_of = [&](int st, int q, int c) {
      return __builtin_bit_cast(int4v, __builtin_amdgcn_raw_buffer_load_b128(weights, in_stage + (uint32_t)c * 256u, (uint32_t)min(st, nst - 1) * 8192u + (uint32_t)q * 1024u, 0));
    };
    int4v b[4][2];
    // A stage.  The registers of a weight digit take the next stage as soon as its last product is issued (left to itself the
    // compiler moves these loads to the end).
    auto multiply = [&](int st) {
      const unsigned char* As = smem + (st & 1) * T::STAGE + (g >> 1) * T::STEP + (g & 1) * T::HALF + i16 * 16;
      int4v a[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) a[r] = *reinterpret_cast<const int4v*>(As + 3 * T::DIGIT + r * 256);
#pragma unroll
      for (int i = 3; i >= 0; --i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
          for (int e = 3 - i; e <= 3; ++e)
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[i + e - 3][r][c] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[r], b[e][c], acc[i + e - 3][r][c], 0, 0, 0);
          if (i > 0) a[r] = *reinterpret_cast<const int4v*>(As + (i - 1) * T::DIGIT + r * 256);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) b[3 - i][c] = weights_of(st + 1, 3 - i, c);
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    Regs regs;
    load_stage(src, 0, regs);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int c = 0; c < 2; ++c) b[q][c] = weights_of(0, q, c);
    store_stage(0, regs);
    load_stage(src, 1, regs);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
      store_stage(st + 1, regs);               // (past the end: digits of zero, into a buffer nobody reads)
      load_stage(src, st + 2, regs);
      multiply(st);
      __syncthreads();
    }
    {
      auto add = [](int a, int b) { return a + b; };
      int sum[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) sum[q] = of_row(sq[q], add);
      if (part == 0) line_at(line) = line_of(sum, row_most, C);
    }
    // ---- sums; then, a row's eight columns per thread at a time, bounds and rounding: the tile stays in LDS, its open
    // elements go to a list
    unsigned char* const sums = smem;
    unsigned char* const out = smem + T::SUMS;
    uint16_t* const list = reinterpret_cast<uint16_t*>(smem + T::SUMS + T::OUT);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          *reinterpret_cast<float*>(sums + (r * 16 + 4 * g + e) * T::SUM_ROW + 4 * (wave * 32 + c * 16 + i16)) =
              digit_sum(acc[0][r][c][e], acc[1][r][c][e], acc[2][r][c][e], acc[3][r][c][e]);
    __syncthreads();
    const int c8 = tid % (kColumns / 8) * 8, nn = n0 + c8;      // eight columns of one head (N is a multiple of 16)
    const int which = nn >= p.h_kv * p.kv[0] ? 1 : 0, kv = p.kv[which];
    const int in_part = which ? nn - p.h_kv * p.kv[0] : nn;
    uint16_t* const to = p.dst[which] + (size_t)(in_part / kv) * p.cap * kv + in_part % kv;
    auto place = [&](int r) -> uint16_t* {                 // null: nothing is written
      const int row = row0 + r;
      if (row >= rows || nn >= w.N) return nullptr;
      const int seq = row / p.n;
      int at = row - seq * p.n;
      if (p.append) {
        const int L = p.lens_in[seq];
        if (L < 0 || L > p.cap - p.n) return nullptr;      // (n <= cap; a sum could wrap)
        at += L;
      }
      return to + ((size_t)seq * p.h_kv * p.cap + at) * kv;
    };
    constexpr int PASS = 256 / (kColumns / 8);             // rows at a time
    uint32_t pending = 0;                      // of this thread's parts of rows: those with an open element
    Line cols[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cols[j] = line_at(kRows + c8 + j);
#pragma unroll
    for (int u = 0; u < kRows / PASS; ++u) {
      const int r = tid / (kColumns / 8) + u * PASS;
      const float4 mid[2] = {*reinterpret_cast<const float4*>(sums + r * T::SUM_ROW + 4 * c8), *reinterpret_cast<const float4*>(sums + r * T::SUM_ROW + 4 * c8 + 16)};
      const Line mine = line_at(r);
      uint32_t v[8], open = 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        bool o;
        v[j] = rounded_sum((&mid[j >> 2].x)[j & 3], mine, cols[j], &o);
        open |= o ? 1u << j : 0u;
      }
      const uint4 packed = make_uint4(v[0] | v[1] << 16, v[2] | v[3] << 16, v[4] | v[5] << 16, v[6] | v[7] << 16);
      uint16_t* const at = place(r);
      if (open && at) {                        // (written once they are known)
        *reinterpret_cast<uint4*>(out + r * T::ROW + 2 * c8) = packed;
        pending |= 1u << u;
        for (; open; open &= open - 1) list[atomicAdd(count, 1)] = (uint16_t)(r * kColumns + c8 + __builtin_ctz(open));
      } else if (at) {
        *reinterpret_cast<uint4*>(at) = packed;
      }
    }
    __syncthreads();
    const int left = *count;
    const float* columns = reinterpret_cast<const float*>(p.ws + w.columns());
    auto nan_at = [&](int at) { return is_nan(line_at(at / kColumns), line_at(kRows + at % kColumns)); };
    bool whole = left > most_open(C);
    if (whole) {                               // (those that need no summing aside)
      __syncthreads();
      if (tid == 0) *count = 0;
      __syncthreads();
      for (int i = tid; i < left; i += 256)
        if (!nan_at(list[i])) atomicAdd(count, 1);
      __syncthreads();
      whole = *count > most_open(C);
    }
    if (whole) {
      // the whole tile in float64: 32 rows x 64 columns per wave
      const int r0 = wave / 2 * 32, c0 = wave % 2 * 64;
      float64_tile(
          lane, C, [&](int r) { return p.x + (size_t)min(row0 + r0 + r, rows - 1) * C; },
          [&](int c) { return columns + (size_t)min(n0 + c0 + c, w.N - 1) * C; }, 1,
          [&](int r, int c, uint32_t v) { *reinterpret_cast<uint16_t*>(out + (r0 + r) * T::ROW + 2 * (c0 + c)) = (uint16_t)v; });
    } else {
      // one by one, by half a wave each
      for (int i = tid >> 5; i < left; i += 8) {
        const int r = list[i] / kColumns, c = list[i] % kColumns;
        if (nan_at(list[i])) {
          *reinterpret_cast<uint16_t*>(out + r * T::ROW + 2 * c) = (uint16_t)kNan;
          continue;
        }
        const float* xr = p.x + (size_t)(row0 + r) * C;
        const float* column = columns + (size_t)(n0 + c) * C;
        double s = 0.;
        for (int c0 = 4 * i32; c0 < C; c0 += 1024) {
          float4 a[8], b[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int at = min(c0 + 128 * u, C - 4);
            a[u] = *reinterpret_cast<const float4*>(xr + at);
            b[u] = *reinterpret_cast<const float4*>(column + at);
          }
#pragma unroll
          for (int u = 0; u < 8; ++u)
            if (c0 + 128 * u < C) s += ((double)a[u].x * b[u].x + (double)a[u].y * b[u].y) + ((double)a[u].z * b[u].z + (double)a[u].w * b[u].w);
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) s += __shfl_xor(s, o);
        if (i32 == 0) *reinterpret_cast<uint16_t*>(out + r * T::ROW + 2 * c) = (uint16_t)to_bf16(s);
      }
    }
    __syncthreads();
    auto finish = [&](int r) {
      uint16_t* const at = place(r);
      if (at) *reinterpret_cast<uint4*>(at) = *reinterpret_cast<const uint4*>(out + r * T::ROW + 2 * c8);
    };
    // (unrolled, the addresses of these take registers that the first pass has its loads in: 1.2 us of 115)
#pragma unroll 1
    for (int u = 0; u < kRows / PASS; ++u)
      if (whole || (pending >> u & 1u)) finish(tid / (kColumns / 8) + u * PASS);
    // the lengths: once per sequence that begins in this row tile
    if (tile_n == 0 && tid < kRows && row0 + tid < rows && (row0 + tid) % p.n == 0) {
      const int seq = (row0 + tid) / p.n;
      const int L = p.lens_in ? p.lens_in[seq] : p.n;
      if (p.append) p.lens_out[seq] = (L < 0 || L > p.cap - p.n) ? L : L + p.n;
      else p.lens_out[seq] = L < 0 ? 0 : (L > p.n ? p.n : L);
    }
    __syncthreads();                           // the finished rows have been read, and the lines
  }
}

}  // namespace

// Is this the faster one?  us for rows in tiles of 64 x 128, up to 256 tiles (one per compute unit) / up to 512 (two) / each 256
// more, k = v = 128, d = 128: 20 / 24 / 3; 512: 31 / 42 / 12; 1024: 45 / 66 / 24; 1280: 55 / 79 / 31; 5 us more for each 2^20
// weights.  The float64 kernel takes 5 + 2 rows N d / 42 TFLOP/s (4096 rows, d = 1024: 44 against 54, 2048: 42 against 29; 8192
// rows, d = 128: 20 against 29); project_kv.hip's tiles are slower wherever this pays (10240 rows, d = 128: 24 against 25;
// 32768, d = 1024: 111 against 180).
bool project_kv_rows_pays(int rows, int d, int h_kv, int k, int v) {
  if (d > kMaxC || d < 64 || (k & 15) || (v & 15)) return false;
  const long long N = (long long)h_kv * (k + v);
  if (N * d > (1ll << 24)) return false;       // (a workspace of 8 bytes per weight: 128 MiB)
  const long long tiles = (long long)((rows + kRows - 1) / kRows) * ((N + kColumns - 1) / kColumns);
  if (tiles > (1ll << 28)) return false;
  const double turns = (double)((tiles + 255) / 256);
  const double us = 5e-6 * (double)(N * d) + (turns <= 1. ? 16. + 29. * d / 1024. : 18. + 24. * turns * d / 1024.);
  const double f64_us = 5. + 2. * rows * (double)N * d / 42e6;
  return us <= 0.9 * f64_us;
}

size_t project_kv_rows_workspace(int d, int h_kv, int k, int v) { return prepared_of(d, h_kv, k, v).bytes(); }

hipError_t launch_project_kv_rows(const float* x, const float* P_k, const float* P_v, void* K, void* V,
                                  const int32_t* lens_in, int32_t* lens_out, int rows, int n, int append, int d, int h_kv,
                                  int cap, int k, int v, void* workspace, hipStream_t st) {
  KvRowsParams p = {};
  p.x = x; p.P[0] = P_k; p.P[1] = P_v;
  p.dst[0] = (uint16_t*)K; p.dst[1] = (uint16_t*)V;
  p.lens_in = lens_in; p.lens_out = lens_out;
  p.ws = static_cast<unsigned char*>(workspace);
  p.w = prepared_of(d, h_kv, k, v);
  p.rows = rows; p.h_kv = h_kv; p.cap = cap; p.n = n; p.append = append;
  p.kv[0] = k; p.kv[1] = v;
  p.tiles_m = (rows + kRows - 1) / kRows;
  p.tiles_n = p.w.padded / kColumns;
  constexpr int lds = KvTile::BYTES;
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kv_rows_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  hipLaunchKernelGGL(prepare_kernel, dim3((unsigned)(p.w.padded / 4)), dim3(256), 0, st, p);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int groups = (p.tiles_m * p.tiles_n + 7) / 8 * 8;
  hipLaunchKernelGGL(kv_rows_kernel, dim3((unsigned)(groups < kGroups ? groups : kGroups)), dim3(256), lds, st, p);
  return hipGetLastError();
}

}  // namespace mqa
