// New K / V rows of many positions at once (a memory, a prompt, for callers without a workspace: project_kv_rows.hip is the
// faster one with; or one position of very many sequences) into a bf16 cache: the correctly rounded
// value of the product, which is what the float64 kernel of project.hip writes, without its cost.  (Where the products
// cancel so far that the rounding of the float64 sums themselves decides the bf16 value, the order of those sums shows,
// as it does between any two float64 kernels.)
//
// float64 matrix instructions run at 1/32 of the 16-bit rate and bounded this product (32768 rows, d = 1024, 256
// columns: 42 TFLOP/s, 410 us; this kernel 180: of a tile's 90 us about 20 are the first pass and 20 the open elements; the
// matrix cores are busy 18 %, vector instructions 34 %; two and three stages ahead measured the same).  Here the sum is found with a bound on its error from exact integer products, and
// only the elements whose rounding to bf16 the bound leaves open (0.09 % of normal deviates at d = 1024) are summed in float64.
// (Exact products of operands cut into slices of few bits: after Ozaki, Ogita, Oishi, Rump 2012; here in integers.)
//   * Fixed point: a row of the input and a column of the weights are scaled by a power of two that takes
//     their largest value to [2^29, 2^31 - 2^24], and truncated to integers X, Y of four balanced base-256 digits,
//     X = d3 2^24 + d2 2^16 + d1 2^8 + d0, every digit an int8.
//   * X . Y = sum over (i, j) of 2^(8 (i + j)) (d_i . e_j); the ten products with i + j >= 3 are computed on
//     v_mfma_i32_32x32x32_i8 (twice the 16-bit rate), exactly, in one int32 sum per i + j.
//   * Error, in units of X . Y: the truncation, below sum |X| + sum |Y| + 3 C, and the dropped digit products, by
//     Cauchy-Schwarz below 2^16 (|d2||e0| + |d1||e1| + |d0||e2|) + 2^9 2^14 C; the digits' norms are summed
//     while they are staged (v_dot4), and |X| <= 2^24 (|d3| + 1).
//   * An element is done if both ends of sum +- bound round to the same bf16 (through float32, as the float64
//     kernel rounds): its distance from the nearest tie against the bound; the others are summed by one wave each, in float64,
//     or, where a tile has many (rows or columns of a few large values), all of it on the float64 instructions.  Rows or columns with a NaN are NaN; one
//     with an infinity has no fixed point and goes the float64 way.
//
// Workgroup: 512 threads, 128 x 128 tile, wave (wr, wc) of 4 x 2 holds 32 x 64 of it.  A first pass over the
// operands finds the largest values (they come from L2 the second time); then stages of 32 contraction indices go
// global -> registers (one stage ahead) -> digits -> LDS (two buffers, one barrier per stage), waves 0..3 staging
// rows before they multiply, waves 4..7 columns after they have.
#include "kv_fixed.hpp"

#include <type_traits>

namespace mqa {
namespace {

using namespace kv_fixed;

constexpr int kTile = 128;
constexpr int kBlock = 64 * 16 + 64;            // 16 indices of 64 lines, 16 bytes per line; what eight lanes write (four rows' two
constexpr int kHalf = 2 * kBlock;              // halves, or four columns of each parity) lies on different banks
constexpr int kPlane = 2 * kHalf;              // one digit of 32 indices
constexpr int kOperand = 4 * kPlane;
constexpr int kStage = 2 * kOperand;

struct KvParams {
  const float* x;                // [rows, C]
  const float* P[2];             // [h_kv, C, kv[which]]
  uint16_t* dst[2];              // caches [seq, h_kv, cap, kv[which]]
  const int32_t* lens_in;        // append: rows already there; else valid rows per sequence, or null
  int32_t* lens_out;
  int rows, C, h_kv, cap, n;     // row r is row r % n of sequence r / n
  int kv[2], tiles[2];           // columns per head, column tiles of K and V
  int append, tiles_m;
};

__global__ __launch_bounds__(512)
void project_kv_exact_kernel(KvParams p) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* most = reinterpret_cast<uint32_t*>(smem + 2 * kStage);      // [256] bits of the largest |value| of a row / column
  int* norm = reinterpret_cast<int*>(most + 256);                       // [256][4] sums of the squared digits
  int* count = norm + 1024;

  // column tiles of a row tile are neighbours on one XCD
  const int tiles_n = p.tiles[0] + p.tiles[1];
  const int per_xcd = gridDim.x >> 3;
  const int work = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (work >= p.tiles_m * tiles_n) return;
  const int tile_m = work / tiles_n;
  int tile_n = work - tile_m * tiles_n;
  const int which = tile_n >= p.tiles[0] ? 1 : 0;
  if (which) tile_n -= p.tiles[0];
  const int row0 = tile_m * kTile, n0 = tile_n * kTile;
  const int kv = p.kv[which], N = p.h_kv * kv, C = p.C, rows = p.rows;
  const float* P = p.P[which];
  const size_t head_stride = (size_t)C * kv;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31, g = lane >> 5, wr = wave >> 1, wc = wave & 1;
  const int ts = tid & 255;
  const int nst = (C + 31) >> 5;

  for (int i = tid; i < 1280; i += 512) most[i] = 0;                    // (and the norms behind them)
  if (tid == 0) *count = 0;
  __syncthreads();

  int16v acc[4][2];                            // sums of the digit products with i + j = 3 + t, per column block
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[t][j][e] = 0;

  auto multiply = [&](int buf) {
    const unsigned char* As = smem + buf * kStage + g * kHalf + (wr >> 1) * kBlock + ((wr & 1) * 32 + i32) * 16;
    const unsigned char* Bs = smem + buf * kStage + kOperand + g * kHalf + (wc * 32 + i32) * 16;
    int4v a[4], b[4][2];
#pragma unroll
    for (int q = 3; q >= 0; --q) {
      a[q] = *reinterpret_cast<const int4v*>(As + q * kPlane);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[q][j] = *reinterpret_cast<const int4v*>(Bs + q * kPlane + j * kBlock);
    }
#pragma unroll
    for (int i = 3; i >= 0; --i)
#pragma unroll
      for (int e = 3; e >= 0; --e)
        if (i + e >= 3)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i + e - 3][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[e][j], acc[i + e - 3][j], 0, 0, 0);
  };

  // staging: a thread holds sixteen indices (half a stage) of a row or a column
  auto run = [&](auto role) {
    constexpr bool ROWS = decltype(role)::value;
    const int half = ROWS ? ts & 1 : ts >> 7;
    const int line = ROWS ? ts >> 1 : (ts & 1) * 64 + ((ts & 127) >> 1);       // row of the tile; column: even ones first, then odd ones
    const float* src;
    if constexpr (ROWS) {
      src = p.x + (size_t)min(row0 + line, rows - 1) * C;
    } else {
      const int n = min(n0 + (ts & 127), N - 1);
      src = P + (size_t)(n / kv) * head_stride + n % kv;
    }
    struct Regs { float x[16]; };
    auto load_stage = [&](int st, Regs& rg) {  // (indices past the end are clamped in eights, and dropped before use)
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int c = min(32 * st + 16 * half + 8 * o, C - 8);
        if constexpr (ROWS) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const float4 v = *reinterpret_cast<const float4*>(src + c + 4 * i);
            rg.x[8 * o + 4 * i] = v.x; rg.x[8 * o + 4 * i + 1] = v.y; rg.x[8 * o + 4 * i + 2] = v.z; rg.x[8 * o + 4 * i + 3] = v.w;
          }
        } else {
          const float* at = src + (size_t)c * kv;
#pragma unroll
          for (int i = 0; i < 8; ++i) rg.x[8 * o + i] = at[(size_t)i * kv];
        }
      }
    };
    uint32_t* my_most = most + (ROWS ? 0 : 128);
    int* my_norm = norm + (ROWS ? 0 : 512);

    // ---- first pass: the largest magnitudes (a clamped load repeats a value: no harm)
    {
      uint32_t m = 0;
      constexpr int AHEAD = 4;
      Regs rg[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) load_stage(u, rg[u]);
      for (int s0 = 0; s0 < nst; s0 += AHEAD)
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
#pragma unroll
          for (int k = 0; k < 16; ++k) m = max(m, __float_as_uint(rg[u].x[k]) & 0x7fffffffu);
          load_stage(s0 + u + AHEAD, rg[u]);
        }
      atomicMax(&my_most[line], m);
    }
    __syncthreads();
    const float scale = __uint_as_float((uint32_t)(fixed_exponent(my_most[line]) + 127) << 23);
    int sq[4] = {0, 0, 0, 0};
    auto store_stage = [&](int st, Regs& rg) {
      const float by[2] = {32 * st + 16 * half >= C ? 0.f : scale, 32 * st + 16 * half + 8 >= C ? 0.f : scale};      // (C is a multiple of 8)
      unsigned char* dst = smem + (st & 1) * kStage + (ROWS ? 0 : kOperand) + half * kHalf + (line >> 6) * kBlock + (line & 63) * 16;
      int4v d[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) {            // bytes of four values -> four digits' words
        const float* x = rg.x + 4 * w;
        const Digits4 t = digits_of(x[0] * by[w >> 1], x[1] * by[w >> 1], x[2] * by[w >> 1], x[3] * by[w >> 1]);
#pragma unroll
        for (int q = 0; q < 4; ++q) d[q][w] = t.word[q];
#pragma unroll
        for (int q = 0; q < 4; ++q) sq[q] = __builtin_amdgcn_sdot4(d[q][w], d[q][w], sq[q], false);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) *reinterpret_cast<int4v*>(dst + q * kPlane) = d[q];
    };
    Regs regs;
    load_stage(0, regs);
    store_stage(0, regs);
    load_stage(1, regs);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
      if constexpr (ROWS) multiply(st & 1);
      store_stage(st + 1, regs);               // (past the end: digits of zero)
      load_stage(st + 2, regs);
      if constexpr (!ROWS) multiply(st & 1);
      __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) atomicAdd(&my_norm[4 * line + q], sq[q]);
    __syncthreads();
  };
  if (wave < 4) run(std::true_type{});
  else run(std::false_type{});

  // ---- sums, bounds, rounding.  Register e of lane (i, g) is row 8 (e/4) + 4 g + e%4 of the block; the lane's two column
  // blocks are the columns 2 i', 2 i' + 1 (one 4-byte store)
  const int slot = wc * 32 + i32, n = n0 + 2 * slot;
  uint16_t* list = reinterpret_cast<uint16_t*>(smem);        // [16384] elements that are left open: row << 7 | column
  auto place = [&](int row, int col) -> uint16_t* {          // null: nothing is written
    const int seq = row / p.n;
    int at = row - seq * p.n;
    if (p.append) {
      const int L = p.lens_in[seq];
      if (L < 0 || L > p.cap - p.n) return nullptr;            // (n <= cap; a sum could wrap)
      at += L;
    }
    return p.dst[which] + (((size_t)seq * p.h_kv + col / kv) * p.cap + at) * kv + col % kv;
  };
  // the lines take the places of their sums of squares
  static_assert(sizeof(Line) <= 16, "a line takes the place of its four sums");
  auto line_at = [&](int i) -> Line& { return *reinterpret_cast<Line*>(norm + 4 * i); };
  if (tid < 256) {
    const int4v sums = *reinterpret_cast<const int4v*>(norm + 4 * tid);      // (all of them, before the first float goes into their place)
    const int squares[4] = {sums[0], sums[1], sums[2], sums[3]};
    line_at(tid) = line_of(squares, most[tid], C);
  }
  __syncthreads();
  const Line col[2] = {line_at(128 + slot), line_at(192 + slot)};
  for (int chunk = 0; chunk < 4; ++chunk) {
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
      // (the registers of a chunk, by constant indices)
      int t[4][2];
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (c == chunk)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < 2; ++j) t[q][j] = acc[q][j][4 * c + e4];
      const int r = wr * 32 + 8 * chunk + 4 * g + e4, row = row0 + r;
      if (row >= rows || n >= N) continue;
      const Line mine = line_at(r);
      uint32_t out = 0;
      bool open[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint32_t v = rounded_sum(digit_sum(t[0][j], t[1][j], t[2][j], t[3][j]), mine, col[j], &open[j]);
        if (open[j]) {
          if (is_nan(mine, col[j])) v = kNan, open[j] = false;
          else list[atomicAdd(count, 1)] = (uint16_t)(r << 7 | (2 * slot + j));
        }
        out |= v << (16 * j);
      }
      uint16_t* at = place(row, n);
      if (at) {
        if (!open[0] && !open[1]) *reinterpret_cast<uint32_t*>(at) = out;
        else if (!open[0]) at[0] = (uint16_t)out;
        else if (!open[1]) at[1] = (uint16_t)(out >> 16);
      }
    }
  }
  __syncthreads();
  const int left = *count;
  if (left > kMostOpen) {
    const int r0 = row0 + wr * 32, c0 = n0 + wc * 64;
    float64_tile(
        lane, C, [&](int r) { return p.x + (size_t)min(r0 + r, rows - 1) * C; },
        [&](int c) { const int at = min(c0 + c, N - 1); return P + (size_t)(at / kv) * head_stride + at % kv; }, kv,
        [&](int r, int c, uint32_t v) {
          uint16_t* at = r0 + r < rows && c0 + c < N ? place(r0 + r, c0 + c) : nullptr;
          if (at) *at = (uint16_t)v;
        });
  }
  else for (int i = wave; i < left; i += 8) {
    const int r = list[i] >> 7, col = n0 + (list[i] & 127);
    const float* xr = p.x + (size_t)(row0 + r) * C;
    const float* w = P + (size_t)(col / kv) * head_stride + col % kv;
    double s = 0.;
    for (int c0 = lane; c0 < C; c0 += 64 * 8) {              // 16 loads in flight: a wave's time here is their latency
      float a[8], b[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int c = min(c0 + 64 * u, C - 1);
        a[u] = xr[c];
        b[u] = w[(size_t)c * kv];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (c0 + 64 * u < C) s += (double)a[u] * (double)b[u];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) {
      uint16_t* at = place(row0 + r, col);
      if (at) *at = (uint16_t)to_bf16(s);
    }
  }

  // the lengths: once per sequence that begins in this row tile
  if (which == 0 && tile_n == 0 && tid < kTile && row0 + tid < rows && (row0 + tid) % p.n == 0) {
    const int seq = (row0 + tid) / p.n;
    const int L = p.lens_in ? p.lens_in[seq] : p.n;
    if (p.append) p.lens_out[seq] = (L < 0 || L > p.cap - p.n) ? L : L + p.n;
    else p.lens_out[seq] = L < 0 ? 0 : (L > p.n ? p.n : L);
  }
}

}  // namespace

// Is this kernel the faster one?  Rounds of one tile per compute unit, 100 us each at d = 1024, against the float64 kernel's
// 42 TFLOP/s: pays from about 140 tiles on (at 256: 105 against 210 us)
static long long tiles_n_of(int h_kv, int kv) { return ((long long)h_kv * kv + kTile - 1) / kTile; }
bool project_kv_exact_pays(int rows, int d, int h_kv, int k, int v) {
  if (d > kMaxC || (k & 1) || (v & 1)) return false;
  const long long tiles = (rows + kTile - 1) / kTile * (tiles_n_of(h_kv, k) + tiles_n_of(h_kv, v));
  const double exact_us = 5. + 100. * d / 1024. * (double)((tiles + 255) / 256);
  const double f64_us = 5. + 2. * rows * ((double)h_kv * k + (double)h_kv * v) * d / 42e6;
  return exact_us <= 0.9 * f64_us;
}

hipError_t launch_project_kv_exact(const float* x, const float* P_k, const float* P_v, void* K, void* V,
                                   const int32_t* lens_in, int32_t* lens_out, int rows, int n, int append, int d, int h_kv,
                                   int cap, int k, int v, hipStream_t st) {
  if (!project_kv_exact_pays(rows, d, h_kv, k, v)) return hipErrorNotSupported;
  KvParams p = {};
  p.x = x; p.P[0] = P_k; p.P[1] = P_v;
  p.dst[0] = (uint16_t*)K; p.dst[1] = (uint16_t*)V;
  p.lens_in = lens_in; p.lens_out = lens_out;
  p.rows = rows; p.C = d; p.h_kv = h_kv; p.cap = cap; p.n = n; p.append = append;
  p.kv[0] = k; p.kv[1] = v;
  p.tiles[0] = (int)tiles_n_of(h_kv, k);
  p.tiles[1] = (int)tiles_n_of(h_kv, v);
  p.tiles_m = (rows + kTile - 1) / kTile;
  const long long tiles = (long long)p.tiles_m * (p.tiles[0] + p.tiles[1]);
  constexpr size_t lds = 2 * kStage + 1280 * 4 + 16;
  static bool done[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(project_kv_exact_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  hipLaunchKernelGGL(project_kv_exact_kernel, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(512), lds, st, p);
  return hipGetLastError();
}

}  // namespace mqa
