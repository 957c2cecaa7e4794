// Causal attention of a whole prompt (bf16 cache, k = v = 128): the rows of a group are n queries x h heads that share
// its K and V (multi-query), or the n queries of one head; row r sees positions below L - n + r / h + 1.
//
// Long prompts are bound by the matrix cores and by the vector work between the two products, so everything
// that does not depend on the row is done once per workgroup instead of once per wave:
//   * A workgroup of four waves takes 128 rows, 32 per wave, and walks over the positions in tiles of 64.  The
//     tile is fetched with whole-row loads (one tile ahead in registers), V is transposed while it is stored to
//     LDS (16 byte permutes per thread and tile; every wave for itself took 64), and all waves read their operands from there.
//   * v_mfma_f32_32x32x16_bf16: S^T[32 pos x 32 rows] = K . q^T with q in registers; a lane has one row and
//     positions 8 (e / 4) + 4 g + e % 4, e < 16, of a block of 32.  O^T[32 cols x 32 rows] += V^T . P^T: step t takes
//     the positions of registers 8 t .. 8 t + 7, so the weights are B operands as they are, and V^T is stored in
//     that order: 16 bytes = positions 16 t + 4 g + 0..3 and 16 t + 8 + 4 g + 0..3 of one column.
//   * q and the weights are split into bf16 hi + lo terms (two products each), as in decode_mfma.hip.
//   * Two workgroups share a compute unit; the longest rows are started first.  Where there are not two for each, a workgroup is
//     two teams of four waves over the same rows, every second tile each, whose states are merged at the end.
// Measured (us; before: 32 rows per wave in decode_mfma.hip, every wave loading and transposing for itself; on one box): b=8,
// n=4096, h=8: 757 -> 582 (472 TFLOP/s of causal flops, four bf16 products each: 0.94 PFLOP/s); b=32, n=1024: 241 -> 192; b=128,
// n=128: 44.5 -> 36.8; one sequence of 4096: 168 -> 155; multi-head b=3, n=1000, h=16: 84 -> 63.  A tile's two
// blocks of 32 positions go through the softmax together: one after the other measured 609, and 178 for the one sequence (one
// wave per SIMD: nothing else fills the waits).  Storing the next tile between the products: 640 (registers spill).
// Positions at and beyond a row's limit get the logit -inf; V rows beyond the workgroup's last limit are stored as zeros,
// so the cache may hold anything there.  Before that limit a weight of 0 meets what V holds, and 0 . infinity is not 0: the tiles
// that not all rows see whole are searched for values that are not finite while they are stored, and a workgroup that
// finds one computes its rows again position by position.  The search costs 1 % at most (clearing the operands of
// such positions instead: 2 to 15 %, the product loop has no registers left for the masks).
#include "common.hpp"

namespace mqa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float floatx16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kRowBytes = 256;                 // one cache row
constexpr int kBufferWord3 = 0x00020000;       // raw 32-bit-element buffer, no swizzle
constexpr uint32_t kNoTile = 0x80000000u;      // an offset no cache reaches: zeros, nothing is fetched
constexpr float kSlack = 8.f;                  // log2 of the largest softmax weight kept before the running state is rescaled
constexpr int kTilePos = 64;
constexpr int kKBytes = kTilePos * kRowBytes, kBuffer = 2 * kKBytes;       // K tile, then V^T: 128 columns of 128 bytes

__device__ __forceinline__ floatx16 mfma32(const u32x4& a, const u32x4& b, const floatx16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// hi + lo bf16 terms of a pair: hi = rne(x), lo = rne(x - hi) (the difference is exact in float32)
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& hi, uint32_t& lo) {
  hi = pack_bf16_pair(a, b);
  lo = pack_bf16_pair(a - __uint_as_float(hi << 16), b - __uint_as_float(hi & 0xffff0000u));
}

// One row by one wave in plain float32 over the positions below its limit: a lane has a position of 64 for the
// logits, then two columns for the weighted sum.
__device__ __forceinline__ void plain_row(const DecodeParams& p, int seq, int row, int lim, int lane) {
  const float* q = p.q + ((size_t)seq * p.G + row) * 128;
  const uint16_t* K = static_cast<const uint16_t*>(p.K) + (size_t)seq * p.cap * 128;
  const uint32_t* V = static_cast<const uint32_t*>(p.V) + (size_t)seq * p.cap * 64;
  float m = -INFINITY, l = 0.f, a = 0.f, b = 0.f;
  for (int p0 = 0; p0 < lim; p0 += 64) {
    const int n = min(64, lim - p0);
    float z = -INFINITY;
    if (lane < n) {
      z = 0.f;
      for (int c = 0; c < 128; ++c) z = fmaf(q[c] * p.qscale, bf16_bits_to_float(K[(size_t)(p0 + lane) * 128 + c]), z);
    }
    const float mnew = fmaxf(m, wave_max(z)), ref = mnew == -INFINITY ? 0.f : mnew;
    const float w = lane < n ? __builtin_amdgcn_exp2f(z - ref) : 0.f, alpha = __builtin_amdgcn_exp2f(m - ref);
    l = l * alpha + wave_sum(w);
    a *= alpha;
    b *= alpha;
    m = mnew;
    for (int j = 0; j < n; ++j) {
      const uint32_t v = V[(size_t)(p0 + j) * 64 + lane];
      const float x = __shfl(w, j);
      a = fmaf(x, bf16_bits_to_float(v & 0xffffu), a);
      b = fmaf(x, __uint_as_float(v & 0xffff0000u), b);
    }
  }
  const float inv = l > 0.f ? 1.0f / l : 0.f;                // (a row with nothing to see: zeros)
  *reinterpret_cast<float2*>(p.o + ((size_t)seq * p.G + row) * 128 + 2 * lane) = make_float2(a * inv, b * inv);
}

template <int TEAMS>
__global__ __launch_bounds__(256 * TEAMS, 2)
void prompt_kernel(DecodeParams p) {
  extern __shared__ __align__(16) unsigned char smem_all[];  // per team: two buffers; at the end the waves' outputs
  const int team = TEAMS > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 8) : 0;
  unsigned char* const smem = smem_all + team * (2 * kBuffer);
  const int tid = threadIdx.x & 255, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i32 = lane & 31, g = lane >> 5;

  // Work item -> (sequence, row block), last (longest) row blocks first.  Whole sequences per XCD where they divide
  // evenly (its L2 then holds their K and V), else row blocks in turn over the XCDs.
  const int nb = gridDim.x, bid = blockIdx.x;
  const int wid = p.nseq % 8 == 0 ? (bid & 7) * (nb >> 3) + (bid >> 3) : bid;
  const int seq = wid / p.HG, row_block = p.HG - 1 - (wid - seq * p.HG);
  const int row0 = row_block * 128 + wave * 32;              // the wave's rows
  const int G = p.G, h = p.causal_h, nq = G / h;

  auto rows_of = [&](const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(base)) + (size_t)seq * p.cap * kRowBytes, 0, p.cap * kRowBytes, kBufferWord3);
  };
  const __amdgpu_buffer_rsrc_t Kbuf = rows_of(p.K), Vbuf = rows_of(p.V);
  int L = p.lens[seq / p.lens_div];
  L = L < 0 ? 0 : (L > p.cap ? p.cap : L);
  auto limit = [&](int row) { return max(0, L - nq + min(row, G - 1) / h + 1); };
  const int lim = limit(row0 + i32), lim_min = limit(row0), lim_max = limit(row0 + 31);
  const int end = limit(row_block * 128 + 127);              // of the workgroup
  const int lim_first = limit(row_block * 128);              // its first row's
  const int ntiles = (end + kTilePos - 1) / kTilePos;
  const int teams = TEAMS > 1 && ntiles > 4 ? TEAMS : 1;     // team e: the tiles e, e + teams, ...; of few tiles the first has them all (no merge)
  const int turns = (ntiles + teams - 1) / teams;
  int* const any_odd = reinterpret_cast<int*>(smem_all + TEAMS * 2 * kBuffer);
  int odd = 0;                                               // V holds something not finite that not all rows see

  // ---- staging: K chunk x = tid + 256 j (row x / 16, 16-byte chunk x % 16), kept at chunk ^ (row & 15); V rows 4 quad .. + 3,
  // columns 8 cg .. + 7, transposed.  V^T: 16-byte chunk (u, t, g) of column c at chunk ^ ((c >> 3) ^ c) & 7
  const int quad = tid >> 4, cg = tid & 15;
  const int v_chunk = (quad >> 3) * 4 + ((quad >> 2) & 1) * 2 + (quad & 1), v_half = (quad >> 1) & 1;
  u32x4 kst[4], vst[4];
  auto load_tile = [&](int t) {
    const uint32_t at = t < ntiles ? (uint32_t)t * (uint32_t)(kTilePos * kRowBytes) : kNoTile;
#pragma unroll
    for (int j = 0; j < 4; ++j) kst[j] = __builtin_amdgcn_raw_buffer_load_b128(Kbuf, at + (uint32_t)(tid + 256 * j) * 16u, 0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) vst[j] = __builtin_amdgcn_raw_buffer_load_b128(Vbuf, at + (uint32_t)((4 * quad + j) * kRowBytes + cg * 16), 0, 0);
  };
  auto store_tile = [&](int t, int buffer) {
    unsigned char* kb = smem + buffer * kBuffer;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = tid + 256 * j, row = x >> 4;
      *reinterpret_cast<u32x4*>(kb + row * kRowBytes + (((x & 15) ^ (row & 15)) << 4)) = kst[j];
    }
    if ((t + 1) * kTilePos > lim_first) {      // rows past the last limit may hold anything
      uint32_t most = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (t * kTilePos + 4 * quad + j >= end) vst[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int w = 0; w < 4; ++w) most = max(most, max(vst[j][w] & 0x7fff0000u, vst[j][w] << 16 & 0x7fff0000u));
      }
      if (__any(most >= 0x7f800000u)) odd = 1;
    }
    unsigned char* vb = kb + kKBytes + 8 * v_half;
#pragma unroll
    for (int w = 0; w < 4; ++w)
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        const uint32_t sel = par ? 0x07060302u : 0x05040100u;
        const int c = 2 * w + par, col = 8 * cg + c;
        const u32x2 x = u32x2{__builtin_amdgcn_perm(vst[1][w], vst[0][w], sel), __builtin_amdgcn_perm(vst[3][w], vst[2][w], sel)};
        *reinterpret_cast<u32x2*>(vb + col * 128 + ((v_chunk ^ ((cg ^ c) & 7)) << 4)) = x;
      }
  };

  if (team < teams) load_tile(team);
  if (threadIdx.x == 0) *any_odd = 0;
  // ---- q as B operands: lane (i, g) holds elements 16 s + 8 g .. + 7 of row i
  u32x4 qh[8], ql[8];
  if (team < teams) {
    const float4* src = reinterpret_cast<const float4*>(p.q + ((size_t)seq * G + min(row0 + i32, G - 1)) * 128) + 2 * g;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float4 a = src[4 * s], b = src[4 * s + 1];
      const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t hi, lo;
        split_pair(x[2 * d] * p.qscale, x[2 * d + 1] * p.qscale, hi, lo);
        qh[s][d] = hi;
        ql[s][d] = lo;
      }
    }
  }
  floatx16 acc[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[cb][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // logits of a tile's two blocks of 32 positions
  floatx16 sc[2];
  auto logits = [&](int buffer) {
    const unsigned char* kb = smem + buffer * kBuffer + i32 * kRowBytes;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[u][e] = 0.f;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      u32x4 a[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) a[u] = *reinterpret_cast<const u32x4*>(kb + 32 * u * kRowBytes + (((2 * s + g) ^ (i32 & 15)) << 4));
#pragma unroll
      for (int u = 0; u < 2; ++u) sc[u] = mfma32(a[u], qh[s], sc[u]);
#pragma unroll
      for (int u = 0; u < 2; ++u) sc[u] = mfma32(a[u], ql[s], sc[u]);
    }
  };
  // online softmax (lazy rescaling, see decode_mfma.hip) and weighted sum
  auto weigh = [&](int t, int buffer) {
    const int p0 = t * kTilePos;
    const unsigned char* vb = smem + buffer * kBuffer + kKBytes;
    if (p0 + kTilePos > lim_min) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (p0 + 32 * u + 8 * (e >> 2) + 4 * g + (e & 3) >= lim) sc[u][e] = -INFINITY;
    }
    float mx = fmaxf(sc[0][0], sc[1][0]);
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, fmaxf(sc[0][e], sc[1][e]));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mnew = fmaxf(m_run, mx);
    if (__any(mnew > m_run + kSlack)) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - (mnew == -INFINITY ? 0.f : mnew));      // (a row that has seen nothing yet)
      l_run *= alpha;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] *= alpha;
      m_run = mnew;
    }
    const float mref = m_run == -INFINITY ? 0.f : m_run;
    float sum[2] = {0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int u = s >> 1;
      u32x4 hi, lo;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const float x = __builtin_amdgcn_exp2f(sc[u][8 * (s & 1) + 2 * d] - mref), y = __builtin_amdgcn_exp2f(sc[u][8 * (s & 1) + 2 * d + 1] - mref);
        sum[0] += x;
        sum[1] += y;
        uint32_t hh, ll;
        split_pair(x, y, hh, ll);
        hi[d] = hh;
        lo[d] = ll;
      }
      const int chunk = 2 * s + g;
      u32x4 a[4];
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int col = 32 * cb + i32;
        a[cb] = *reinterpret_cast<const u32x4*>(vb + col * 128 + ((chunk ^ (((col >> 3) ^ col) & 7)) << 4));
      }
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = mfma32(a[cb], hi, acc[cb]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) acc[cb] = mfma32(a[cb], lo, acc[cb]);
    }
    l_run += sum[0] + sum[1];
  };

  if (ntiles > 0 && team < teams) {
    store_tile(team, 0);
    load_tile(team + teams);
  }
  __syncthreads();
  for (int u = 0; u < turns; ++u) {
    // (buffer u + 1 was last read in round u - 1, which the barrier at its end closed)
    const int t = u * teams + team;
    const bool sees = team < teams && t * kTilePos < lim_max;      // (the same for the whole wave; past the last tile: none)
    if (u + 1 < turns && team < teams) {
      store_tile(t + teams, (u + 1) & 1);
      load_tile(t + 2 * teams);
    }
    if (odd) *any_odd = 1;
    if (sees) { logits(u & 1); weigh(t, u & 1); }
    __syncthreads();
  }

  if (__builtin_expect(*any_odd, 0)) {
    constexpr int ROWS = 32 / TEAMS;
    for (int row = row0 + team * ROWS; row < min(row0 + (team + 1) * ROWS, G); ++row) plain_row(p, seq, row, limit(row), lane);
    return;
  }
  if (teams > 1) {
    // the second team's states meet the first's in LDS: sums in its own buffers, maxima and sums of weights where the first's wave
    // will put its rows (its own reads come before its writes)
    float* const at = reinterpret_cast<float*>(smem_all + 2 * kBuffer) + wave * (64 * 64) + lane;
    float* const ml = reinterpret_cast<float*>(smem_all) + wave * (32 * 128) + lane;
    if (team == 1) {
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) at[(cb * 16 + e) * 64] = acc[cb][e];
      ml[0] = m_run;
      ml[64] = l_run;
    }
    __syncthreads();
    if (team == 0) {
      const float m = ml[0], l = ml[64], top = fmaxf(m_run, m), ref = top == -INFINITY ? 0.f : top;
      const float mine = __builtin_amdgcn_exp2f(m_run - ref), other = __builtin_amdgcn_exp2f(m - ref);      // (0 for a state that saw nothing)
      l_run = l_run * mine + l * other;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[cb][e] = acc[cb][e] * mine + at[(cb * 16 + e) * 64] * other;
    }
  }

  // ---- output: through the wave's quarter of LDS, so that rows leave as whole lines.  acc[cb][e] is column 32 cb + 8 (e / 4)
  // + 4 g + e % 4 of row i32
  float4* rows = reinterpret_cast<float4*>(smem_all + wave * (32 * 512));
  if (team == 0) {
    const float lsum = l_run + __shfl_xor(l_run, 32);
    const float inv = lsum > 0.f ? 1.0f / lsum : 0.f;        // (a row with nothing to see: zeros)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        rows[i32 * 32 + ((8 * cb + 2 * q + g) ^ i32)] =
            make_float4(acc[cb][4 * q] * inv, acc[cb][4 * q + 1] * inv, acc[cb][4 * q + 2] * inv, acc[cb][4 * q + 3] * inv);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 32 / TEAMS; r += 2) {
    const int row = r + g + team * (32 / TEAMS);
    if (row0 + row < G) reinterpret_cast<float4*>(p.o + ((size_t)seq * G + row0 + row) * 128)[i32] = rows[row * 32 + (i32 ^ row)];
  }
}

template <int TEAMS>
hipError_t launch_teams(const DecodeParams& p, unsigned nblocks, hipStream_t st) {
  constexpr int lds = TEAMS * 2 * kBuffer + 16;
  static bool done[64] = {};                   // once per device
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (!done[dev]) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(prompt_kernel<TEAMS>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    done[dev] = true;
  }
  hipLaunchKernelGGL(prompt_kernel<TEAMS>, dim3(nblocks), dim3(256 * TEAMS), lds, st, p);
  return hipGetLastError();
}

}  // namespace

// Two teams where a compute unit has one workgroup at most and the capacity is more than two tiles each.  us, one team / two: one sequence of 4096, h=8:
// 146 / 107, of 1024: 41 / 33; multi-head n=700, prefix 100, b=4, h=5: 36 / 29; h=1, n=2000: 83 / 61.  A workgroup that turns out to have four tiles
// or fewer leaves them to its first team, the second one waiting at the barriers without its q: 128 positions of 2048, b=16 11.7 / 11.4 (shared and
// merged 13.2), 64 of 1024, b=32 9.1 / 9.4 (12.1).
hipError_t launch_prompt(const DecodeParams& p, hipStream_t st) {
  const long long nblocks = (long long)p.nseq * p.HG;        // HG: blocks of 128 rows
  if (nblocks > 0x7fffffffll) return hipErrorInvalidValue;
  return nblocks <= 256 && p.cap > 4 * kTilePos ? launch_teams<2>(p, (unsigned)nblocks, st) : launch_teams<1>(p, (unsigned)nblocks, st);
}

}  // namespace mqa
