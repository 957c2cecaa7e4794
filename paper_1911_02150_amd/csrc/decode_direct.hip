// Decode attention for float32 caches (k = v = 64 or 128) and bf16 caches with k = v = 64, on the
// float32 matrix instructions.  Same contract and partial-state format as the bf16 MFMA kernel
// (decode_mfma.hip); everything is multiplied and accumulated in float32.
//
// What bounds it is the one read of K and V; v_mfma_f32_16x16x4_f32 takes 32 bytes of a float32 cache per clock
// and compute unit with 16 heads, three times what HBM delivers, although fewer heads leave columns idle.  So
// the cache goes from memory straight into the registers of the operands: no LDS, no barrier, no
// vector arithmetic but the softmax.
//   * One workgroup per (sequence, position range, group of 16*HB heads); wave w takes the tiles of 16
//     positions w, w + NW, ... and the NW states are merged through LDS at the end.
//   * logits^T tile = K_tile[16 pos x k] . q^T[k x 16 heads]: lane (i, g), i = lane % 16, g = lane / 16, loads
//     elements 16 s + 4 g .. + 3 of row i; the matrix step (s, e) contracts elements 16 s + 4 g + e, g = 0..3.
//     q sits in registers in the same layout.  The lane gets the logits of head i, positions 4 g + r.
//   * O^T[16 cols x 16 heads] += V^T[16 cols x 4 pos] . P^T[4 pos x 16 heads]: step r takes positions 4 g + r, so
//     the lane's four weights are its B operands as they are; for A it loads columns 64 jj + 4 i .. + 3 of the rows
//     4 g + r (256 contiguous bytes of four rows per instruction), and block (jj, e) is columns 64 jj + 4 i + e.
//   * A tile's registers are refilled with the wave's next tile as soon as they are read.
// Measured (us, the plain float32 kernel of decode_generic.hip -> this; with the merge of the ranges): float32, k = 128:
// b=32, h=8, m=2048: 32.0 -> 17.1; b=502, h=18, m=132: 102 -> 28; b=37, h=33, ragged to 4986: 301 -> 67; k = 64: b=207,
// h=2, ragged to 2106: 59 -> 38; bf16, k = 64: b=60, h=11, m=2053: 57 -> 18.5; b=115, h=1, m=3591: 63 -> 37.
// No shape was found where the plain kernel is the faster one, so it only keeps the widths this one lacks.
// Rows at and beyond the length are never used: their logits become -inf and their V registers zero.
// K and V are read through buffer descriptors of the sequence's capacity (zeros beyond it), so that the
// first tile is requested before the length has arrived.
#include "common.hpp"

namespace mqa {
namespace {

typedef __attribute__((ext_vector_type(4))) float floatx4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr int kBufferWord3 = 0x00020000;     // raw 32-bit-element buffer, no swizzle
constexpr uint32_t kNoTile = 0x80000000u;    // an offset no cache reaches: nothing is fetched
constexpr float kSlack = 8.f;                // log2 of the largest softmax weight kept before the running state is rescaled

// four consecutive cache elements, as loaded, and as floats
template <typename T> struct Four;
template <> struct Four<float> {
  u32x4 x;
  template <int AUX> __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t b, uint32_t off) { x = __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, AUX); }
  __device__ __forceinline__ float operator[](int e) const { return __uint_as_float(x[e]); }
  __device__ __forceinline__ void clear() { x = u32x4{0u, 0u, 0u, 0u}; }
};
template <> struct Four<uint16_t> {
  u32x2 x;
  template <int AUX> __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t b, uint32_t off) { x = __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, AUX); }
  __device__ __forceinline__ float operator[](int e) const { return __uint_as_float((e & 1) ? x[e >> 1] & 0xffff0000u : x[e >> 1] << 16); }
  __device__ __forceinline__ void clear() { x = u32x2{0u, 0u}; }
};

template <int KD, int HB, int NW> constexpr int merge_floats() { return NW * 16 * HB * (KD + 4) + 2 * NW * 16 * HB; }

template <typename T, int KD, int HB, int NW, bool NTL>
__global__ __launch_bounds__(NW * 64)
void decode_direct_kernel(DecodeParams p, int HG) {
  constexpr int KS = KD / 16;                 // loads per K row and lane
  constexpr int JJ = KD / 64;                 // loads per V row and lane
  constexpr int NH = 16 * HB;
  constexpr uint32_t ROW = KD * sizeof(T);    // bytes
  constexpr int AUX = NTL ? 2 : 0;            // non-temporal: every row is read once (unless a second head group follows)
  extern __shared__ __align__(16) float merge[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g = lane >> 4;

  // consecutive work items share an XCD
  const int nb = gridDim.x, bid = blockIdx.x;
  const int wid = ((nb & 7) == 0) ? (bid & 7) * (nb >> 3) + (bid >> 3) : bid;
  const int hg = wid % HG, srange = (wid / HG) % p.S, seq = wid / (HG * p.S);
  const int head0 = hg * NH;
  int begin = srange * p.chunk;

  auto rows_of = [&](const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(base)) + (size_t)seq * p.cap * ROW, 0, (int)(p.cap * ROW), kBufferWord3);
  };
  const __amdgpu_buffer_rsrc_t Kbuf = rows_of(p.K), Vbuf = rows_of(p.V);
  const uint32_t klane = i16 * ROW + 4 * g * sizeof(T), vlane = 4 * g * ROW + 4 * i16 * sizeof(T);
  Four<T> kr[KS], vr[4][JJ];
  auto tile_offset = [&](int t, bool wanted) -> uint32_t { return wanted ? (uint32_t)(begin + 16 * t) * ROW : kNoTile; };
  auto load_k = [&](uint32_t toff) {
#pragma unroll
    for (int s = 0; s < KS; ++s) kr[s].template load<AUX>(Kbuf, klane + toff + (uint32_t)(16 * s * sizeof(T)));
  };
  auto load_v = [&](uint32_t toff) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int jj = 0; jj < JJ; ++jj) vr[r][jj].template load<AUX>(Vbuf, vlane + toff + (uint32_t)(r * ROW + 64 * jj * sizeof(T)));
  };

  // q first (it is needed first), then the first tile, before the length is known
  floatx4 q[HB][KS];
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {
    const int head = min(head0 + 16 * hb + i16, p.G - 1);      // (columns past the last head are not stored)
    const floatx4* src = reinterpret_cast<const floatx4*>(p.q + ((size_t)seq * p.G + head) * KD) + g;
#pragma unroll
    for (int s = 0; s < KS; ++s) q[hb][s] = src[4 * s];
  }
  if (p.window == 0) {
    load_k(tile_offset(wave, true));
    load_v(tile_offset(wave, true));
  }
  int L = p.lens[seq / p.lens_div];
  L = L < 0 ? 0 : (L > p.cap ? p.cap : L);
  const int lo = window_lo(L, p.window);
  if (p.window > 0) {                          // the ranges start at the 32-aligned position below the window
    begin += window_base(L, p.window);
    load_k(tile_offset(wave, true));
    load_v(tile_offset(wave, true));
  }
  const int end = min(begin + p.chunk, L);
  if (end <= begin) {                          // (ranges past the length write nothing; the combine pass skips them)
    if (p.PS == 0)
      for (int idx = tid; idx < NH * (KD / 4); idx += NW * 64) {
        const int hl = idx / (KD / 4), c4 = idx % (KD / 4);
        if (head0 + hl < p.G)
          reinterpret_cast<float4*>(p.o + ((size_t)seq * p.G + head0 + hl) * KD)[c4] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    return;
  }
  const int ntiles = (end - begin + 15) >> 4;
#pragma unroll
  for (int hb = 0; hb < HB; ++hb)
#pragma unroll
    for (int s = 0; s < KS; ++s) q[hb][s] *= p.qscale;

  floatx4 acc[HB][4 * JJ];
  float m_run[HB], l_run[HB];
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {
    m_run[hb] = -INFINITY;
    l_run[hb] = 0.f;
#pragma unroll
    for (int j = 0; j < 4 * JJ; ++j) acc[hb][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  for (int t = wave; t < ntiles; t += NW) {
    const int p0 = begin + 16 * t;
    const uint32_t next = tile_offset(t + NW, t + NW < ntiles);
    floatx4 sc[HB];
    {
      floatx4 half[HB][2];                     // two chains: a matrix step waits for the one before the last
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) half[hb][0] = half[hb][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int hb = 0; hb < HB; ++hb)
            half[hb][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[s][e], q[hb][s][e], half[hb][e & 1], 0, 0, 0);
#pragma unroll
      for (int hb = 0; hb < HB; ++hb) sc[hb] = half[hb][0] + half[hb][1];
    }
    load_k(next);
    if (__builtin_expect(p0 + 16 > end || p0 < lo, 0)) {       // drop positions outside [lo, end)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int pos = p0 + 4 * g + r;
        if (pos >= end || pos < lo) {
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) sc[hb][r] = -INFINITY;
#pragma unroll
          for (int jj = 0; jj < JJ; ++jj) vr[r][jj].clear();
        }
      }
    }
#pragma unroll
    for (int hb = 0; hb < HB; ++hb) {
      float mx = fmaxf(fmaxf(sc[hb][0], sc[hb][1]), fmaxf(sc[hb][2], sc[hb][3]));
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      // the reference of the exponentials moves only when a row's maximum has grown by more than 2^kSlack
      const float mnew = fmaxf(m_run[hb], mx);
      if (__any(mnew > m_run[hb] + kSlack)) {
        const float alpha = __builtin_amdgcn_exp2f(m_run[hb] - (mnew == -INFINITY ? 0.f : mnew));      // (a window's first tile may hold nothing)
        l_run[hb] *= alpha;
#pragma unroll
        for (int j = 0; j < 4 * JJ; ++j) acc[hb][j] *= alpha;
        m_run[hb] = mnew;
      }
      const float mref = m_run[hb] == -INFINITY ? 0.f : m_run[hb];
#pragma unroll
      for (int r = 0; r < 4; ++r) sc[hb][r] = __builtin_amdgcn_exp2f(sc[hb][r] - mref);
      l_run[hb] += (sc[hb][0] + sc[hb][1]) + (sc[hb][2] + sc[hb][3]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float v = vr[r][jj][e];
#pragma unroll
          for (int hb = 0; hb < HB; ++hb) acc[hb][4 * jj + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, sc[hb][r], acc[hb][4 * jj + e], 0, 0, 0);
        }
    load_v(next);
  }

  // ---- merge the NW states.  Lane (i, g) holds, of head i, columns 64 jj + 16 g + 4 r + e (block (jj, e), register r)
  float* so = merge;                                        // [NW][NH][KD + 4]
  float* sm = so + NW * NH * (KD + 4);                      // [NH][NW] maxima
  float* sl = sm + NW * NH;                                 // [NH][NW] sums
#pragma unroll
  for (int hb = 0; hb < HB; ++hb) {
    if (head0 + 16 * hb + i16 < p.G) {
      float* row = so + ((size_t)wave * NH + 16 * hb + i16) * (KD + 4);
#pragma unroll
      for (int jj = 0; jj < JJ; ++jj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          *reinterpret_cast<float4*>(row + 64 * jj + 16 * g + 4 * r) =
              make_float4(acc[hb][4 * jj][r], acc[hb][4 * jj + 1][r], acc[hb][4 * jj + 2][r], acc[hb][4 * jj + 3][r]);
    }
    float lq = l_run[hb];
    lq += __shfl_xor(lq, 16);
    lq += __shfl_xor(lq, 32);
    if (g == 0) {
      sm[(16 * hb + i16) * NW + wave] = m_run[hb];
      sl[(16 * hb + i16) * NW + wave] = lq;
    }
  }
  __syncthreads();
  const int heads = min(NH, p.G - head0);
  for (int idx = tid; idx < heads * (KD / 4); idx += NW * 64) {
    const int hl = idx / (KD / 4), c4 = idx % (KD / 4);
    float f[NW];
    float M = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      f[w] = sm[hl * NW + w];
      M = fmaxf(M, f[w]);
    }
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float fw = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(f[w] - M);
      const float4 x = reinterpret_cast<const float4*>(so + ((size_t)w * NH + hl) * (KD + 4))[c4];
      a.x += fw * x.x; a.y += fw * x.y; a.z += fw * x.z; a.w += fw * x.w;
      lsum += fw * sl[hl * NW + w];
    }
    const size_t row = (size_t)seq * p.G + head0 + hl;
    if (p.PS == 0) {
      const float inv = 1.0f / lsum;           // (the range holds a position: only logits of -inf alone leave 0, and NaN)
      a.x *= inv; a.y *= inv; a.z *= inv; a.w *= inv;
      reinterpret_cast<float4*>(p.o + row * KD)[c4] = a;
    } else {
      const size_t pidx = row * p.PS + p.slot0 + srange;
      reinterpret_cast<float4*>(p.part_o + pidx * KD)[c4] = a;
      if (c4 == 0) {
        p.part_m[pidx] = M;
        p.part_l[pidx] = lsum;
      }
    }
  }
}

template <typename T, int KD, int HB, int NW>
hipError_t launch_direct(const DecodeParams& p, hipStream_t st) {
  const int HG = (p.G + 16 * HB - 1) / (16 * HB);
  const long long nblocks = (long long)p.nseq * p.S * HG;
  if (nblocks > 0x7fffffffll) return hipErrorNotSupported;
  constexpr size_t lds = merge_floats<KD, HB, NW>() * sizeof(float);
  void (*kern)(DecodeParams, int) = HG == 1 ? decode_direct_kernel<T, KD, HB, NW, true> : decode_direct_kernel<T, KD, HB, NW, false>;
  if (lds > 64 * 1024) {      // once per device and variant
    static bool done[64][2] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (!done[dev][HG == 1]) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      done[dev][HG == 1] = true;
    }
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)nblocks), dim3(NW * 64), lds, st, p, HG);
  return hipGetLastError();
}

template <typename T, int KD>
hipError_t pick_direct(const DecodeParams& p, hipStream_t st) {
  if (p.G > 16) return p.chunk <= 64 ? launch_direct<T, KD, 2, 4>(p, st) : launch_direct<T, KD, 2, 8>(p, st);
  return p.chunk <= 64 ? launch_direct<T, KD, 1, 4>(p, st) : launch_direct<T, KD, 1, 8>(p, st);
}

}  // namespace

bool direct_shape_ok(int k, int v, int is_bf16, int cap) {
  return k == v && (k == 64 || (k == 128 && !is_bf16)) && (long long)cap * k * (is_bf16 ? 2 : 4) < (1ll << 31);      // 31-bit byte offsets
}

// Returns hipErrorNotSupported for shapes this kernel does not cover (the caller then uses the generic one).
hipError_t launch_decode_direct(const DecodeParams& p, int is_bf16, hipStream_t st) {
  if (!direct_shape_ok(p.k, p.v, is_bf16, p.cap) || p.causal_h > 0) return hipErrorNotSupported;
  if (is_bf16) return pick_direct<uint16_t, 64>(p, st);
  return p.k == 128 ? pick_direct<float, 128>(p, st) : pick_direct<float, 64>(p, st);
}

}  // namespace mqa
