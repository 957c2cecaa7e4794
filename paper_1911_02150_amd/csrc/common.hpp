// Shared declarations of the gfx950 decode library: kernel parameter blocks and
// the host-side launchers each .hip file exports to the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace mqa {

constexpr int kMaxSplits = 64;          // upper bound on position ranges per sequence a caller can ask for
constexpr int kMaxAutoSplits = 256;     // ... and that the heuristics choose (one sequence alone fills the chip)
constexpr float kLog2e = 1.4426950408889634f;

// One decode launch.  "Sequences" here are KV groups: a multi-query call has
// nseq = b groups of G = h heads; a multi-head call has nseq = b*h groups of
// G = 1 head, and lens is indexed by seq / lens_div (lens_div = h).
// What differs between the two caches of a two-segment launch (see DecodeParams).
struct DecodeSegment {
  const void* K;
  const void* V;
  const int32_t* lens;
  int G, cap, chunk, S, HG, slot0, lens_div;
};

struct DecodeParams {
  const float* q;        // [nseq, G, k]
  const void* K;         // [nseq, cap, k]
  const void* V;         // [nseq, cap, v]
  const int32_t* lens;   // [nseq / lens_div]
  const int32_t* order;  // MFMA kernel: null, or a permutation of the groups, longest first (scheduling only)
  float* o;              // [nseq, G, v]
  // Partial softmax states, one per (row, slot): row = seq*G + head over the whole call,
  // slot = slot0 + range.  PS slots per row; PS = 0 means "no partials: write o directly".
  float* part_o;         // [nseq*G, PS, v]  un-normalised partial outputs
  float* part_m;         // [nseq*G, PS]     running maxima (log2 domain)
  float* part_l;         // [nseq*G, PS]     sums of 2^(logit - max)
  int PS, slot0;
  int nseq, G, cap, lens_div;
  int k, v;
  int window;            // > 0: attend only to the last `window` valid positions (0 = all)
  int causal_h;          // > 0 (MFMA kernel): the G rows of a group are n = G/causal_h consecutive queries
                         // x causal_h heads; query j sits at position L-n+j and sees positions <= its own
  int chunk;             // positions per range (multiple of 32)
  int S;                 // ranges per sequence
  int HG;                // head groups per sequence (MFMA kernel: ceil(G / (16*HB)))
  int merge_alias;       // MFMA kernel: 1 = the wave-merge buffers re-use the q operands' LDS
  int persist;           // MFMA kernel, 64-head form: > 0 = that many workgroups (the grid) each take several ranked
                         // sequences in turn instead of one workgroup per sequence; the ranking is `order`, or, if
                         // that is null, made by every workgroup for itself
  float qscale;          // scale * log2(e): logits are kept in the log2 domain
  // MFMA kernel, two-segment launches only: workgroups [nblocks0, grid) work on seg1 instead of
  // the fields above (same q, o and partial-state rows)
  int nblocks0;
  DecodeSegment seg1;
  __host__ __device__ DecodeSegment seg0() const { return DecodeSegment{K, V, lens, G, cap, chunk, S, HG, slot0, lens_div}; }
#ifdef MQA_TIMELINE
  long long* timeline;   // debug builds only: [waves][8] wall-clock stamps
#endif
};

// The merge of the partial states.  The slots of a row come from up to two launches
// ("segments": e.g. the memory shared by the hypotheses of a beam and each hypothesis' own
// rows); a segment wrote slot s only if its range s starts before the row's length there.
struct CombineSegment {
  const int32_t* lens;   // length of row r in this segment: lens[r / rows_per_len]
  int rows_per_len;
  int cap, window, chunk, S;
};
struct CombineParams {
  const float* part_o;   // [rows, PS, v]
  const float* part_m;   // [rows, PS]
  const float* part_l;   // [rows, PS]
  float* o;              // [rows, v]
  long long rows;
  int v, PS, nseg;
  CombineSegment seg[2]; // segment 0 owns slots [0, seg[0].S), segment 1 the next seg[1].S
};

struct Tuning {
  int splits = 0;
  int kernel = 0;
  int flags = 0;
};

// decode_mfma.hip: bf16 cache, k = v = 128; 16 or 32 heads per workgroup.
bool mfma_shape_ok(int G, int k, int v, int is_bf16, int cap);
int mfma_heads_per_block(int G, int flags, int causal);
int mfma_persistent_workgroups(int nseq, int G, int S, int HG, int window, int causal, int flags, int* inline_rank);
hipError_t launch_decode_mfma(const DecodeParams& p, int flags, hipStream_t st);
// both segments in one launch (p.seg1 filled in, 32 heads per workgroup in both); p.order must be null
hipError_t launch_decode_mfma_two(const DecodeParams& p, long long nblocks0, long long nblocks1, hipStream_t st);

// prompt_mfma.hip: causal rows, bf16 cache, k = v = 128, p.HG blocks of 128 rows per group
hipError_t launch_prompt(const DecodeParams& p, hipStream_t st);

// decode_direct.hip: k = v = 64 or 128 in float32, 64 in bf16 (hipErrorNotSupported: another shape).
bool direct_shape_ok(int k, int v, int is_bf16, int cap);
hipError_t launch_decode_direct(const DecodeParams& p, int is_bf16, hipStream_t st);

// decode_generic.hip: any k, v <= 256, float32 or bf16 cache.
hipError_t launch_decode_generic(const DecodeParams& p, int is_bf16, hipStream_t st);

// small_kernels.hip
hipError_t launch_combine(const CombineParams& p, hipStream_t st);
hipError_t launch_length_order(const int32_t* lens, int lens_div, int nseq, int cap, int32_t* order, hipStream_t st);
constexpr int kMaxOrdered = 1 << 16;      // groups the single-workgroup length ranking handles
hipError_t launch_reorder(const void* K_src, const void* V_src, const int32_t* lens_src, const int32_t* parent,
                          void* K_dst, void* V_dst, int32_t* lens_dst, int n, int h_kv, int cap,
                          size_t k_row_bytes, size_t v_row_bytes, hipStream_t st);
hipError_t launch_append(void* K, void* V, const float* k_new, const float* v_new, int32_t* lens,
                         int b, int h_kv, int cap, int k, int v, int n, int is_bf16, hipStream_t st);
hipError_t launch_stream_read(const void* src, size_t bytes, float* sink, hipStream_t st);
hipError_t launch_stream_copy(const void* src, void* dst, size_t bytes, hipStream_t st);

// project.hip
// epilogue: 0 store, 1 store max(x, 0), 2 add to what out holds
hipError_t launch_project(int mode, const float* in, const float* P, float* out,
                          int rows, int d, int h, int kv, int epilogue, hipStream_t st);

// gemm.hip: the same GEMM for large row counts / wide outputs (hipErrorNotSupported: too small, use launch_project's own kernel)
int gemm_form(int mode, int rows, int d, int h, int kv, int apart);      // the edge of its tiles; 0: not this kernel
bool gemm_fits(bool outp, int d, int h, int kv, int edge);               // do its 32-bit offsets inside a tile fit?
double gemm_us(bool outp, int rows, int N, int C);                       // its time, or the split-contraction kernel's, by the rule there
hipError_t launch_gemm_parts(int mode, const float* in, const float* P, float* out, int rows, int d, int h, int kv, int epilogue,
                             int edge, int S, hipStream_t st);           // S parts of the contraction, one behind another in `out`
constexpr int kApart = 4;      // `apart` of the fused q/K/V projection, us: a launch of its own for q
hipError_t launch_gemm_tiled(int mode, const float* in, const float* P, float* out,
                             int rows, int d, int h, int kv, int epilogue, int apart, hipStream_t st);
hipError_t launch_project_qkv_append(const float* x, const float* P_q, const float* P_k, const float* P_v,
                                     float* q, void* K, void* V, const int32_t* lens_in, int32_t* lens_out,
                                     int rows, int d, int h, int h_kv, int cap, int k, int v, int is_bf16,
                                     int mem_rows, int append, hipStream_t st);

// project_kv.hip: the new K / V rows of many positions into a bf16 cache (n rows per sequence; append: behind the
// lens_in[] rows already there, else lens_in[] valid rows from position 0 on; hipErrorNotSupported: too few)
bool project_kv_exact_pays(int rows, int d, int h_kv, int k, int v);
hipError_t launch_project_kv_exact(const float* x, const float* P_k, const float* P_v, void* K, void* V,
                                   const int32_t* lens_in, int32_t* lens_out, int rows, int n, int append, int d, int h_kv,
                                   int cap, int k, int v, hipStream_t st);

// project_terms.hip: decode-sized products; tiles of 16 RB x 16 CB, the contraction cut among S workgroups (S = 0: not there;
// parts with RB = CB = 8: gemm.hip's 128 x 128 tiles)
struct TermsForm { int RB, CB, S; };
TermsForm terms_form(bool outp, int rows, int d, int h, int kv);
TermsForm terms_parts_form(bool outp, int rows, int d, int h, int kv);
size_t terms_parts_bytes(bool outp, int rows, int d, int h, int kv);
hipError_t launch_project_terms(bool outp, const float* in, const float* P, float* out, int rows, int d, int h, int kv, int epilogue,
                                hipStream_t st);
hipError_t launch_project_add_layernorm(bool outp, const float* in, const float* P, float* x, float* y, int rows, int d, int h, int kv,
                                        float eps, void* workspace, hipStream_t st);

// project_kv_rows.hip: the same from a workspace of project_kv_rows_workspace(...) bytes (not append: lens_in may be null)
bool project_kv_rows_pays(int rows, int d, int h_kv, int k, int v);
size_t project_kv_rows_workspace(int d, int h_kv, int k, int v);
hipError_t launch_project_kv_rows(const float* x, const float* P_k, const float* P_v, void* K, void* V,
                                  const int32_t* lens_in, int32_t* lens_out, int rows, int n, int append, int d, int h_kv,
                                  int cap, int k, int v, void* workspace, hipStream_t st);

// gemm.hip: a product of two plain matrices in its tiles, and if *only on the device is not 0, or only_rows[i] for the rows 256 i .. 256 i + 255
int gemm_edge(int rows, int N, int C);
hipError_t launch_gemm_if(const int32_t* only, const int32_t* only_rows, int edge, const float* in, const float* P, float* out, int rows, int C, int N, int epilogue,
                          hipStream_t st);

// packed.hip: a stack's feed-forward from packed operands.  bytes: of its workspace, 0 where there is no such form; faster: than the calls it stands for;
// forms and edges: the tiles of its products, and of those in their place where two terms do not hold the values
struct FeedForwardPlan { size_t bytes; int faster, form1, form2, edge1, edge2; };
FeedForwardPlan feed_forward_plan(int rows, int d, int ff);
hipError_t launch_feed_forward(const FeedForwardPlan& f, const float* W1, const float* W2, float* x, int rows, int d, int ff, float eps, void* workspace,
                               hipStream_t st);

// stack_kernels.hip (packed, if: d a multiple of 32 up to 4096)
hipError_t launch_layernorm(const float* x, float* y, int rows, int d, float eps, hipStream_t st);
hipError_t launch_layernorm_packed(const int32_t* flag, int32_t* bad, const float* x, unsigned char* packed, float scale, int rows, int d, float eps, hipStream_t st);
hipError_t launch_layernorm_if(const int32_t* only, const int32_t* only_rows, const float* x, float* y, int rows, int d, float eps, hipStream_t st);
hipError_t launch_embed(const int32_t* tokens, const int32_t* pos, const float* E, const float* P, float* x,
                        int rows, int d, int vocab, int max_pos, hipStream_t st);
hipError_t launch_add(float* a, const float* b, size_t n, hipStream_t st);
hipError_t launch_relu(float* a, size_t n, hipStream_t st);
hipError_t launch_argmax(const float* x, int32_t* out, int rows, int n, hipStream_t st);

// ---------------------------------------------------------------- device helpers
// First position a sequence of length L attends to, and the 32-aligned position its ranges start from.
__device__ __forceinline__ int window_lo(int L, int window) { return window > 0 ? max(0, L - window) : 0; }
__device__ __forceinline__ int window_base(int L, int window) { return window_lo(L, window) & ~31; }

// Workgroups go to the eight XCDs in turn: the column tile of workgroup x of a row of them, such that neighbouring tiles
// (that share cache lines of weights with n contiguous) are on one XCD and every XCD has a run of them.  For tiles of 16
// columns, half a line: 1024 x 4096, 1 row: 8.3 -> 7.0 us, 8: 8.5 -> 8.0; multi-head q/K/V of one row 7.8 -> 6.6.  Wider tiles are better spread
// (project_terms.hip, 128 rows: 15.0 / 15.7).
__device__ __forceinline__ int column_tile(int x, int tiles) { return tiles % 8 ? x : x % 8 * (tiles / 8) + x / 8; }

// what a GEMM does with a finished output element (see launch_project)
__device__ __forceinline__ float apply_epilogue(float x, const float* dst, int epilogue) {
  if (epilogue == 1) return fmaxf(x, 0.f);
  if (epilogue == 2) return x + *dst;
  return x;
}

__device__ __forceinline__ float bf16_bits_to_float(uint32_t bits16) {
  return __uint_as_float(bits16 << 16);
}

// float32 -> bf16 bits, round to nearest even; NaN stays NaN (quiet).
__device__ __forceinline__ uint32_t float_to_bf16_rne(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

// two floats -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16_pair(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, b2));
}

// A pair of floats as two packed fp16 pairs whose sums are nearly the floats: each term is the nearest
// fp16 of what the terms before it leave (the difference is exact).  The floats are scaled beforehand:
// below 2^-2 the second term loses bits, above 65504 the first overflows.
struct Split2 { uint32_t hi, lo; };
__device__ __forceinline__ Split2 split2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) _Float16 h2;
  Split2 s;
  s.hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a, b}, h2));
  asm("" : "+v"(s.hi));            // (the two halves are read from the packed register, not rounded once more each)
  const h2 h = __builtin_bit_cast(h2, s.hi);
  s.lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{a - (float)h[0], b - (float)h[1]}, h2));
  return s;
}
// The power of two that takes `most` to [2^top, 2^(top + 1)), and the exponent that takes it back.
__device__ __forceinline__ float split_scale(float most, int top) {
  return __uint_as_float((uint32_t)min(254, 254 + top - (int)(__float_as_uint(most) >> 23)) << 23);
}
__device__ __forceinline__ int split_exponent(float scale) { return 127 - (int)(__float_as_uint(scale) >> 23); }

// Four neighbouring values of a layernorm's row, and where they go in a packed matrix of `rows` lines (packed.hip).
__device__ __forceinline__ void store_packed4(unsigned char* packed, float scale, int rows, int row, int column, float a, float b, float c, float d) {
  const Split2 s = split2(a * scale, b * scale), t = split2(c * scale, d * scale);
  unsigned char* at = packed + ((size_t)(column >> 5) * 2 * rows + row) * 64 + (column & 31) * 2;
  *reinterpret_cast<uint2*>(at) = make_uint2(s.hi, t.hi);
  *reinterpret_cast<uint2*>(at + (size_t)rows * 64) = make_uint2(s.lo, t.lo);
}

// A row's values in two fp16 terms, by gemm.hip's measure (`holds`): few octets (eight neighbouring values; none of up to 7 with any but zeros, 2 and an
// eighth of more) have one below kFull, which the terms cut off at 2^-25 of 1, and if one has, some value is from kFarAbove on
constexpr float kFull = 0.0625f, kFarAbove = 128.f;
__device__ __forceinline__ bool row_holds(int small, int octets, int far) { return small <= (octets < 8 ? 0 : 2 + octets / 8) && (small == 0 || far > 0); }

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  return x;
}

}  // namespace mqa
