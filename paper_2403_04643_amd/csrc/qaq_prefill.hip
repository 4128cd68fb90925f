// Prompt encoding: the last n causal score rows of a prompt, from the unquantized fp16
// keys, installed as the attention window (Section 2.1 prompt encoding; Section 4.2
// "attention window").
//
// Per KV head this is a dense contraction [G*n query rows x D] . [D x T keys], so it runs on
// the fp16 matrix instruction (fp32 accumulation; products of fp16 numbers are exact in
// fp32).  k_prefill_logits reads every key once: a wavefront keeps 64 keys in registers as B
// operands and sweeps the query rows of the head over them in blocks of 16.  It leaves
// logit/sqrt(D) (minus infinity where a token lies after the query's position) in the score
// buffer, and for every query row the maximum and the sum of exponentials over its 64 keys;
// k_prefill_softmax merges these, turns each row into scores in place and writes the maximum
// over the query heads of a KV head into the ring rows.
#include "qaq_internal.h"

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int kThreads = 256;
constexpr int kChunk = 64;         // keys per wavefront of the logits kernel = tokens per (maximum, sum) pair
constexpr int kShare = 4;          // tokens per thread of the softmax kernel

// tokens a query row attends to: row i belongs to position T - n + i of a prompt of T tokens
__device__ __forceinline__ int row_length(int T, int n, int i) { return T - n + i + 1; }

// The (maximum, sum) pairs of score row i of (sequence, query head) bq: NT tiles x 4 pairs.  They lie where
// the attention call keeps its partial results (D + 4 floats per tile and query head; 8 rows x 4 x 2
// are at most 64), which nobody needs while a prompt is encoded.
__device__ __forceinline__ float2* row_pairs(const QaqView& v, int bq, int i) {
  static_assert(QAQ_MAX_WINDOW * (QAQ_TT / kChunk) * 2 <= 64 + 4, "the pairs fit the attention call's partials");
  return (float2*)(v.partial + (size_t)bq * v.NT * (v.D + 4)) + (size_t)i * v.NT * (QAQ_TT / kChunk);
}

// maximum / sum over the 16 lanes of a row, in every one of them
__device__ __forceinline__ float row16_max(float x) {
  asm volatile(QAQ_DPP_STEP("v_max_f32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_f32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_f32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_max_f32_dpp", "row_mirror row_mask:0xf bank_mask:0xf")
               "s_nop 1"
               : "+v"(x));
  return x;
}
__device__ __forceinline__ float row16_sum(float x) {
  asm volatile(QAQ_DPP_STEP("v_add_f32_dpp", "quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_add_f32_dpp", "quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_add_f32_dpp", "row_half_mirror row_mask:0xf bank_mask:0xf")
               QAQ_DPP_STEP("v_add_f32_dpp", "row_mirror row_mask:0xf bank_mask:0xf")
               "s_nop 1"
               : "+v"(x));
  return x;
}

template <int D>
__global__ __launch_bounds__(kThreads) void k_prefill_logits(QaqPrefillArgs a) {
  constexpr int NS = D / 32;       // matrix instructions along the head dimension
  const QaqView& v = a.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int col = lane & 15, kb = lane >> 4;
  const int bh = blockIdx.x, b = bh / v.Hkv, h = bh % v.Hkv;     // heads fastest (see k_build)
  const int t_wave = blockIdx.y * QAQ_TT + 64 * wave;
  if (t_wave >= a.T) return;
  const int T_seq = qaq_seq_len(v, b, a.T);      // tokens of this sequence's prompt (rows of K past them are padding)

  // 64 keys of this wavefront: lane (col, kb) holds channels 32s + 8kb .. +8 of key 16g + col
  h8 key[4][NS];
  const __half* kbase = a.k + (size_t)bh * a.T * D;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int t = min(t_wave + 16 * g + col, a.T - 1);    // clamped: the tail reads a valid row and is masked below
#pragma unroll
    for (int s = 0; s < NS; ++s) key[g][s] = __builtin_nontemporal_load((const h8*)(kbase + (size_t)t * D + 32 * s + 8 * kb));
  }

  const int R = a.G * a.n_rows;    // query rows of this KV head: (query head g, prompt row i) -> g * n + i
  const float scale = rsqrtf((float)D);
  for (int r0 = 0; r0 < R; r0 += 16) {
    h8 qa[NS];
    {
      const int r = r0 + col;
      const bool live = r < R;
      const int hq = h * a.G + (live ? r / a.n_rows : 0), i = live ? r % a.n_rows : 0;
      const __half* qrow = a.q + (((size_t)b * v.Hq + hq) * a.n_rows + i) * D;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        qa[s] = *(const h8*)(qrow + 32 * s + 8 * kb);
        if (!live) qa[s] = (h8)(_Float16)0;
      }
    }
    f4 acc[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      acc[g] = (f4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < NS; ++s) acc[g] = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], key[g][s], acc[g], 0, 0, 0);
    }
    // element j of a result: query row 4kb + j of the block, key `col` of group g
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int r = r0 + 4 * kb + j;
      const int rc = min(r, R - 1);
      const int hq = h * a.G + rc / a.n_rows, i = rc % a.n_rows;
      const int len = row_length(T_seq, a.n_rows, i);
      float* row = a.scores + (((size_t)i * v.B + b) * v.Hq + hq) * a.T;
      float x[4], m = -INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int t = t_wave + 16 * g + col;
        x[g] = t < len ? acc[g][j] * scale : -INFINITY;
        m = fmaxf(m, x[g]);
        if (r < R && t < a.T) row[t] = x[g];
      }
      m = row16_max(m);
      float l = 0.0f;
      if (m > -INFINITY) {
#pragma unroll
        for (int g = 0; g < 4; ++g) l += expf(x[g] - m);        // exp(-inf) = 0 past the row's end
      }
      l = row16_sum(l);
      if (col == 0 && r < R) row_pairs(v, b * v.Hq + hq, i)[t_wave / kChunk] = make_float2(m, l);
    }
  }
}

// Softmax of the score rows in place, and the ring rows: one workgroup per (share of 4 x 256 tokens,
// prompt row, (sequence, KV head)), for all G query heads of the KV head, so that the ring entry --
// the maximum over them -- is written once.  Every workgroup merges the heads' (maximum, sum) pairs for
// itself (a wavefront per head, 8 bytes per 64 tokens, from the L2).  Bound by HBM: a score is read
// and written once.  Before, one workgroup took the whole row, head after head, and read what exceeded 4096
// tokens three times: 16 x 64 heads, 8192 tokens, 5 rows 256 us, now 60; 8 x 32 heads, 4096 tokens
// 18 -> 16 us; 2 x 32 heads, 12001 tokens 37 -> 14 us.
constexpr int kMaxMergeHeads = 16;         // query heads merged per pass over the pairs (more: further passes)
__global__ __launch_bounds__(kThreads) void k_prefill_softmax(QaqPrefillArgs a) {
  __shared__ float s_m[kMaxMergeHeads], s_l[kMaxMergeHeads];
  const QaqView& v = a.v;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bh = blockIdx.x, b = bh / v.Hkv, h = bh % v.Hkv;      // heads fastest (see k_build)
  const int i = blockIdx.z;
  const int len = row_length(qaq_seq_len(v, b, a.T), a.n_rows, i);
  const int n_pair = (a.T + kChunk - 1) / kChunk;
  const int t0 = blockIdx.y * (kShare * kThreads) + tid;
  float best[kShare];
#pragma unroll
  for (int k = 0; k < kShare; ++k) best[k] = 0.0f;
  for (int g0 = 0; g0 < a.G; g0 += kMaxMergeHeads) {
    const int ng = min(a.G - g0, kMaxMergeHeads);
    if (g0) __syncthreads();
    for (int g = wave; g < ng; g += 4) {
      const float2* pairs = row_pairs(v, b * v.Hq + h * a.G + g0 + g, i);
      float m = -INFINITY, l = 0.0f;
      for (int p = lane; p < n_pair; p += 64) {
        const float2 x = pairs[p];
        if (x.x > -INFINITY) {
          const float mm = fmaxf(m, x.x);
          l = l * expf(m - mm) + x.y * expf(x.x - mm);
          m = mm;
        }
      }
      const float M = wave_max(m);
      const float Lw = wave_sum(m > -INFINITY ? l * expf(m - M) : 0.0f);
      if (lane == 0) { s_m[g] = M; s_l[g] = Lw; }
    }
    __syncthreads();
#pragma unroll 2
    for (int g = 0; g < ng; ++g) {
      float* row = a.scores + (((size_t)i * v.B + b) * v.Hq + (h * a.G + g0 + g)) * a.T;
      const float m = s_m[g], l = s_l[g];
      float x[kShare];
#pragma unroll
      for (int k = 0; k < kShare; ++k) {
        const int t = t0 + k * kThreads;
        x[k] = t < len ? row[t] : -INFINITY;
      }
#pragma unroll
      for (int k = 0; k < kShare; ++k) {
        const int t = t0 + k * kThreads;
        const float s = t < len ? expf(x[k] - m) / l : 0.0f;
        if (t < a.T) row[t] = s;
        best[k] = fmaxf(best[k], s);
      }
    }
  }
  const size_t ring0 = (size_t)i * ((size_t)v.B * v.Hkv * v.Tmax) + qaq_bh(v, b, h) * v.Tmax;
#pragma unroll
  for (int k = 0; k < kShare; ++k) {
    const int t = t0 + k * kThreads;
    if (t < len) qaq_ring_store(v, ring0 + t, best[k]);
  }
}

}  // namespace

hipError_t qaq_launch_prefill_window(const QaqPrefillArgs& a, hipStream_t s) {
  const QaqView& v = a.v;
  const dim3 grid(v.B * v.Hkv, (a.T + QAQ_TT - 1) / QAQ_TT);
  if (v.D == 128) hipLaunchKernelGGL(k_prefill_logits<128>, grid, dim3(kThreads), 0, s, a);
  else if (v.D == 64) hipLaunchKernelGGL(k_prefill_logits<64>, grid, dim3(kThreads), 0, s, a);
  else return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int share = kShare * kThreads;
  hipLaunchKernelGGL(k_prefill_softmax, dim3(v.B * v.Hkv, (a.T + share - 1) / share, a.n_rows), dim3(kThreads), 0, s, a);
  return hipGetLastError();
}
