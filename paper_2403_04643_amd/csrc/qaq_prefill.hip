// Prompt encoding: the last n causal score rows of a prompt, from the unquantized fp16
// keys, installed as the attention window (Section 2.1 prompt encoding; Section 4.2
// "attention window").
//
// Per KV head this is a dense contraction [G*n query rows x D] . [D x T keys], so it runs on
// the fp16 matrix instruction (fp32 accumulation; products of fp16 numbers are exact in
// fp32).  k_prefill_logits reads every key once: a wavefront keeps 64 keys in registers as B
// operands and sweeps the query rows of the head over them in blocks of 16.  It leaves
// logit/sqrt(D) (minus infinity where a token lies after the query's position) in the score
// buffer; k_prefill_softmax turns each row into scores in place and, where a KV head has one query head,
// fills the window's rows; where it has several, k_prefill_ring writes their maximum there.
#include "qaq_internal.h"

namespace {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4 __attribute__((ext_vector_type(4)));
constexpr int kThreads = 256;
constexpr int kShare = 4;          // tokens per thread of the kernel that fills the window's rows

// tokens a query row attends to: row i belongs to position T - n + i of a prompt of T tokens
__device__ __forceinline__ int row_length(int T, int n, int i) { return T - n + i + 1; }

__device__ __forceinline__ float block_reduce(float x, bool is_max, float* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const float y = __shfl_xor(x, o);
    x = is_max ? fmaxf(x, y) : x + y;
  }
  __syncthreads();                 // red[] may still be read from the previous reduction
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  return is_max ? fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])) : (red[0] + red[1]) + (red[2] + red[3]);
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
    // (plain loads: the prompt's append reads the keys again, as far as the last-level cache has kept them; as streaming
    // loads window and append of 2 x 32 heads x 12001 tokens take 176 us, so 166; 8 x 32 x 4096 227 and 220)
#pragma unroll
    for (int s = 0; s < NS; ++s) key[g][s] = *(const h8*)(kbase + (size_t)t * D + 32 * s + 8 * kb);
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
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < NS; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(qa[s], key[g][s], acc, 0, 0, 0);
      const int t = t_wave + 16 * g + col;
      if (t < a.T) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {      // element j of the result: query row 4kb + j of the block, key `col`
          const int r = r0 + 4 * kb + j;
          if (r < R) {
            const int hq = h * a.G + r / a.n_rows, i = r % a.n_rows;
            a.scores[(((size_t)i * v.B + b) * v.Hq + hq) * a.T + t] =
                t < row_length(T_seq, a.n_rows, i) ? acc[j] * scale : -INFINITY;
          }
        }
      }
    }
  }
}

// Softmax of the score rows in place: one workgroup per (query head, prompt row).  Bound by HBM: a thread keeps its
// logits -- every 256th of the row -- in registers, KEEP of them: 16 and 32 for many rows of up to 4096 and 8192 tokens, so
// that a score is read once and written once; 64 for rows of more than 32768, whose others are read again, for the sum and for
// the scores (what lies between: the wide form below).  The sum's order is part of what the scores are to the last bit:
// a score that decides a width must not depend on how a row is shared out.  Before, one workgroup took the rows of all
// G heads one after the other, with 16 logits in registers: 16 x 64 heads, 8192 tokens, 5 rows 256 us, now 59 (and 27 for
// the window's rows); 8 x 32 heads, 4096 tokens 18 -> 13.
template <int KEEP>
__global__ __launch_bounds__(kThreads) void k_prefill_softmax(QaqPrefillArgs a) {
  __shared__ float red[4];
  const QaqView& v = a.v;
  const int tid = threadIdx.x;
  const int bq = blockIdx.x, b = bq / v.Hq, i = blockIdx.y;      // heads fastest (see k_build)
  const int len = row_length(qaq_seq_len(v, b, a.T), a.n_rows, i);
  float* row = a.scores + ((size_t)i * v.B * v.Hq + bq) * a.T;
  float mine[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int t = tid + k * kThreads;
    mine[k] = t < len ? row[t] : -INFINITY;
  }
  float m = -INFINITY;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) m = fmaxf(m, mine[k]);
  for (int t = tid + KEEP * kThreads; t < len; t += kThreads) m = fmaxf(m, row[t]);
  m = block_reduce(m, true, red);
  float l = 0.0f;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    mine[k] = expf(mine[k] - m);                    // exp(-inf) = 0 past the row's end
    l += mine[k];
  }
  for (int t = tid + KEEP * kThreads; t < len; t += kThreads) l += expf(row[t] - m);
  l = block_reduce(l, false, red);
  const bool ring = a.G == 1;                       // (else the maximum over the heads goes there: k_prefill_ring)
  const size_t ring0 = (size_t)i * ((size_t)v.B * v.Hkv * v.Tmax) + (size_t)bq * v.Tmax;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int t = tid + k * kThreads;
    if (t < a.T) {
      const float s = t < len ? mine[k] / l : 0.0f;
      row[t] = s;
      if (ring && t < len) qaq_ring_store(v, ring0 + t, s);
    }
  }
  for (int t = tid + KEEP * kThreads; t < a.T; t += kThreads) {
    const float s = t < len ? expf(row[t] - m) / l : 0.0f;
    row[t] = s;
    if (ring && t < len) qaq_ring_store(v, ring0 + t, s);
  }
}

// The same for rows that are long or few: sixteen wavefronts per row.  Four leave most of the chip idle where rows are few, compute
// every exponential of a row on four SIMDs, and read again what their registers do not hold of rows of more than 16384 tokens (figures: see
// the launcher).  Rows of up to 8192, 16384 and 20464 tokens take 8, 16 and 20 logits per thread, so that two rows share a compute
// unit; longer ones 32, a compute unit each.  The exponentials go through LDS so that
// their sum keeps the order it has there: thread j adds every 256th from the j-th on, then the four wavefronts' sums.
constexpr int kWide = 1024, kWideMost = 32;       // threads, most logits of each: rows up to 32768 tokens, 128 KB of LDS
constexpr int kWideTwo = (160 * 1024 / 2 - 64) / 4;       // longest row of which a compute unit's LDS holds two: 20464 tokens, 20 logits per thread
template <int KEEP>
__global__ __launch_bounds__(kWide, (KEEP <= 20 ? 8 : 4)) void k_prefill_softmax_wide(QaqPrefillArgs a) {
  extern __shared__ float e_row[];                // [T]
  __shared__ float red[kWide / 64];
  const QaqView& v = a.v;
  const int tid = threadIdx.x;
  const int bq = blockIdx.x, b = bq / v.Hq, i = blockIdx.y;
  const int len = row_length(qaq_seq_len(v, b, a.T), a.n_rows, i);
  float* row = a.scores + ((size_t)i * v.B * v.Hq + bq) * a.T;
  float mine[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int t = tid + k * kWide;
    mine[k] = t < len ? row[t] : -INFINITY;
  }
  float m = -INFINITY;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) m = fmaxf(m, mine[k]);
  m = wave_max(m);
  if ((tid & 63) == 0) red[tid >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWide / 64; ++w) m = fmaxf(m, red[w]);
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int t = tid + k * kWide;
    if (t >= len) break;
    mine[k] = expf(mine[k] - m);
    e_row[t] = mine[k];
  }
  __syncthreads();                                // (red[] has been read, too)
  if (tid < kThreads) {
    float l = 0.0f;
#pragma unroll 8
    for (int t = tid; t < len; t += kThreads) l += e_row[t];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) l += __shfl_xor(l, o);
    if ((tid & 63) == 0) red[tid >> 6] = l;
  }
  __syncthreads();
  const float l = (red[0] + red[1]) + (red[2] + red[3]);
  const bool ring = a.G == 1;
  const size_t ring0 = (size_t)i * ((size_t)v.B * v.Hkv * v.Tmax) + (size_t)bq * v.Tmax;
#pragma unroll
  for (int k = 0; k < KEEP; ++k) {
    const int t = tid + k * kWide;
    if (t >= a.T) break;
    const float s = t < len ? mine[k] / l : 0.0f;
    row[t] = s;
    if (ring && t < len) qaq_ring_store(v, ring0 + t, s);
  }
}

// Grouped queries: the window's rows, the maximum of the scores over the G query heads of a KV head (what the kernel
// before has just written: from the last-level cache).
__global__ __launch_bounds__(kThreads) void k_prefill_ring(QaqPrefillArgs a) {
  const QaqView& v = a.v;
  const int bh = blockIdx.x, b = bh / v.Hkv, h = bh % v.Hkv, i = blockIdx.z;
  const int len = row_length(qaq_seq_len(v, b, a.T), a.n_rows, i);
  const float* row = a.scores + (((size_t)i * v.B + b) * v.Hq + h * a.G) * a.T;
  const size_t ring0 = (size_t)i * ((size_t)v.B * v.Hkv * v.Tmax) + qaq_bh(v, b, h) * v.Tmax;
  for (int k = 0; k < kShare; ++k) {
    const int t = (blockIdx.y * kShare + k) * kThreads + threadIdx.x;
    if (t >= len) return;
    float s = 0.0f;                                 // probabilities: >= 0
#pragma unroll 8
    for (int g = 0; g < a.G; ++g) s = fmaxf(s, row[(size_t)g * a.T + t]);
    qaq_ring_store(v, ring0 + t, s);
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
  const dim3 rows(v.B * v.Hq, a.n_rows), block(kThreads);
  // Which form: sixteen wavefronts per row where the rows are few (two per compute unit) or long, four where there are many of
  // up to 8192 tokens.  Logits and scores of 64 channels, five rows per head, us, four | sixteen: 1 x 8 heads x 2000 tokens 9.2 | 8.7,
  // 1 x 32 x 3000 11.9 | 10.7, 2 x 50 x 6000 29.5 | 26.9, 8 x 32 x 4000 38.2 | 40.6, 4 x 32 x 8000 40.4 | 40.8, 16 x 64 x 8192
  // 163.1 | 166.7, x 12000 261 | 233, 2 x 32 x 12001 37.8 | 32.5, 8 x 32 x 9000 110.8 | 99.2, 1 x 32 x 32000 94 | 43.  Short rows, 128
  // channels: 1 x 32 x 64 7.4 | 6.7, x 512 8.8 | 8.2, 3 x 32 x 100 8.4 | 7.8, x 500 9.6 | 9.2, 1 x 8 x 1 token and row 5.7 | 4.9.
  // Past 16384 tokens, 128 channels, four | sixteen with a compute unit per row | sixteen with two rows on one (as far as its LDS holds
  // two): 16 x 64 heads on 8 x 16385 465 | 482 | 451, x 20464 664 | 561 | 541, 1 x 64 on 8 x 16640, 8 rows 51.0 | 52.6 | 48.1,
  // 8 x 32 x 17400 336 | 332 | 325, 1 x 32 x 16385 42.4 | 36.2 | 36.1.
  const bool wide = a.T <= kWide * kWideMost && (a.T > 32 * kThreads || (long long)rows.x * rows.y <= 2ll * qaq_compute_units());
  const size_t row_bytes = (size_t)a.T * sizeof(float);
  if (wide && a.T <= 8 * kWide) hipLaunchKernelGGL(k_prefill_softmax_wide<8>, rows, dim3(kWide), row_bytes, s, a);
  else if (wide && a.T <= 16 * kWide) hipLaunchKernelGGL(k_prefill_softmax_wide<16>, rows, dim3(kWide), row_bytes, s, a);
  else if (wide && a.T <= kWideTwo) hipLaunchKernelGGL(k_prefill_softmax_wide<20>, rows, dim3(kWide), row_bytes, s, a);
  else if (wide) hipLaunchKernelGGL(k_prefill_softmax_wide<kWideMost>, rows, dim3(kWide), row_bytes, s, a);
  else if (a.T <= 16 * kThreads) hipLaunchKernelGGL(k_prefill_softmax<16>, rows, block, 0, s, a);
  else if (a.T <= 32 * kThreads) hipLaunchKernelGGL(k_prefill_softmax<32>, rows, block, 0, s, a);
  else hipLaunchKernelGGL(k_prefill_softmax<64>, rows, block, 0, s, a);
  e = hipGetLastError();
  if (e != hipSuccess || a.G == 1) return e;
  const int share = kShare * kThreads;
  hipLaunchKernelGGL(k_prefill_ring, dim3(v.B * v.Hkv, (a.T + share - 1) / share, a.n_rows), block, 0, s, a);
  return hipGetLastError();
}
