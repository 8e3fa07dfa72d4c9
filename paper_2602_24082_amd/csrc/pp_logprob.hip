// Per-response log-probabilities and the ranked-pair DPO / Bradley-Terry loss.
//
// The DPO reward of Sec. 2.1 is built from sequence log-probabilities
// log pi(y|x) = sum_t log softmax(logits_{t-1})[y_t].  In a packed row (Sec. 3.2)
// the first token of every response is predicted by the last prompt position,
// the others by the position before them.  Kernels:
//
//   logprob_rows   one workgroup per needed logit row: one streaming pass over
//                  the vocabulary for (max, sum exp), then the label logits
//                  -> tok[label position] = logit[label] - logsumexp
//                  (HBM-bound: reads each needed logit row once)
//   logprob_bwd    one workgroup per flat logit row: the gradient of the
//                  weighted response sums, -c softmax + label terms, zeros for
//                  rows that predict nothing (HBM-bound: one read of the needed
//                  rows, one write of every row)
//   segsum         one wave per (row, response) slot: fixed-order sum of the
//                  response's token log-probs -> seq[b, k]
//   pair_loss      one workgroup: z = beta (pol - ref), softplus over ranked
//                  pairs, per-row mean, mean over rows, closed-form gradient.

#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "pp_device.h"
#include "pp_launch.h"

namespace pp {
namespace {

// threads per log-prob workgroup (one workgroup per logit row: 1024 threads
// with 4 vectors each keep 64 KB of the row in flight) and 16-byte vectors in
// flight per thread
#ifndef PP_LP_THREADS
#define PP_LP_THREADS 1024
#endif
#ifndef PP_LP_UNROLL
#define PP_LP_UNROLL 4
#endif
constexpr int kLpThreads = PP_LP_THREADS;
constexpr int kLpUnroll = PP_LP_UNROLL;  // 16-byte vectors in flight per thread per step

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The larger of two, NaN if either is: a NaN logit makes its row's maximum NaN, and so
// its sum (fmaxf would pass over it).
__device__ __forceinline__ float max_or_nan(float a, float b) { return __builtin_elementwise_maximum(a, b); }

// Online (max, sum 2^(x*log2e - m*log2e)) accumulator.
struct MaxSum {
  float m;  // running max of x (natural units)
  float s;  // sum of exp(x - m)
};

__device__ __forceinline__ MaxSum combine(MaxSum a, MaxSum b) {
  const float m = max_or_nan(a.m, b.m);
  if (m == kNegInf) return {kNegInf, 0.f};
  return {m, fmaf(a.s, fast_exp2((a.m - m) * kLog2e), b.s * fast_exp2((b.m - m) * kLog2e))};
}

template <typename T>
__device__ __forceinline__ float elem(const T* p, int64_t i);
template <>
__device__ __forceinline__ float elem<__bf16>(const __bf16* p, int64_t i) {
  return (float)p[i];
}
template <>
__device__ __forceinline__ float elem<float>(const float* p, int64_t i) {
  return p[i];
}

// Unpacks one 16-byte vector into floats.
template <typename T>
struct Vec16;
template <>
struct Vec16<__bf16> {
  static constexpr int N = 8;
  __device__ __forceinline__ static void unpack(const u32x4& u, float* f) {
    const uint32_t w[4] = {u[0], u[1], u[2], u[3]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};
template <>
struct Vec16<float> {
  static constexpr int N = 4;
  __device__ __forceinline__ static void unpack(const u32x4& u, float* f) {
    f[0] = __uint_as_float(u[0]);
    f[1] = __uint_as_float(u[1]);
    f[2] = __uint_as_float(u[2]);
    f[3] = __uint_as_float(u[3]);
  }
};

// A logit row of `vocab` elements starting at x as 16-byte vectors: `head`
// elements up to the first 16-byte boundary, `nvec` vectors, and what is left.
// Rows of a vocabulary that is no multiple of a vector's elements start anywhere;
// each of the head and tail elements (fewer than two vectors together) belongs to
// one thread (extra()).
template <typename T>
struct RowSplit {
  static constexpr int N = 16 / (int)sizeof(T);
  int head, nvec, n_extra;
  __device__ __forceinline__ RowSplit(const T* x, int vocab) {
    const int off = (int)(reinterpret_cast<uintptr_t>(x) & 15);
    head = min(vocab, ((16 - off) & 15) / (int)sizeof(T));
    nvec = (vocab - head) / N;
    n_extra = vocab - nvec * N;
  }
  // whether the row starts or ends off a boundary
  __device__ __forceinline__ bool odd() const { return n_extra > 0; }
  // index of the head or tail element of thread tid (valid for tid < n_extra)
  __device__ __forceinline__ int extra(int tid) const { return tid < head ? tid : tid + nvec * N; }
};

// A sum of 2^(x*log2e - ml) with ml = m*log2e rounded is off by the factor of that
// rounding, 2^(m*log2e - ml): up to 1e-6 for logits of 16.  Taken out of the sums of odd
// rows, whose values had a difference each, (x - m)*log2e, while they were summed one by one
// (50257 fp32 values: log-probs off by 5.5e-7 rms either way, 5.7e-7 without this).
__device__ __forceinline__ float exact_base(float s, float m, float ml, bool odd) {
  constexpr float kLn2 = 0.6931471805599453f;
  const float off = odd ? fmaf(m, kLog2e, -ml) * kLn2 : 0.f;
  return fmaf(s, -off, s);
}

// Online (max, sum) over the vectors first + tid, first + tid + THREADS, ... below
// nvec of thread tid, kLpUnroll loads in flight.
template <typename T, int THREADS>
__device__ __forceinline__ MaxSum stream_max_sum(const u32x4* __restrict__ xv, int first, int nvec, bool odd) {
  const int tid = threadIdx.x;
  constexpr int N = Vec16<T>::N;
  MaxSum acc = {kNegInf, 0.f};
  for (int base = first; base < nvec; base += THREADS * kLpUnroll) {
    u32x4 u[kLpUnroll];
#pragma unroll
    for (int j = 0; j < kLpUnroll; ++j) {
      const int vi = base + j * THREADS + tid;
      u[j] = vi < nvec ? __builtin_nontemporal_load(xv + vi) : u32x4{0, 0, 0, 0};
    }
    float f[kLpUnroll * N];
#pragma unroll
    for (int j = 0; j < kLpUnroll; ++j) Vec16<T>::unpack(u[j], f + j * N);
    float mloc = kNegInf;
#pragma unroll
    for (int j = 0; j < kLpUnroll; ++j) {
      const int vi = base + j * THREADS + tid;
      if (vi < nvec) {
#pragma unroll
        for (int e = 0; e < N; ++e) mloc = max_or_nan(mloc, f[j * N + e]);
      }
    }
    const float m = max_or_nan(acc.m, mloc);
    if (m != kNegInf) {
      const float ml = m * kLog2e;
      float s = acc.s * fast_exp2(acc.m * kLog2e - ml);
#pragma unroll
      for (int j = 0; j < kLpUnroll; ++j) {
        const int vi = base + j * THREADS + tid;
        if (vi < nvec) {
#pragma unroll
          for (int e = 0; e < N; ++e) s += fast_exp2(fmaf(f[j * N + e], kLog2e, -ml));
        }
      }
      acc = {m, exact_base(s, m, ml, odd)};
    }
  }
  return acc;
}

// (max, sum) of all the row for any values, with a difference to the maximum so far
// for every element: what a workgroup does again when the fast form below does not
// hold.  Little code, slow and rare.
template <typename T, int THREADS>
__device__ __forceinline__ MaxSum any_max_sum(const u32x4* __restrict__ xv, int nvec) {
  constexpr int N = Vec16<T>::N;
  MaxSum acc = {kNegInf, 0.f};
#pragma unroll 1
  for (int vi = threadIdx.x; vi < nvec; vi += THREADS) {
    float f[N];
    Vec16<T>::unpack(xv[vi], f);
#pragma unroll
    for (int e = 0; e < N; ++e) acc = combine(acc, MaxSum{f[e], 1.f});
  }
  return acc;
}

// A row's logsumexp, lse = m + ln s rounded.
struct RowLse {
  float m, s, lse;
  // exp(x - m) as one fma and one exp2, 2^(x*log2e - m*log2e), needs m*log2e to be
  // finite.  A maximum out there is far: a type's lowest value in every masked entry, as
  // masks are often written, or its largest.  A thread that met nothing but such values
  // makes s infinite or NaN (lowest) or 0 (largest).
  __device__ __forceinline__ bool far() const { return fabsf(m) >= 1e38f && fabsf(m) < __builtin_huge_valf(); }
  __device__ __forceinline__ bool redo() const {
    return fabsf(m) < __builtin_huge_valf() && (far() || !(s < __builtin_huge_valf()));
  }
  // Where m is so large that lse no longer holds ln s, differences to it are formed part
  // by part.
  __device__ __forceinline__ float log_prob(float x) const { return far() ? (x - m) - logf(s) : x - lse; }
  __device__ __forceinline__ float far_softmax(float x) const { return fast_exp2(((x - m) - logf(s)) * kLog2e); }
};

// The workgroup's (max, sum)s combined in a fixed order, for every thread.  `work` is
// run by thread 0 beside the last step.
template <int THREADS, typename Work>
__device__ __forceinline__ RowLse block_lse(MaxSum acc, Work&& work) {
  for (int off = 32; off > 0; off >>= 1) {
    MaxSum o;
    o.m = __shfl_xor(acc.m, off, 64);
    o.s = __shfl_xor(acc.s, off, 64);
    acc = combine(acc, o);
  }
  __shared__ float sm[THREADS / 64], ss[THREADS / 64];
  __shared__ RowLse s_lse;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  if (lane == 0) {
    sm[wave] = acc.m;
    ss[wave] = acc.s;
  }
  __syncthreads();
  if (tid == 0) {
    MaxSum t = {sm[0], ss[0]};
    for (int w = 1; w < THREADS / 64; ++w) t = combine(t, MaxSum{sm[w], ss[w]});
    s_lse = {t.m, t.s, t.m + logf(t.s)};
    work();
  }
  __syncthreads();
  return s_lse;
}

// ln sum_v exp(x[v]) of one logit row, for every thread of a kLpThreads
// workgroup: one streaming pass of aligned 16-byte loads (kLpUnroll in flight per
// thread) keeping an online (max, sum) per thread, the row's head and tail
// elements last, then a fixed-order workgroup combine.  HBM bound.  Rows that
// start on no 16-byte boundary used to be read element by element: 2224 rows of
// 50257 fp32 took 135 us and take 69 us (6.5 TB/s).
template <typename T>
__device__ RowLse row_logsumexp(const T* __restrict__ x, int vocab) {
  const int tid = threadIdx.x;
  const RowSplit<T> rs(x, vocab);
  const float xe = tid < rs.n_extra ? elem<T>(x, rs.extra(tid)) : kNegInf;
  const u32x4* xv = reinterpret_cast<const u32x4*>(x + rs.head);
  MaxSum acc = stream_max_sum<T, kLpThreads>(xv, 0, rs.nvec, rs.odd());
  if (tid < rs.n_extra) acc = combine(acc, MaxSum{xe, 1.f});
  RowLse r = block_lse<kLpThreads>(acc, [] {});
  if (r.redo()) {
    acc = any_max_sum<T, kLpThreads>(xv, rs.nvec);
    if (tid < rs.n_extra) acc = combine(acc, MaxSum{xe, 1.f});
    __syncthreads();
    r = block_lse<kLpThreads>(acc, [] {});
  }
  return r;
}

template <typename T>
__global__ __launch_bounds__(kLpThreads) void logprob_rows_kernel(
    const T* __restrict__ logits, const int32_t* __restrict__ tokens,
    const LogitRowItem* __restrict__ rows, const int32_t* __restrict__ labels,
    float* __restrict__ tok, int vocab) {
  const LogitRowItem it = rows[blockIdx.x];
  const T* x = logits + it.logit_row * (int64_t)vocab;
  const RowLse lse = row_logsumexp<T>(x, vocab);
  for (int j = threadIdx.x; j < it.label_cnt; j += kLpThreads) {
    const int32_t pos = labels[it.label_off + j];
    const int32_t y = tokens[pos];
    tok[pos] = (y >= 0 && y < vocab) ? lse.log_prob(elem<T>(x, y)) : __builtin_nanf("");
  }
}

// Packs floats into one 16-byte vector of T (bf16: round to nearest even).
template <typename T>
struct Pack16;
template <>
struct Pack16<__bf16> {
  __device__ __forceinline__ static u32x4 pack(const float* f) {
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    const f32x8 v = {f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]};
    return __builtin_bit_cast(u32x4, __builtin_convertvector(v, bf16x8));
  }
};
template <>
struct Pack16<float> {
  __device__ __forceinline__ static u32x4 pack(const float* f) {
    return u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
  }
};

// A 16-byte vector of T at any address that is a multiple of T's size (one
// global load or store all the same: the GPU takes unaligned vectors).
template <typename T>
struct __attribute__((packed, aligned(sizeof(T)))) Vec16Any {
  u32x4 v;
};

// Log-prob backward: one workgroup per flat logit row r.  With c = the sum of
// g over the labels that row r predicts,
//   dlogits[r, v] = -c softmax(x_r)[v] + sum_{labels y = v} g,
// the gradient of sum_bk g_bk seq_bk; rows that predict nothing get 0 and a
// label outside the vocabulary makes its row NaN.
//
// The row is held in registers: thread t loads the 16-byte vectors t, t + THREADS,
// ... (R of them), its logsumexp is formed from them (thread maximum, then thread
// sum of exponentials, then a fixed-order workgroup combine), and the gradient is
// computed from the same registers and streamed out, so each row costs one read and
// one write of HBM.  Rows that predict nothing are streamed zeros.
//
// A workgroup first loads, then computes, then stores, so several of them per
// compute unit are what keeps loads and stores in flight together, as far as the
// rows leave registers for them (launch_logprob_bwd picks the shape):
//   512 threads x 8 vectors (4 workgroups): up to 32768 bf16 or 16384 fp32 values,
//   1024 x 8 (2 workgroups): twice that,
//   1024 x 19 (128 VGPRs, one workgroup): 155648 bf16 or 77824 fp32 values, so a
//     152064-entry bf16 vocabulary fits as well as a 128256-entry one; it kept HBM
//     busier than 512 x 40 (0.73 against 0.77 ms on the 8B-shaped batch) and than
//     768 x 27 or 1024 x 20 (both spill).
// 3864 gathered rows of 32000 bf16 values take 92 us (155 us with the 1024 x 19
// shape), 2224 of 50257 bf16 86 us.
//
// OVER: longer rows keep 1024 x 16 vectors and stream the rest twice, the second
// time soon after the first and from the caches (2047 rows of 128256 fp32 values:
// 588 us when all of the row was read twice, 474 us).
//
// EDGE: rows that start on no 16-byte boundary.  The vectors lie on the input
// row's boundaries (so the logsumexp does not depend on where the output goes),
// the stores where the output row has them, and one thread each takes the head
// and tail elements; that costs registers (R 18 instead of 19).  Element by element
// those 2224 rows took 283 us.
template <int R>
__device__ __forceinline__ void opaque(u32x4 (&u)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j) asm volatile("" : "+v"(u[j]));
}

template <typename T, int THREADS, int R, bool EDGE, bool OVER>
__global__ __launch_bounds__(THREADS, R <= 8 ? 8 : 4) void logprob_bwd_kernel(LogprobBwdLaunch a) {
  constexpr int N = Vec16<T>::N;
  const int tid = threadIdx.x;
  const int vocab = a.vocab;
  // dense: workgroup = flat logit row r, output row r; gathered: workgroup =
  // gather record, output row = record index
  const int64_t o_row = blockIdx.x;
  const int item = a.gathered ? (int)blockIdx.x : a.row_item[blockIdx.x];
  const int64_t r = a.gathered ? a.rows[item].logit_row : (int64_t)blockIdx.x;
  if (a.gathered && a.row_index && tid == 0) a.row_index[item] = (int32_t)r;
  T* out = reinterpret_cast<T*>(a.dlogits) + o_row * (int64_t)vocab;
  const T* x = reinterpret_cast<const T*>(a.logits) + r * (int64_t)vocab;
  int head = 0, nvec = vocab / N, n_extra = 0;  // vocab % N == 0 without EDGE
  if constexpr (EDGE) {
    const RowSplit<T> rs(x, vocab);
    head = rs.head;
    nvec = rs.nvec;
    n_extra = rs.n_extra;
  }
  const int xi = tid < head ? tid : tid + nvec * N;  // this thread's head or tail element, if tid < n_extra
  auto store = [&](int vi, const u32x4& v) {
    if constexpr (EDGE) reinterpret_cast<Vec16Any<T>*>(out + head)[vi].v = v;
    else __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out) + vi);
  };
  if (item < 0) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int vi = j * THREADS + tid;
      if (vi < nvec) store(vi, u32x4{0, 0, 0, 0});
    }
    if constexpr (OVER) {
      for (int vi = R * THREADS + tid; vi < nvec; vi += THREADS) store(vi, u32x4{0, 0, 0, 0});
    }
    if (EDGE && tid < n_extra) out[xi] = (T)0.f;
    return;
  }
  const u32x4* xv = reinterpret_cast<const u32x4*>(x + head);
  u32x4 u[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int vi = j * THREADS + tid;
    u[j] = vi < nvec ? __builtin_nontemporal_load(xv + vi) : u32x4{0, 0, 0, 0};
  }
  float xe = kNegInf;
  if (EDGE && tid < n_extra) xe = elem<T>(x, xi);
  const LogitRowItem it = a.rows[item];
  __shared__ int s_y[kMaxRowLabels];
  __shared__ float s_g[kMaxRowLabels];
  __shared__ float s_c;
  __shared__ int s_bad;
  const int cnt = it.label_cnt;
  if (tid == 0) s_bad = 0;
  __syncthreads();
  for (int j = tid; j < cnt; j += THREADS) {
    const int32_t y = a.tokens[a.labels[it.label_off + j]];
    s_y[j] = y;
    s_g[j] = a.dseq[a.label_out[it.label_off + j]];
    if (y < 0 || y >= vocab) s_bad = 1;
  }
  MaxSum over = {kNegInf, 0.f};  // of the vectors past the registers
  if constexpr (OVER) over = stream_max_sum<T, THREADS>(xv, R * THREADS, nvec, n_extra > 0);
  // logsumexp of the row from the registers
  float m = kNegInf;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (j * THREADS + tid < nvec) {
      float f[N];
      Vec16<T>::unpack(u[j], f);
#pragma unroll
      for (int e = 0; e < N; ++e) m = max_or_nan(m, f[e]);
    }
  }
  // the packed vectors count as rewritten here, so each pass below unpacks
  // them again instead of keeping the whole row live as floats
  opaque(u);
  float s = 0.f;
  if (m != kNegInf) {
    const float ml = m * kLog2e;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j * THREADS + tid < nvec) {
        float f[N];
        Vec16<T>::unpack(u[j], f);
#pragma unroll
        for (int e = 0; e < N; ++e) s += fast_exp2(fmaf(f[e], kLog2e, -ml));
      }
    }
    if constexpr (EDGE) s = exact_base(s, m, ml, n_extra > 0);
  }
  MaxSum acc = {m, s};
  if constexpr (OVER) acc = combine(acc, over);
  if (EDGE && tid < n_extra) acc = combine(acc, MaxSum{xe, 1.f});
  RowLse lse = block_lse<THREADS>(acc, [&] {
    float c = 0.f;
    for (int j = 0; j < cnt; ++j) c += s_g[j];
    s_c = c;
  });
  const float c = s_c;
  const float lse2 = lse.lse * kLog2e;
  const bool bad = s_bad != 0;
  auto finish = [&](int vi, float* f) {  // f: the softmax of vector vi
#pragma unroll
    for (int e = 0; e < N; ++e) f[e] *= -c;
    for (int l = 0; l < cnt; ++l) {
      const int d = s_y[l] - (head + vi * N);
      if ((unsigned)d < (unsigned)N) {
#pragma unroll
        for (int e = 0; e < N; ++e) f[e] += (e == d) ? s_g[l] : 0.f;
      }
    }
    if (bad) {
#pragma unroll
      for (int e = 0; e < N; ++e) f[e] = __builtin_nanf("");
    }
    store(vi, Pack16<T>::pack(f));
  };
  auto finish_extra = [&](float softmax) {
    float f = -c * softmax;
    for (int l = 0; l < cnt; ++l) f += s_y[l] == xi ? s_g[l] : 0.f;
    out[xi] = (T)(bad ? __builtin_nanf("") : f);
  };
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(lse.redo() ? 1 : 0), 0)) {
    acc = any_max_sum<T, THREADS>(xv, nvec);
    if (EDGE && tid < n_extra) acc = combine(acc, MaxSum{xe, 1.f});
    __syncthreads();
    lse = block_lse<THREADS>(acc, [] {});
#pragma unroll 1
    for (int vi = tid; vi < nvec; vi += THREADS) {
      float f[N];
      Vec16<T>::unpack(xv[vi], f);
#pragma unroll
      for (int e = 0; e < N; ++e) f[e] = lse.far_softmax(f[e]);
      finish(vi, f);
    }
    if (EDGE && tid < n_extra) finish_extra(lse.far_softmax(xe));
    return;
  }
  auto gradient = [&](int vi, const u32x4& x16) {
    float f[N];
    Vec16<T>::unpack(x16, f);
#pragma unroll
    for (int e = 0; e < N; ++e) f[e] = fast_exp2(fmaf(f[e], kLog2e, -lse2));
    finish(vi, f);
  };
  if constexpr (OVER) {
    for (int base = R * THREADS + tid; base < nvec; base += THREADS * kLpUnroll) {
      u32x4 w[kLpUnroll];
#pragma unroll
      for (int j = 0; j < kLpUnroll; ++j) {
        const int vi = base + j * THREADS;
        w[j] = vi < nvec ? xv[vi] : u32x4{0, 0, 0, 0};
      }
#pragma unroll
      for (int j = 0; j < kLpUnroll; ++j)
        if (base + j * THREADS < nvec) gradient(base + j * THREADS, w[j]);
    }
  }
  opaque(u);
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int vi = j * THREADS + tid;
    if (vi < nvec) gradient(vi, u[j]);
  }
  if (EDGE && tid < n_extra) finish_extra(fast_exp2(fmaf(xe, kLog2e, -lse2)));
}

// One wave per (row, response) slot; lane l sums tokens l, l+64, ... in order,
// then a fixed butterfly, so the result does not depend on scheduling.
__global__ __launch_bounds__(256) void segsum_kernel(const float* __restrict__ tok,
                                                      const RespItem* __restrict__ resp,
                                                      float* __restrict__ seq, int n_resp) {
  const int w = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (w >= n_resp) return;
  const RespItem r = resp[w];
  float s = 0.f;
  for (int j = lane; j < r.len; j += 64) s += tok[r.tok_begin + j];
  s = wave_sum(s);
  if (lane == 0) seq[r.out] = s;
}

__device__ __forceinline__ float softplus_f(float x) {
  // ln(1 + e^x) without overflow
  return fmaxf(x, 0.f) + log1pf(expf(-fabsf(x)));
}

__device__ __forceinline__ float sigmoid_f(float x) {
  if (x >= 0.f) return 1.f / (1.f + expf(-x));
  const float e = expf(x);
  return e / (1.f + e);
}

// Rows of 3 to kLossPairsResp slots have their pairs spread over the threads, in batches
// of up to kLossSpreadRows rows.
constexpr int kLossPairsResp = 8;
constexpr int kLossSpreadRows = 64;

// SPREAD: a thread a pair forms its softplus and sigmoid, then a thread a row and a
// thread a slot add them in the order of the plain form below, a thread a row,
// whose chain of pairs sets the time (8 rows of 4 ranked responses: 6.6 us plain,
// 4.1 us spread).  With two slots there is no chain: 3.5 us plain, 4.0 us spread.
// A turn takes 256 / pairs rows (9 at 8 slots) where the plain form takes 256, so that
// wins in larger batches.  Timed with the events' 3 us, plain / spread in us:
//   slots     8 rows     64 rows    128 rows    2048 rows
//     3     7.3 / 6.2   7.0 / 6.4   7.3 / 8.2    26 / 49
//     4     9.2 / 6.4   9.6 / 8.7   9.6 / 12.3   45 / 99
//     6    14.8 / 6.5  14.2 / 13.4 15.1 / 22.4   94 / 273
//     8    23.1 / 7.0  25.4 / 24.6 25.9 / 42.1  202 / 570
template <bool SPREAD>
__global__ __launch_bounds__(256) void pair_loss_kernel(LossLaunch a) {
  const int tid = threadIdx.x;
  const float inv_rows = 1.f / (float)a.n_qualified;
  float part = 0.f;
  auto count = [&](int b) { return a.num_resp ? a.num_resp[b] : a.nr_inline[b]; };
  auto row_weight = [&](int K) { return a.beta * inv_rows / (0.5f * (float)K * (float)(K - 1)); };
  if constexpr (SPREAD) {
    __shared__ float s_sp[256], s_sg[256];
    const int np = max(1, a.K_max * (a.K_max - 1) / 2);  // pairs a row at most, <= 28
    const int RB = 256 / np;                             // rows a turn
    for (int b0 = 0; b0 < a.B; b0 += RB) {
      const int r = tid / np, q = tid - r * np;  // pair q = p (p - 1) / 2 + c, c < p
      if (r < RB && b0 + r < a.B) {
        int p = 1;
        while (q >= p * (p + 1) / 2) ++p;
        const int c = q - p * (p - 1) / 2;
        if (p < count(b0 + r)) {
          const int64_t o = (int64_t)(b0 + r) * a.K_max;
          const float zp = a.beta * (a.pol[o + p] - (a.ref ? a.ref[o + p] : 0.f));
          const float zc = a.beta * (a.pol[o + c] - (a.ref ? a.ref[o + c] : 0.f));
          const float d = zp - zc;
          s_sp[tid] = softplus_f(-d);
          s_sg[tid] = sigmoid_f(-d);
        }
      }
      __syncthreads();
      for (int i = tid; a.dlogp && i < RB * a.K_max; i += 256) {
        const int r = i / a.K_max, k = i - r * a.K_max, b = b0 + r;
        if (b >= a.B) break;
        const int K = count(b);
        float g = 0.f;
        if (K >= 2 && k < K) {
          const float w = row_weight(K);
          for (int c = 0; c < k; ++c) g -= s_sg[r * np + k * (k - 1) / 2 + c] * w;
          for (int p = k + 1; p < K; ++p) g += s_sg[r * np + p * (p - 1) / 2 + k] * w;
        }
        a.dlogp[(int64_t)b * a.K_max + k] = g;
      }
      if (tid < RB && b0 + tid < a.B) {
        const int K = count(b0 + tid);
        float rl = 0.f;
        if (K >= 2) {
          for (int q = 0; q < K * (K - 1) / 2; ++q) rl += s_sp[tid * np + q];
          rl /= 0.5f * (float)K * (float)(K - 1);
          part += rl;
        }
        if (a.row_loss) a.row_loss[b0 + tid] = rl;
      }
      __syncthreads();  // before the next rows' pairs
    }
  } else {
    for (int b = tid; b < a.B; b += blockDim.x) {
      const int K = count(b);
      const float* pol = a.pol + (int64_t)b * a.K_max;
      const float* ref = a.ref ? a.ref + (int64_t)b * a.K_max : nullptr;
      float* g = a.dlogp ? a.dlogp + (int64_t)b * a.K_max : nullptr;
      if (g)
        for (int k = 0; k < a.K_max; ++k) g[k] = 0.f;
      float rl = 0.f;
      if (K >= 2) {
        const float w = row_weight(K);
        for (int p = 1; p < K; ++p) {          // preferred slot (larger index)
          const float zp = a.beta * (pol[p] - (ref ? ref[p] : 0.f));
          for (int c = 0; c < p; ++c) {
            const float zc = a.beta * (pol[c] - (ref ? ref[c] : 0.f));
            const float d = zp - zc;
            rl += softplus_f(-d);
            if (g) {
              const float sg = sigmoid_f(-d);
              g[p] -= sg * w;
              g[c] += sg * w;
            }
          }
        }
        rl /= 0.5f * (float)K * (float)(K - 1);
        part += rl;
      }
      if (a.row_loss) a.row_loss[b] = rl;
    }
  }
  // fixed-order reduction
  __shared__ float red[256];
  red[tid] = part;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) red[tid] += red[tid + s];
    __syncthreads();
  }
  if (tid == 0) *a.loss = red[0] * inv_rows;
}

}  // namespace

hipError_t launch_logprob(const LogprobLaunch& a, hipStream_t s) {
  hipError_t e = hipSuccess;
  if (a.n_rows > 0) {
    TimingScope t("pp_logprob_rows", s);
    if (a.dtype == kBF16)
      hipLaunchKernelGGL(logprob_rows_kernel<__bf16>, dim3(a.n_rows), dim3(kLpThreads), 0, s,
                         (const __bf16*)a.logits, a.tokens, a.rows, a.labels, a.tok, a.vocab);
    else
      hipLaunchKernelGGL(logprob_rows_kernel<float>, dim3(a.n_rows), dim3(kLpThreads), 0, s,
                         (const float*)a.logits, a.tokens, a.rows, a.labels, a.tok, a.vocab);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (a.n_resp > 0) {
    TimingScope t("pp_segsum", s);
    const int threads = 256, waves_per_block = threads / 64;
    hipLaunchKernelGGL(segsum_kernel, dim3((a.n_resp + waves_per_block - 1) / waves_per_block),
                       dim3(threads), 0, s, a.tok, a.resp, a.seq, a.n_resp);
    e = hipGetLastError();
  }
  return e;
}

namespace {

// The shape with the most workgroups per compute unit whose registers hold a row
// of `nvec` 16-byte vectors.
//
// In a dense gradient whose rows mostly predict nothing the zeros set the time, and
// they are written faster by fewer workgroups at once (few rows' lines in flight).
// Another shape would add a predicting row's sum in another order than the gathered
// form, so the same one is held to one workgroup a unit by LDS that it does not use.
// 16000 rows, a share f of them predicting, us with four (two at 50000) / with one:
//           20000 bf16   12000 fp32   32000 bf16   50000 bf16 (12000 rows)
//   f .02    144 / 140    164 / 157    214 / 207    281 / 269
//      .1    158 / 135    179 / 164    240 / 218    299 / 286
//      .2    171 / 158    192 / 174    259 / 236    316 / 309
//      .3    178 / 188    204 / 200    273 / 274    336 / 319
//      .5    198 / 249    231 / 248    303 / 349    370 / 396
// Below 1700 vectors (12000 bf16) and on rows off the boundaries four are as good.
template <typename T, bool EDGE>
void launch_logprob_bwd_rows(const LogprobBwdLaunch& a, int grid, int nvec, hipStream_t s) {
  constexpr int kMost = EDGE ? 18 : 19;
  constexpr unsigned kHalfLds = 96 << 10;  // more than half of a unit's 160 KB
  const bool few = !EDGE && !a.gathered && nvec >= 1700 && nvec <= 1024 * 8 &&
                   (int64_t)a.n_rows * 14000 <= (int64_t)std::min(nvec, 4900) * a.sumT;
  auto launch = [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), few ? kHalfLds : 0u, s, a);
  };
  if (nvec <= 512 * 8) launch(logprob_bwd_kernel<T, 512, 8, EDGE, false>, 512);
  else if (nvec <= 1024 * 8) launch(logprob_bwd_kernel<T, 1024, 8, EDGE, false>, 1024);
  else if (nvec <= 1024 * kMost) launch(logprob_bwd_kernel<T, 1024, kMost, EDGE, false>, 1024);
  else launch(logprob_bwd_kernel<T, 1024, 16, EDGE, true>, 1024);
}

}  // namespace

hipError_t launch_logprob_bwd(const LogprobBwdLaunch& a, hipStream_t s) {
  const int grid = a.gathered ? a.n_rows : a.sumT;
  if (grid <= 0) return hipSuccess;
  TimingScope t(a.gathered ? "pp_logprob_bwd_rows" : "pp_logprob_bwd", s);
  const int per_vec = a.dtype == kBF16 ? 8 : 4;
  const int nvec = a.vocab / per_vec;
  // every row of both matrices starts on a 16-byte boundary?
  const bool edge = a.vocab % per_vec != 0 || (reinterpret_cast<uintptr_t>(a.logits) & 15) != 0 ||
                    (reinterpret_cast<uintptr_t>(a.dlogits) & 15) != 0;
  if (a.dtype == kBF16) {
    if (edge) launch_logprob_bwd_rows<__bf16, true>(a, grid, nvec, s);
    else launch_logprob_bwd_rows<__bf16, false>(a, grid, nvec, s);
  } else {
    if (edge) launch_logprob_bwd_rows<float, true>(a, grid, nvec, s);
    else launch_logprob_bwd_rows<float, false>(a, grid, nvec, s);
  }
  return hipGetLastError();
}

hipError_t launch_loss(const LossLaunch& a, hipStream_t s) {
  TimingScope t("pp_pair_loss", s);
  if (a.K_max >= 3 && a.K_max <= kLossPairsResp && a.B <= kLossSpreadRows)
    hipLaunchKernelGGL(pair_loss_kernel<true>, dim3(1), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL(pair_loss_kernel<false>, dim3(1), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace pp
