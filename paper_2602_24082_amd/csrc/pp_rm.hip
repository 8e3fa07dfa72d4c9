// Reward-model head over packed rows (Sec. 2.1 reward model; Sec. 3.2 layout).
//
// The reward of the sequence (prompt, response k) is a linear head on the
// hidden state of its last token: o_k + L_k - 1 in the packed row, or the last
// prompt token P - 1 when the response is empty (prompt tokens see only the
// prompt, so their hidden states are those of the unpacked prompt).  The host
// resolves every (row, response) slot to its flat hidden row.  Kernels:
//
//   rm_scores      one workgroup per slot: w . h_row + bias (fixed-order
//                  reduction; 0 for slots without a row)
//   rm_bwd         its first workgroups: dw = sum over slots, in slot order, of
//                  dscore * h_row (one thread per column), and one for dbias, the
//                  sum of the dscores; then one workgroup per flat row: dhidden = (sum of the
//                  slots' dscores) * w on the rows some slot reads, 0 elsewhere
//
// The backward is bound by writing the [sumT, H] gradient once.  dw reads only
// the slots' rows but as a chain over them, so it runs beside that write in one
// launch (17792 rows of 4096 bf16, 32 slots: 22 us + 14 us apart, 23 us together).

#include <hip/hip_runtime.h>

#include "pp_device.h"
#include "pp_launch.h"

namespace pp {
namespace {

constexpr int kRmThreads = 256;

template <typename T>
__device__ __forceinline__ float ld(const T* p, int64_t i) {
  return (float)p[i];
}

// 16 bytes of T, and whether rows of H elements from `p` on start on 16-byte boundaries.
template <typename T>
struct Vec {
  static constexpr int N = 16 / (int)sizeof(T);
  typedef T type __attribute__((ext_vector_type(N)));
};
template <typename T>
__device__ __forceinline__ bool rows_aligned(const void* p, int H) {
  return H % Vec<T>::N == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0;
}

template <typename T>
__global__ __launch_bounds__(kRmThreads) void rm_scores_kernel(RmLaunch a) {
  const int slot = blockIdx.x;
  const int64_t row = a.slot_row[slot];
  const int tid = threadIdx.x;
  float acc = 0.f;
  if (row >= 0) {
    const T* h = reinterpret_cast<const T*>(a.hidden) + row * (int64_t)a.H;
    const T* w = reinterpret_cast<const T*>(a.w);
    if (rows_aligned<T>(a.hidden, a.H) && rows_aligned<T>(a.w, a.H)) {
      using V = typename Vec<T>::type;
      const V* hv = reinterpret_cast<const V*>(h);
      const V* wv = reinterpret_cast<const V*>(w);
#pragma unroll 2
      for (int i = tid; i < a.H / Vec<T>::N; i += kRmThreads) {
        const V x = hv[i], y = wv[i];
#pragma unroll
        for (int e = 0; e < Vec<T>::N; ++e) acc = fmaf((float)x[e], (float)y[e], acc);
      }
    } else {
      for (int i = tid; i < a.H; i += kRmThreads) acc = fmaf(ld<T>(h, i), ld<T>(w, i), acc);
    }
  }
  acc = wave_sum(acc);
  __shared__ float part[kRmThreads / 64];
  if ((tid & 63) == 0) part[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    float s = 0.f;
    for (int i = 0; i < kRmThreads / 64; ++i) s += part[i];
    a.scores[slot] = row >= 0 ? s + a.bias : 0.f;
  }
}

template <typename T>
__device__ __forceinline__ void rm_dhidden_row(const RmBwdLaunch& a, int64_t r) {
  const int rec = a.row_rec[r];
  float g = 0.f;
  if (rec >= 0) {
    const RmRowSlots rs = a.rows[rec];
    for (int j = 0; j < rs.slot_cnt; ++j) g += a.dscores[a.slots[rs.slot_off + j]];
  }
  T* out = reinterpret_cast<T*>(a.dhidden) + r * (int64_t)a.H;
  const T* w = reinterpret_cast<const T*>(a.w);
  if (rows_aligned<T>(a.dhidden, a.H) && rows_aligned<T>(a.w, a.H)) {
    using V = typename Vec<T>::type;
    for (int i = threadIdx.x; i < a.H / Vec<T>::N; i += kRmThreads) {
      V y = {};
      if (rec >= 0) {
        const V x = reinterpret_cast<const V*>(w)[i];
#pragma unroll
        for (int e = 0; e < Vec<T>::N; ++e) y[e] = (T)(g * (float)x[e]);
      }
      reinterpret_cast<V*>(out)[i] = y;
    }
    return;
  }
  for (int i = threadIdx.x; i < a.H; i += kRmThreads) out[i] = (T)(rec >= 0 ? g * ld<T>(w, i) : 0.f);
}

// The slots' records come 64 at a time, one a lane, and 32 slots' elements are in
// flight at once: every further round of loads waits behind dhidden's stores.
template <typename T>
__device__ __forceinline__ void rm_dw_columns(const RmBwdLaunch& a, int block) {
  const int lane = threadIdx.x & 63;
  const int i = min(block * kRmThreads + (int)threadIdx.x, a.H - 1);
  constexpr int S = 32;
  const T* h = reinterpret_cast<const T*>(a.hidden) + i;
  float acc = 0.f;
  for (int s0 = 0; s0 < a.n_slots; s0 += 64) {
    const int n = min(64, a.n_slots - s0);
    const int row_l = lane < n ? (int)a.slot_row[s0 + lane] : -1;  // flat rows fit 31 bits
    const float g_l = lane < n ? a.dscores[s0 + lane] : 0.f;
    for (int j0 = 0; j0 < n; j0 += S) {
      float x[S];
#pragma unroll
      for (int j = 0; j < S; ++j) {
        const int row = __builtin_amdgcn_readlane(row_l, j0 + j);
        if (row >= 0) x[j] = ld<T>(h, row * (int64_t)a.H);
      }
#pragma unroll
      for (int j = 0; j < S; ++j) {
        const float g = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g_l), j0 + j));
        if (__builtin_amdgcn_readlane(row_l, j0 + j) >= 0) acc = fmaf(g, x[j], acc);
      }
    }
  }
  if (block * kRmThreads + (int)threadIdx.x < a.H) a.dw[i] = acc;
}

// dbias = the sum of dscores in slot order: a wave loads 64 at a time (a load per
// addition would take longer than all of dhidden)
__device__ __forceinline__ void rm_dbias(const RmBwdLaunch& a) {
  if (!a.dbias || threadIdx.x >= 64) return;
  float b = 0.f;
  for (int s0 = 0; s0 < a.n_slots; s0 += 64) {
    const int s = s0 + (int)threadIdx.x;
    const bool on = s < a.n_slots && a.slot_row[s] >= 0;
    const float v = on ? a.dscores[s] : 0.f;
    const uint64_t mask = __ballot(on);
    for (int j = 0; j < 64; ++j) {
      const float x = __shfl(v, j, 64);
      if ((mask >> j) & 1) b += x;
    }
  }
  if (threadIdx.x == 0) *a.dbias = b;
}

template <typename T>
__global__ __launch_bounds__(kRmThreads) void rm_bwd_kernel(RmBwdLaunch a, int dw_blocks) {
  const int b = blockIdx.x;
  if (b < dw_blocks) rm_dw_columns<T>(a, b);
  else if (b == dw_blocks) rm_dbias(a);
  else
    for (int64_t r = b - dw_blocks - 1; r < a.sumT; r += gridDim.x - dw_blocks - 1) rm_dhidden_row<T>(a, r);
}

}  // namespace

hipError_t launch_rm_scores(const RmLaunch& a, hipStream_t s) {
  if (a.n_slots <= 0) return hipSuccess;
  TimingScope t("pp_rm_scores", s);
  if (a.dtype == kBF16)
    hipLaunchKernelGGL(rm_scores_kernel<__bf16>, dim3(a.n_slots), dim3(kRmThreads), 0, s, a);
  else
    hipLaunchKernelGGL(rm_scores_kernel<float>, dim3(a.n_slots), dim3(kRmThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_rm_bwd(const RmBwdLaunch& a, hipStream_t s) {
  TimingScope t({"pp_rm_dhidden", "pp_rm_dw"}, s);
  const int dw_blocks = (a.H + kRmThreads - 1) / kRmThreads;
  // a workgroup a row as far as a launch's 2^32 - 1 threads go
  const int64_t most = 0xffffffffll / kRmThreads - dw_blocks - 1;
  const dim3 grid((unsigned)(dw_blocks + 1 + (a.sumT < most ? a.sumT : most)));
  if (a.dtype == kBF16)
    hipLaunchKernelGGL(rm_bwd_kernel<__bf16>, grid, dim3(kRmThreads), 0, s, a, dw_blocks);
  else
    hipLaunchKernelGGL(rm_bwd_kernel<float>, grid, dim3(kRmThreads), 0, s, a, dw_blocks);
  return hipGetLastError();
}

}  // namespace pp
