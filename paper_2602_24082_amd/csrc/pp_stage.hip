// What a call needs on its stream before its own kernels, in one launch:
//   * plan metadata, which the host wrote into mapped pinned memory, copied into
//     the workspace (on the compute queue the copy needs no hand-off to a DMA
//     engine and back, which for an image of a few hundred KB costs more than the
//     copy itself);
//   * bf16 copies (round to nearest even) of fp32 attention inputs;
//   * zeros in the positions of an output that the kernels do not write.
// Each piece is a few us of memory traffic, so what a small call pays is the
// launches: an fp32 forward and backward of 761 tokens (four heads of size 64)
// enqueued seven conversions and two copies of 2 us each, and now two launches.

#include <hip/hip_runtime.h>

#include "pp_device.h"
#include "pp_launch.h"

namespace pp {
namespace {

typedef uint32_t Chunk16 __attribute__((ext_vector_type(4)));

constexpr int kThreads = kStageThreads;

__global__ __launch_bounds__(kThreads) void stage_kernel(StageLaunch a, StageBlocks nb) {
  int b = blockIdx.x;
  if (b < nb.copy) {
    // bytes [0, 16 n16) move as 16-byte vectors, the last few (< 16) one by one
    const int64_t n16 = (int64_t)(a.bytes / 16);
    const int tail = (int)(a.bytes % 16);
    const Chunk16* src = static_cast<const Chunk16*>(a.src);
    Chunk16* dst = static_cast<Chunk16*>(a.dst);
    const int64_t i = (int64_t)b * kThreads + threadIdx.x;
    if (i < n16) dst[i] = src[i];
    if (i < tail) reinterpret_cast<uint8_t*>(dst + n16)[i] = reinterpret_cast<const uint8_t*>(src + n16)[i];
    return;
  }
  b -= nb.copy;
#pragma unroll
  for (int c = 0; c < kStageCasts; ++c) {
    if (b < nb.cast[c]) {
      const float* src = a.cast[c].src;
      __bf16* dst = static_cast<__bf16*>(a.cast[c].dst);
      const int64_t n = a.cast[c].n;
      for (int64_t i = ((int64_t)b * kThreads + threadIdx.x) * 4; i < n; i += (int64_t)nb.cast[c] * kThreads * 4) {
        if (i + 4 <= n) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(src + i);
          *reinterpret_cast<bf16x4*>(dst + i) = __builtin_convertvector(v, bf16x4);
        } else {
          for (int64_t j = i; j < n; ++j) dst[j] = (__bf16)src[j];
        }
      }
      return;
    }
    b -= nb.cast[c];
  }
  const int64_t i = (int64_t)b * kThreads + threadIdx.x;
  if (i < a.n_zero) a.zero[i] = 0.f;
}

}  // namespace

hipError_t launch_stage(const StageLaunch& a, hipStream_t s) {
  const StageBlocks nb = stage_blocks(a);
  if (nb.total == 0) return hipSuccess;
  int64_t casts = 0;
  for (int n : nb.cast) casts += n;
  TimingScope t({nb.copy ? "pp_stage" : nullptr, casts ? "pp_to_bf16" : nullptr, nb.zero ? "pp_fill_zero" : nullptr}, s);
  hipLaunchKernelGGL(stage_kernel, dim3((unsigned)nb.total), dim3(kThreads), 0, s, a, nb);
  return hipGetLastError();
}

}  // namespace pp
