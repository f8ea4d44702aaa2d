// Small kernels: copy-scale for length-1 transforms, the row shuffle of the
// fused 2-D plan in place, and FP64 twiddle-table generation on the GPU (used
// for 1-D lengths >= 2^22).
#include <algorithm>

#include "twiddle.hpp"
#include "variants.hpp"

namespace mfft {

hipError_t launch_scale_copy(int dtype, const void* in, void* out, int64_t n, float scale,
                             hipStream_t s) {
  const unsigned blocks = (unsigned)((n + 255) / 256);
  if (n <= 0) return hipSuccess;
  switch (dtype) {
    case DT_C64:
      hipLaunchKernelGGL(k_scale_copy<float2>, dim3(blocks), dim3(256), 0, s,
                         (const float2*)in, (float2*)out, n, scale);
      break;
    case DT_C16F:
      hipLaunchKernelGGL(k_scale_copy<__half2>, dim3(blocks), dim3(256), 0, s,
                         (const __half2*)in, (__half2*)out, n, scale);
      break;
    default:
      hipLaunchKernelGGL(k_scale_copy<c16bf>, dim3(blocks), dim3(256), 0, s,
                         (const c16bf*)in, (c16bf*)out, n, scale);
      break;
  }
  return hipGetLastError();
}

// Images of R = 2^lg_rows rows of C points, in place: row n1 + (R/r)*j moves to
// row r*n1 + j, where the fused row pass writes it (k_rowcol), so that this
// pass then needs no second buffer.  That is a rotation of the row number's
// bits by log2 r, whose cycles have at most lg_rows rows: a lane holds one
// column of a whole cycle in registers, so no two lanes share an element.
// Workgroup: 256 columns of the cycle that starts at row starts[blockIdx.y].
// Bound by the copy it is: 2^24 points, which the last-level cache holds, 35 us
// (4 x 2048 x 2048) to 47 (4096 x 4096), 2^26 (8 x 4096 x 2048) 210 us, 5.1 TB/s.
constexpr int kMaxCycle = 14;
__global__ void __launch_bounds__(256) k_row_shuffle(float2* x, const int32_t* __restrict__ starts, int lg_rows,
                                                     int lg_r, int C, int64_t batch) {
  const uint32_t first = starts[blockIdx.y], mask = (1u << lg_rows) - 1;
  auto next = [&](uint32_t p) { return ((p << lg_r) | (p >> (lg_rows - lg_r))) & mask; };
  int len = 1;
  for (uint32_t p = next(first); p != first; p = next(p)) ++len;
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= C) return;
  for (int64_t b = blockIdx.z; b < batch; b += gridDim.z) {
    float2* img = x + b * ((int64_t)C << lg_rows) + c;
    float2 v[kMaxCycle];
    uint32_t p = first;
#pragma unroll
    for (int i = 0; i < kMaxCycle; ++i)
      if (i < len) {
        v[i] = img[(int64_t)p * C];
        p = next(p);
      }
#pragma unroll
    for (int i = 0; i < kMaxCycle; ++i)
      if (i < len) {
        p = next(p);  // the cycle closes: row `first` again, then the rest
        img[(int64_t)p * C] = v[i];
      }
  }
}

hipError_t launch_row_shuffle(void* x, const int32_t* starts, int cycles, int lg_rows, int lg_r, int C, int64_t batch,
                              hipStream_t s) {
  if (lg_rows > kMaxCycle || lg_r >= lg_rows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_row_shuffle, dim3((C + 255) / 256, (unsigned)cycles, (unsigned)std::min<int64_t>(batch, 65535)),
                     dim3(256), 0, s, (float2*)x, starts, lg_rows, lg_r, C, batch);
  return hipGetLastError();
}

// One thread per table entry: entry i of segment g is W_M^{e(i)} rounded from
// float64 to float32 (see twiddle.hpp for e(i)).
__global__ void __launch_bounds__(256) k_twiddle_fp64(float2* table, const TwSeg* segs, int nseg) {
  const int g = blockIdx.y;
  if (g >= nseg) return;
  const TwSeg sg = segs[g];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < sg.count;
       i += (int64_t)gridDim.x * 256)
    table[sg.off + i] = seg_value(sg, i);
}

hipError_t launch_twiddle_fp64(float2* table, const TwSeg* d_segs, int nseg, int64_t max_count,
                               hipStream_t s) {
  unsigned bx = (unsigned)((max_count + 255) / 256);
  if (bx > 4096) bx = 4096;
  if (bx == 0) bx = 1;
  hipLaunchKernelGGL(k_twiddle_fp64, dim3(bx, (unsigned)nseg), dim3(256), 0, s, table, d_segs, nseg);
  return hipGetLastError();
}

}  // namespace mfft
