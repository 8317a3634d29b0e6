// Explicit prefix-sum mode: the scans over chunk states and the dispatch of
// the chunk kernels (slim_ps.hpp), which are compiled per element type and
// head dimension in slim_ps_*.hip.
#include "slim_common.hpp"
#include "slim_kernels.hpp"

namespace slim {

namespace {
// s += x with the rounding error carried in c (Kahan's compensated sum)
__device__ __forceinline__ void kahan_add(float& s, float& c, float x) {
  const float y = x - c, t = s + y;
  c = (t - s) - y;
  s = t;
}
}  // namespace

// ---- state before every chunk, in place of the chunk sums, one thread per
// state entry; all relative to one shift: kshift (given), or the largest of
// the chunks' shifts and the initial state's (-> shift_out).
//   mode 0: start from S_in (zero if NULL, relative to in_shift); S_out = the
//           state after the last chunk ([m][d + 1], may be NULL)
//   mode 1: start from S_in - the sum of all chunks (eq. 17: the state before
//           the run from the state after it); S_out = that start
// S_in of head h at S_in + h in_stride ([m][d + 1]).  S_out may be S_in.
// Grid: (entries / 256, heads).
__global__ __launch_bounds__(256) void ps_scan_kernel(PsArgs a, int mode) {
  __shared__ float red[4];
  const int head = blockIdx.y, E = a.d + 1, SP = a.d + 4;
  const bool own = a.seg_shift != nullptr;  // sums relative to their chunk's shift
  const float* ss = own ? a.seg_shift + (size_t)head * a.nch : nullptr;
  float shift = 0.f;
  if (own) {
    float mx = -INFINITY;
    for (int p = threadIdx.x; p < a.nch; p += 256) mx = fmaxf(mx, ss[p]);
    mx = wave_max(mx);
    if (lane_id() == 0) red[wave_id()] = mx;
    __syncthreads();
    shift = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    if (a.S_in != nullptr) shift = fmaxf(shift, a.in_shift[head]);
    if (blockIdx.x == 0 && threadIdx.x == 0) a.shift_out[head] = shift;
  } else if (a.kshift != nullptr) {
    shift = a.kshift[head];
  }
  const int el = blockIdx.x * 256 + threadIdx.x;
  if (el >= a.M * E) return;
  const int m = el / E, e = el - m * E;
  float v = 0.f;
  if (a.S_in != nullptr) {
    v = a.S_in[head * a.in_stride + el];
    if (a.in_shift != nullptr) v *= exp_f32(a.in_shift[head] - shift);
  }
  const size_t step = (size_t)a.M * SP;
  float* S = a.S + (size_t)head * a.nch * step + (size_t)m * SP + e;
  constexpr int U = 8;  // chunks whose loads are issued together
  if (mode == 1) {
    float s = 0.f, cc = 0.f;
    for (int p = 0; p < a.nch; p += U) {
      float t[U];
#pragma unroll
      for (int j = 0; j < U; ++j) t[j] = p + j < a.nch ? S[(size_t)(p + j) * step] : 0.f;
#pragma unroll
      for (int j = 0; j < U; ++j) kahan_add(s, cc, t[j]);
    }
    v -= s;
    if (a.S_out != nullptr) a.S_out[head * (size_t)a.M * E + el] = v;
  }
  float cc = 0.f;
  for (int p = 0; p < a.nch; p += U) {
    float t[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      t[j] = 0.f;
      if (p + j < a.nch) {
        t[j] = S[(size_t)(p + j) * step];
        if (own) t[j] *= exp_f32(ss[p + j] - shift);
      }
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (p + j < a.nch) {
        S[(size_t)(p + j) * step] = v;
        kahan_add(v, cc, t[j]);
      }
  }
  if (mode == 0 && a.S_out != nullptr) a.S_out[head * (size_t)a.M * E + el] = v;
}

// ---- cotangent after every chunk, in place of what the chunks add: starts
// from G_in (zero if NULL), G_out = the cotangent before the first chunk
// (both [m][d + 1]; may be the same)
__global__ __launch_bounds__(256) void ps_rscan_kernel(PsArgs a) {
  const int head = blockIdx.y, E = a.d + 1, SP = a.d + 4;
  const int el = blockIdx.x * 256 + threadIdx.x;
  if (el >= a.M * E) return;
  const int m = el / E, e = el - m * E;
  const size_t sidx = head * (size_t)a.M * E + el, step = (size_t)a.M * SP;
  float* S = a.G + (size_t)head * a.nch * step + (size_t)m * SP + e;
  float v = a.G_in != nullptr ? a.G_in[sidx] : 0.f, cc = 0.f;
  constexpr int U = 8;
  for (int p = a.nch - 1; p >= 0; p -= U) {
    float t[U];
#pragma unroll
    for (int j = 0; j < U; ++j) t[j] = p - j >= 0 ? S[(size_t)(p - j) * step] : 0.f;
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (p - j >= 0) {
        S[(size_t)(p - j) * step] = v;
        kahan_add(v, cc, t[j]);
      }
  }
  a.G_out[sidx] = v;
}

namespace ps {
template <class T, int D>
hipError_t launch_rows_t(int which, const PsArgs& a, int nwg, hipStream_t s);
}

hipError_t launch_ps(int which, const PsArgs& a, int nwg, hipStream_t s) {
  if (which == kPsScan0 || which == kPsScan1 || which == kPsRscan) {
    const dim3 g(((a.d + 1) * a.M + 255) / 256, a.B * a.H);
    if (which == kPsRscan) hipLaunchKernelGGL(ps_rscan_kernel, g, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(ps_scan_kernel, g, dim3(256), 0, s, a, which == kPsScan1 ? 1 : 0);
    return hipGetLastError();
  }
  if (a.bf16) return a.d == 64 ? ps::launch_rows_t<bf16, 64>(which, a, nwg, s) : ps::launch_rows_t<bf16, 32>(which, a, nwg, s);
  return a.d == 64 ? ps::launch_rows_t<float, 64>(which, a, nwg, s) : ps::launch_rows_t<float, 32>(which, a, nwg, s);
}

}  // namespace slim
