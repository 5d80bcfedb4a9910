// rmdf_cfar.hip - two-sided cell-averaging CFAR detector on an FP32 image,
// the detection stage after the prediction-error filter (the paper passes
// the filter output to a threshold and a tracker, Sec. 1, without fixing the
// detector).
//
// Per pixel p: training cells = in-frame pixels within Chebyshev distance
// R = guard + train of p but farther than guard; mu and sigma^2 = mean of x
// and of x^2 over them minus mu^2; detection where n > 0 and
// |x(p) - mu| > k sigma.  One workgroup per 64 x TH output tile: the tile and
// its R-pixel halo are staged in LDS once, box sums along rows (outer and
// guard widths, x and x^2) go to LDS, and each thread sums one output's
// columns.  HBM traffic is one read of the image (plus the halo) and one
// write of the detections.  What bounds it is the chain of LDS reads and sums
// of one workgroup, a frame of detector size having fewer workgroups than the
// chip holds: so a thread sums CF_Q rows side by side, and small frames take
// tiles of 4 rows instead of 16.  Per image at R = 6 (one row at a time, tiles
// of 16, before): 320x256 10.7 -> 4.1 us, 640x512 11.1 -> 7.2, 1280x1024
// 30.6 -> 22.4; at R = 16: 19.0 -> 8.8, 19.5 -> 13.6, 54.8 -> 35.9.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <type_traits>

#include "../../include/rmdf.h"
#include "rmdf_internal.h"

namespace rmdf {
namespace {

constexpr int CF_TW = 64, CF_RMAX = 16;
constexpr int CF_XS = CF_TW + 2 * CF_RMAX;   // staged row stride
constexpr int CF_Q = 4;                      // rows a thread sums side by side

// Thread (g, c) = (wavefront, lane) takes column c of rows g, g + 4, ...
template <int TH>
__global__ void __launch_bounds__(256) k_cfar(const float* __restrict__ x, int H, int W, int G, int R, float k,
                                              unsigned char* __restrict__ det, float* __restrict__ level) {
  constexpr int HR = TH + 2 * CF_RMAX;       // staged rows (at most)
  __shared__ float s_x[HR * CF_XS];
  __shared__ float4 s_h[HR * CF_TW];         // per row and column: outer sums of x and x^2, guard sums
  const int tx0 = blockIdx.x * CF_TW, ty0 = blockIdx.y * TH;
  const int hw = CF_TW + 2 * R, hh = TH + 2 * R;
  const int c = threadIdx.x & 63, g = threadIdx.x >> 6;
  auto sample = [&](int r, int cc) {
    const int gy = ty0 - R + r, gx = tx0 - R + cc;
    return (gy >= 0 && gy < H && gx >= 0 && gx < W) ? x[(size_t)gy * W + gx] : 0.f;
  };
  // the wavefront's rows g, g + 4, ...: CF_Q, then 2, then 1 at a time
  auto rows = [&](auto work) {
    int r = g;
    for (; r + 4 * (CF_Q - 1) < hh; r += 4 * CF_Q) work(std::integral_constant<int, CF_Q>{}, r);
    for (; r + 4 < hh; r += 8) work(std::integral_constant<int, 2>{}, r);
    if (r < hh) work(std::integral_constant<int, 1>{}, r);
  };
  rows([&](auto nq, int r0) {
    constexpr int Q = decltype(nq)::value;
    float v[Q], e[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) v[q] = sample(r0 + 4 * q, c);
    if (c + CF_TW < hw) {
#pragma unroll
      for (int q = 0; q < Q; ++q) e[q] = sample(r0 + 4 * q, c + CF_TW);
#pragma unroll
      for (int q = 0; q < Q; ++q) s_x[(r0 + 4 * q) * CF_XS + c + CF_TW] = e[q];
    }
#pragma unroll
    for (int q = 0; q < Q; ++q) s_x[(r0 + 4 * q) * CF_XS + c] = v[q];
  });
  __syncthreads();
  // row sums centred on output column c: outer width 2R+1, guard width 2G+1
  rows([&](auto nq, int r0) {
    constexpr int Q = decltype(nq)::value;
    const float* row = s_x + r0 * CF_XS + c;  // row[R + d] is column c + d
    float so[Q] = {}, qo[Q] = {}, si[Q] = {}, qi[Q] = {};
    auto outer = [&](int d) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float v = row[4 * q * CF_XS + d];
        so[q] += v;
        qo[q] += v * v;
      }
    };
    for (int d = 0; d < R - G; ++d) outer(d);
    for (int d = R - G; d <= R + G; ++d) {
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const float v = row[4 * q * CF_XS + d];
        so[q] += v;
        qo[q] += v * v;
        si[q] += v;
        qi[q] += v * v;
      }
    }
    for (int d = R + G + 1; d <= 2 * R; ++d) outer(d);
#pragma unroll
    for (int q = 0; q < Q; ++q) s_h[(r0 + 4 * q) * CF_TW + c] = make_float4(so[q], qo[q], si[q], qi[q]);
  });
  __syncthreads();
#pragma unroll
  for (int r = g; r < TH; r += 4) {
    const int gy = ty0 + r, gx = tx0 + c;
    if (gy >= H || gx >= W) continue;
    const float4* col = s_h + r * CF_TW + c;
    float so = 0.f, qo = 0.f, si = 0.f, qi = 0.f;
    auto outer = [&](int d) {
      const float2 v = *reinterpret_cast<const float2*>(col + d * CF_TW);
      so += v.x;
      qo += v.y;
    };
#pragma unroll 4
    for (int d = 0; d < R - G; ++d) outer(d);
#pragma unroll 4
    for (int d = R - G; d <= R + G; ++d) {
      const float4 v = col[d * CF_TW];
      so += v.x;
      qo += v.y;
      si += v.z;
      qi += v.w;
    }
#pragma unroll 4
    for (int d = R + G + 1; d <= 2 * R; ++d) outer(d);
    // in-frame cells of the outer and guard squares (the frame is a rectangle)
    const int nxo = min(gx + R, W - 1) - max(gx - R, 0) + 1, nyo = min(gy + R, H - 1) - max(gy - R, 0) + 1;
    const int nxi = min(gx + G, W - 1) - max(gx - G, 0) + 1, nyi = min(gy + G, H - 1) - max(gy - G, 0) + 1;
    const int n = nxo * nyo - nxi * nyi;
    float sig = 0.f;
    unsigned char d = 0;
    if (n > 0) {
      const float inv = 1.0f / (float)n;
      const float mu = (so - si) * inv;
      sig = sqrtf(fmaxf((qo - qi) * inv - mu * mu, 0.f));
      d = fabsf(s_x[(r + R) * CF_XS + c + R] - mu) > k * sig ? 1 : 0;
    }
    det[(size_t)gy * W + gx] = d;
    if (level) level[(size_t)gy * W + gx] = sig;
  }
}

template <int TH>
void launch_cfar(const float* x, int H, int W, int G, int R, float k, unsigned char* det, float* level, hipStream_t s) {
  const dim3 grid((W + CF_TW - 1) / CF_TW, (H + TH - 1) / TH);
  hipLaunchKernelGGL(k_cfar<TH>, grid, dim3(256), 0, s, x, H, W, G, R, k, det, level);
}

// Tiles of 4 rows or of 16: a workgroup takes as long as its staged rows, TH + 2R; 3
// of the small and 2 of the large fit a CU (LDS), the large ones ending in whole
// rounds.  (us, 4 and 16 rows: 320x256 R = 6 4.1 and 8.1; 640x512 R = 6 7.2 and 8.5,
// R = 16 17.4 and 13.6; 1280x1024 R = 1 13.7 and 14.6, R = 3 21.2 and 18.4.)
// (A launch is limited to 65536 rows of workgroups: images of more rows of small
// tiles than that take the large ones.)
bool short_tiles(int H, int W, int R) {
  if ((H + 3ll) / 4 > 65535) return false;
  const long long xb = (W + CF_TW - 1) / CF_TW, n4 = xb * ((H + 3) / 4), n16 = xb * ((H + 15) / 16);
  return std::max(n4, 768ll) * (4 + 2 * R) < 768 * ((n16 + 511) / 512) * (16 + 2 * R);
}

}  // namespace
}  // namespace rmdf

extern "C" rmdf_status rmdf_cfar(const float* x_dev, int H, int W, int guard, int train, float k,
                                 unsigned char* det_dev, float* level_dev, void* stream) {
  auto bad = [](const char* m) {
    rmdf_internal_set_create_error(m);
    return RMDF_E_INVAL;
  };
  if (!x_dev || !det_dev) return bad("cfar: NULL image or detection pointer");
  if (H < 1 || W < 1) return bad("cfar: H, W must be >= 1");
  if (guard < 0 || train < 1 || guard + train > rmdf::CF_RMAX) return bad("cfar: need guard >= 0, train >= 1, guard + train <= 16");
  if (!(k >= 0.f) || !(k < INFINITY)) return bad("cfar: k must be finite and >= 0");
  const int R = guard + train;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (rmdf::short_tiles(H, W, R))
    rmdf::launch_cfar<4>(x_dev, H, W, guard, R, k, det_dev, level_dev, st);
  else
    rmdf::launch_cfar<16>(x_dev, H, W, guard, R, k, det_dev, level_dev, st);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    rmdf_internal_set_create_error(std::string("cfar launch: ") + hipGetErrorString(e));
    return RMDF_E_DEVICE;
  }
  return RMDF_OK;
}
