// rmdf_mlp_train.hip - loss and gradients of one training batch of the learned
// velocity surrogate in three launches:
//
//   k_train_rows    everything that stays within a sample: H1 = relu(X W1^T + b1),
//                   H2 = relu(H1 W2^T + b2), the head, its loss and gradient, dH2
//                   and dH1; per tile of 32 samples also the partial sums of
//                   dW3, db3, the loss, db2 and db1
//   k_train_wgrad   dW1 = dH1^T X and dW2 = dH2^T H1, the batch split over
//                   workgroups (partial sums per chunk of samples)
//   k_train_reduce  sums the partials
//
// Layer by layer (two GEMMs, head, five transposes, three GEMMs, two column
// sums) a batch of 4096 took 262 us: the weight-gradient GEMM ran on 18
// workgroups (51 us), the head spent 82 us on wavefront reductions and
// atomics for dW3, and 17 launches cost more than the arithmetic (1.3
// GFLOP).  Here the sums over samples are split over the chip and added in a
// fixed order, and no intermediate is transposed through memory.  Now 38 us
// (rows 23, latency of its chain of stages; weight gradients 13; sums 4).
//
// Rounding points are those of the layer-by-layer kernels (k_gemm_nt, k_head):
// H1, H2, dH2, dH1 are BF16, every MFMA chain over a layer's inputs runs in
// ascending 16-wide steps from zero with the bias added to the finished sum,
// and the head is the same FP32 chain, so the BF16 intermediates are the same
// bits; only sums over samples are ordered differently.
#include <hip/hip_runtime.h>

#include "../../include/rmdf.h"
#include "rmdf_internal.h"

namespace rmdf {
namespace train {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int N0 = 1152, N1 = 128, N2 = 64;
constexpr int TR = 32;                           // samples per k_train_rows workgroup
constexpr int XCH = N0 / 8;                      // 16-byte chunks per feature row
constexpr int NSTEP = N0 / 16;                   // MFMA steps of layer 1
constexpr int GRP = 8;                           // steps whose W1 operands are loaded together
// per-tile partial sums: dW3 [3][64], db3 [3], loss, db2 [64], db1 [128]
constexpr int P_DB3 = 3 * N2, P_LOSS = P_DB3 + 3, P_DB2 = P_LOSS + 1, P_DB1 = P_DB2 + N2, P_N = P_DB1 + N1;
constexpr int WG_MAX_CHUNKS = 16;                // of the batch, in k_train_wgrad
constexpr int KB = 64;                           // samples per k_train_wgrad step
constexpr int KLD = KB + 8;                      // LDS row of KB samples: 144 B, 16-byte aligned

__device__ __forceinline__ unsigned short bf16_bits(float f) {
  unsigned int u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (unsigned short)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf16_float(unsigned short b) { return __uint_as_float(((unsigned int)b) << 16); }

// Row layouts in LDS: 16-byte chunk c of a row at slot c ^ (row mod 16) (within
// its group of 16, feature and H1 rows) or c ^ (row mod 8) (H2 and dH2 rows), so
// that an MFMA operand read of 16 rows covers all banks.
__device__ __forceinline__ int x_slot(int row, int c) { return (c & ~15) | ((c ^ row) & 15); }

// One workgroup (four wavefronts) per TR samples.  Wavefront w owns columns
// 32w .. 32w+31 of H1 and dH1; W1 and W2 operands come from the caches.
__global__ void __launch_bounds__(256) k_train_rows(const unsigned short* __restrict__ X, const float* __restrict__ lab,
                                                    int n, const unsigned short* __restrict__ W1,
                                                    const float* __restrict__ b1, const unsigned short* __restrict__ W2,
                                                    const float* __restrict__ b2, const float* __restrict__ W3,
                                                    const float* __restrict__ b3, float wv, float half_step,
                                                    unsigned short* __restrict__ H1, unsigned short* __restrict__ dH2,
                                                    unsigned short* __restrict__ dH1, float* __restrict__ part) {
  __shared__ __align__(16) unsigned short sX[TR * N0];   // features; later dH1 rows
  __shared__ __align__(16) unsigned short sH1[TR * N1];
  __shared__ __align__(16) unsigned short sH2[TR * N2];
  __shared__ __align__(16) unsigned short sG[TR * N2];   // dH2
  __shared__ float sW[3 * N2 + 3], sO[3][TR], sD[3][TR];
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = blockIdx.x * TR;
  // samples of this tile (a multiple of 8).  The sums over samples stop here: the
  // rows past n hold row n - 1 again with a zero gradient, and zero times an
  // overflowed activation is not zero.
  const int rows = min(TR, n - m0);
  float* P = part + (size_t)blockIdx.x * P_N;

  // the tile's features straight into LDS: 1 KB per load, rows past n re-read
  // row n - 1 (their results are dropped or zero)
#pragma unroll
  for (int q = 0; q < TR * XCH / 256; ++q) {
    const int s = (w * (TR * XCH / 256) + q) * 64 + lane, row = s / XCH, c = x_slot(row, s - row * XCH);
    __builtin_amdgcn_global_load_lds((const void*)(X + (size_t)min(m0 + row, n - 1) * N0 + c * 8),
                                     (lds_void*)(sX + (w * (TR * XCH / 256) + q) * 512), 16, 0, 0);
  }
  for (int i = tid; i < 3 * N2 + 3; i += 256) sW[i] = (i < 3 * N2) ? W3[i] : b3[i - 3 * N2];
  const int col = 32 * w + r32;
  const unsigned short* w1p = W1 + (size_t)col * N0 + 8 * h;
  bf16x8 bq[2][GRP];
  auto load_w1 = [&](int g, bf16x8 (&b)[GRP]) {
#pragma unroll
    for (int i = 0; i < GRP; ++i) b[i] = *reinterpret_cast<const bf16x8*>(w1p + 16 * (g * GRP + i));
  };
  load_w1(0, bq[0]);
  // W2^T operands of the backward step: W2[k][col], k = 16 s + 8 h + e
  bf16x8 bt[N2 / 16];
#pragma unroll
  for (int s = 0; s < N2 / 16; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) bt[s][e] = __builtin_bit_cast(__bf16, W2[(16 * s + 8 * h + e) * N1 + col]);
  // the direct loads count in vmcnt: each wavefront waits for its own (vmcnt 0,
  // lgkmcnt 0), then the barrier makes all of them visible
  __builtin_amdgcn_s_waitcnt(7 << 4);
  __syncthreads();

  // ---- layer 1
  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
  for (int g = 0; g < NSTEP / GRP; ++g) {
    if (g + 1 < NSTEP / GRP) load_w1(g + 1, bq[(g + 1) & 1]);
#pragma unroll
    for (int i = 0; i < GRP; ++i) {
      const int c = 2 * (g * GRP + i) + h;
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(sX + (r32 * XCH + x_slot(r32, c)) * 8);
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bq[g & 1][i], acc, 0, 0, 0);
    }
  }
  // MFMA result: column lane % 32, row (i / 4) * 8 + (lane / 32) * 4 + i % 4
  {
    const float bias = b1[col];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = (i >> 2) * 8 + h * 4 + (i & 3);
      float v = acc[i] + bias;
      v = v > 0.f ? v : 0.f;
      sH1[row * N1 + (((col >> 3) ^ (row & 15)) * 8) + (col & 7)] = bf16_bits(v);
    }
  }
  __syncthreads();

  // ---- layer 2 (wavefronts 0 and 1), H1 to memory (all)
  for (int i = tid; i < TR * N1 / 8; i += 256) {
    const int row = i >> 4, c = i & 15;
    if (m0 + row < n)
      *reinterpret_cast<uint4*>(H1 + (size_t)(m0 + row) * N1 + c * 8) =
          *reinterpret_cast<const uint4*>(sH1 + row * N1 + ((c ^ (row & 15)) * 8));
  }
  if (w < 2) {
    f32x16 a2;
#pragma unroll
    for (int i = 0; i < 16; ++i) a2[i] = 0.f;
    const unsigned short* w2p = W2 + (size_t)col * N1 + 8 * h;
#pragma unroll
    for (int k = 0; k < N1 / 16; ++k) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(sH1 + r32 * N1 + (((2 * k + h) ^ (r32 & 15)) * 8));
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(w2p + 16 * k);
      a2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, a2, 0, 0, 0);
    }
    const float bias = b2[col];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = (i >> 2) * 8 + h * 4 + (i & 3);
      float v = a2[i] + bias;
      v = v > 0.f ? v : 0.f;
      sH2[row * N2 + (((col >> 3) ^ (row & 7)) * 8) + (col & 7)] = bf16_bits(v);
    }
  }
  __syncthreads();
  auto h2 = [&](int row, int j) { return bf16_float(sH2[row * N2 + (((j >> 3) ^ (row & 7)) * 8) + (j & 7)]); };

  // ---- head: thread (q, row), then the loss and its gradient per row
  if (tid < 3 * TR) {
    const int q = tid / TR, row = tid % TR;
    float s = sW[3 * N2 + q];
#pragma unroll 16
    for (int j = 0; j < N2; ++j) s += sW[q * N2 + j] * h2(row, j);
    sO[q][row] = s;
  }
  __syncthreads();
  if (tid < 64) {
    const int b = m0 + r32;
    float d0 = 0.f, d1 = 0.f, d2 = 0.f, l = 0.f;
    if (h == 0 && b < n) {
      const float o2 = sO[2][r32];
      const float ex = sO[0][r32] - lab[2 * b], ey = sO[1][r32] - lab[2 * b + 1];
      const float t = (fmaxf(fabsf(ex), fabsf(ey)) <= half_step) ? 1.f : 0.f;
      const float sp = 1.f / (1.f + expf(-o2));
      const float inv = 1.f / (float)n;
      // BCE with logits, stable form: max(o,0) - o t + log(1 + exp(-|o|))
      l = wv * (ex * ex + ey * ey) * inv + (fmaxf(o2, 0.f) - o2 * t + log1pf(expf(-fabsf(o2)))) * inv;
      d0 = 2.f * wv * ex * inv;
      d1 = 2.f * wv * ey * inv;
      d2 = (sp - t) * inv;
    }
    if (h == 0) {
      sD[0][r32] = d0;
      sD[1][r32] = d1;
      sD[2][r32] = d2;
    }
    float s[4] = {d0, d1, d2, l};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      for (int off = 32; off > 0; off >>= 1) s[q] += __shfl_xor(s[q], off, 64);
      if (lane == 0) P[P_DB3 + q] = s[q];
    }
  }
  __syncthreads();

  // ---- dH2 (BF16, masked by H2 > 0): thread = one 16-byte chunk of a row
  {
    const int row = tid >> 3, c = tid & 7;
    const float d0 = sD[0][row], d1 = sD[1][row], d2 = sD[2][row];
    unsigned int u[4];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int j = 8 * c + e;
      const float g = sW[j] * d0 + sW[64 + j] * d1 + sW[128 + j] * d2;
      const unsigned int v = bf16_bits(h2(row, j) > 0.f ? g : 0.f);
      u[e >> 1] = (e & 1) ? (u[e >> 1] | (v << 16)) : v;
    }
    const uint4 o = make_uint4(u[0], u[1], u[2], u[3]);
    *reinterpret_cast<uint4*>(sG + row * N2 + ((c ^ (row & 7)) * 8)) = o;
    if (m0 + row < n) *reinterpret_cast<uint4*>(dH2 + (size_t)(m0 + row) * N2 + c * 8) = o;
  }
  if (tid < 3 * N2) {
    const int q = tid / N2, j = tid % N2;
    float s = 0.f;
    for (int r0 = 0; r0 < rows; r0 += 8)
#pragma unroll
      for (int r = r0; r < r0 + 8; ++r) s += sD[q][r] * h2(r, j);
    P[tid] = s;
  }
  __syncthreads();

  // ---- dH1 = (dH2 W2) masked by H1 > 0; column sums of dH2 and dH1
  if (tid < N2) {
    float s = 0.f;
    for (int r0 = 0; r0 < rows; r0 += 8)
#pragma unroll
      for (int r = r0; r < r0 + 8; ++r) s += bf16_float(sG[r * N2 + (((tid >> 3) ^ (r & 7)) * 8) + (tid & 7)]);
    P[P_DB2 + tid] = s;
  }
  f32x16 ag;
#pragma unroll
  for (int i = 0; i < 16; ++i) ag[i] = 0.f;
#pragma unroll
  for (int s = 0; s < N2 / 16; ++s) {
    const bf16x8 a = *reinterpret_cast<const bf16x8*>(sG + r32 * N2 + (((2 * s + h) ^ (r32 & 7)) * 8));
    ag = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, bt[s], ag, 0, 0, 0);
  }
  float cs = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = (i >> 2) * 8 + h * 4 + (i & 3);
    const int at = row * N1 + (((col >> 3) ^ (row & 15)) * 8) + (col & 7);
    const unsigned short v = bf16_bits((bf16_float(sH1[at]) > 0.f) ? ag[i] : 0.f);
    sX[at] = v;
    cs += row < rows ? bf16_float(v) : 0.f;
  }
  cs += __shfl_xor(cs, 32, 64);
  if (h == 0) P[P_DB1 + col] = cs;
  __syncthreads();
  for (int i = tid; i < TR * N1 / 8; i += 256) {
    const int row = i >> 4, c = i & 15;
    if (m0 + row < n)
      *reinterpret_cast<uint4*>(dH1 + (size_t)(m0 + row) * N1 + c * 8) =
          *reinterpret_cast<const uint4*>(sX + row * N1 + ((c ^ (row & 15)) * 8));
  }
}

// C[128][64] partial of A^T B over one chunk of samples: A [n][128], B [n][64 of
// ldb].  blockIdx.x < N0 / 64: dW1 (A = dH1, B = 64 feature columns); the last:
// dW2^T (A = H1, B = dH2).  Samples are the contraction, so both operands are
// transposed on the way into LDS: a thread reads two columns of eight
// samples (rows of 128 or 256 contiguous bytes across lanes) and writes each
// column's eight values as one 16-byte piece.
__global__ void __launch_bounds__(256) k_train_wgrad(const unsigned short* __restrict__ X,
                                                     const unsigned short* __restrict__ H1,
                                                     const unsigned short* __restrict__ dH2,
                                                     const unsigned short* __restrict__ dH1, int n, int rows,
                                                     float* __restrict__ p1, float* __restrict__ p2) {
  __shared__ __align__(16) unsigned short sA[N1 * KLD];
  __shared__ __align__(16) unsigned short sB[64 * KLD];
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, h = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool first = blockIdx.x < N0 / 64;
  const unsigned short* A = first ? dH1 : H1;
  const unsigned short* B = first ? X + 64 * blockIdx.x : dH2;
  const int ldb = first ? N0 : N2;
  const int k_begin = blockIdx.y * rows, k_end = min(n, k_begin + rows);
  unsigned int va[2][8], vb[8];
  auto load = [&](int k0) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int task = tid + 256 * t, kg = task >> 6, cp = task & 63;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int k = k0 + 8 * kg + e;
        va[t][e] = (k < k_end) ? *reinterpret_cast<const unsigned int*>(A + (size_t)k * N1 + 2 * cp) : 0u;
      }
    }
    const int kg = tid >> 5, cp = tid & 31;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = k0 + 8 * kg + e;
      vb[e] = (k < k_end) ? *reinterpret_cast<const unsigned int*>(B + (size_t)k * ldb + 2 * cp) : 0u;
    }
  };
  auto store = [&](unsigned short* s, int cp, int kg, const unsigned int (&v)[8]) {
    uint4 lo, hi;
    lo = make_uint4(__builtin_amdgcn_perm(v[1], v[0], 0x05040100), __builtin_amdgcn_perm(v[3], v[2], 0x05040100),
                    __builtin_amdgcn_perm(v[5], v[4], 0x05040100), __builtin_amdgcn_perm(v[7], v[6], 0x05040100));
    hi = make_uint4(__builtin_amdgcn_perm(v[1], v[0], 0x07060302), __builtin_amdgcn_perm(v[3], v[2], 0x07060302),
                    __builtin_amdgcn_perm(v[5], v[4], 0x07060302), __builtin_amdgcn_perm(v[7], v[6], 0x07060302));
    *reinterpret_cast<uint4*>(s + (2 * cp) * KLD + 8 * kg) = lo;
    *reinterpret_cast<uint4*>(s + (2 * cp + 1) * KLD + 8 * kg) = hi;
  };
  f32x16 acc[2];
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[u][i] = 0.f;
  load(k_begin);
  for (int k0 = k_begin; k0 < k_end; k0 += KB) {
    __syncthreads();                             // the previous step's reads are done
    store(sA, tid & 63, tid >> 6, va[0]);
    store(sA, tid & 63, (tid >> 6) + 4, va[1]);
    store(sB, tid & 31, tid >> 5, vb);
    __syncthreads();
    if (k0 + KB < k_end) load(k0 + KB);
#pragma unroll
    for (int s = 0; s < KB / 16; ++s) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(sA + (32 * w + r32) * KLD + 16 * s + 8 * h);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(sB + (32 * u + r32) * KLD + 16 * s + 8 * h);
        acc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[u], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int m = 32 * w + (i >> 2) * 8 + h * 4 + (i & 3), c = 32 * u + r32;
      if (first) p1[((size_t)blockIdx.y * N1 + m) * N0 + 64 * blockIdx.x + c] = acc[u][i];
      else p2[((size_t)blockIdx.y * N2 + c) * N1 + m] = acc[u][i];
    }
}

// Sums of the partials in ascending order.  Blocks [0, NB_W): four weights per
// thread over the chunks; then one wavefront per small sum over the tiles.
constexpr int NB_W1 = N1 * N0 / 4 / 256, NB_W = NB_W1 + N2 * N1 / 4 / 256;
__global__ void __launch_bounds__(256) k_train_reduce(const float* __restrict__ p1, const float* __restrict__ p2,
                                                      int chunks, const float* __restrict__ part, int tiles,
                                                      float* __restrict__ dW1, float* __restrict__ dW2,
                                                      float* __restrict__ dW3, float* __restrict__ db1,
                                                      float* __restrict__ db2, float* __restrict__ db3,
                                                      float* __restrict__ loss) {
  if (blockIdx.x < NB_W) {
    const bool first = blockIdx.x < NB_W1;
    const size_t i = (size_t)(first ? blockIdx.x : blockIdx.x - NB_W1) * 256 + threadIdx.x;
    const size_t stride = (first ? N1 * N0 : N2 * N1) / 4;
    const float4* src = reinterpret_cast<const float4*>(first ? p1 : p2) + i;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int c = 0; c < chunks; ++c) {
      const float4 v = src[c * stride];
      s = make_float4(s.x + v.x, s.y + v.y, s.z + v.z, s.w + v.w);
    }
    float* dst = (first ? dW1 : dW2) + 4 * i;
    dst[0] = s.x;
    dst[1] = s.y;
    dst[2] = s.z;
    dst[3] = s.w;
    return;
  }
  const int j = (blockIdx.x - NB_W) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= P_N) return;
  float s = 0.f;
  for (int t = lane; t < tiles; t += 64) s += part[(size_t)t * P_N + j];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (lane != 0) return;
  if (j < P_DB3) dW3[j] = s;
  else if (j < P_LOSS) db3[j - P_DB3] = s;
  else if (j == P_LOSS) loss[0] = s;
  else if (j < P_DB1) db2[j - P_DB2] = s;
  else db1[j - P_DB1] = s;
}

// Sections of the caller's work buffer, each starting on a 256-byte boundary.
struct Work {
  size_t H1, dH2, dH1, part, p1, p2, bytes;
  int chunks, rows, tiles;
};
static Work work_of(int n) {
  Work k;
  k.tiles = (n - 1) / TR + 1;                    // (n >= 8; n + TR may not be an int)
  const int blocks = (n - 1) / KB + 1;           // steps of KB samples
  k.rows = ((blocks - 1) / WG_MAX_CHUNKS + 1) * KB;
  k.chunks = (n - 1) / k.rows + 1;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    const size_t at = o;
    o += (bytes + 255) & ~size_t(255);
    return at;
  };
  k.H1 = take((size_t)n * N1 * 2);
  k.dH2 = take((size_t)n * N2 * 2);
  k.dH1 = take((size_t)n * N1 * 2);
  k.part = take((size_t)k.tiles * P_N * 4);
  k.p1 = take((size_t)k.chunks * N1 * N0 * 4);
  k.p2 = take((size_t)k.chunks * N2 * N1 * 4);
  k.bytes = o;
  return k;
}

}  // namespace train
}  // namespace rmdf

using namespace rmdf::train;

extern "C" {

rmdf_status rmdf_mlp_grads_work(int n, size_t* bytes) {
  if (n < 8 || (n % 8) || !bytes) return RMDF_E_INVAL;
  *bytes = work_of(n).bytes;
  return RMDF_OK;
}

rmdf_status rmdf_mlp_grads(const void* X, const float* labels, int n, const void* W1, const float* b1, const void* W2,
                           const float* b2, const float* W3, const float* b3, float wv, float half_step, float* dW1,
                           float* db1, float* dW2, float* db2, float* dW3, float* db3, float* loss, void* work,
                           size_t work_bytes, void* stream) {
  auto misaligned = [](const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; };
  if (!X || !labels || n < 8 || (n % 8) || !W1 || !b1 || !W2 || !b2 || !W3 || !b3 || !dW1 || !db1 || !dW2 || !db2 ||
      !dW3 || !db3 || !loss || !work || misaligned(X, 16) || misaligned(W1, 16) || misaligned(W2, 16) ||
      misaligned(work, 256))
    return RMDF_E_INVAL;
  const Work k = work_of(n);
  if (work_bytes < k.bytes) return RMDF_E_INVAL;
  const hipStream_t s = static_cast<hipStream_t>(stream);
  char* base = static_cast<char*>(work);
  unsigned short* H1 = reinterpret_cast<unsigned short*>(base + k.H1);
  unsigned short* dH2 = reinterpret_cast<unsigned short*>(base + k.dH2);
  unsigned short* dH1 = reinterpret_cast<unsigned short*>(base + k.dH1);
  float* part = reinterpret_cast<float*>(base + k.part);
  float* p1 = reinterpret_cast<float*>(base + k.p1);
  float* p2 = reinterpret_cast<float*>(base + k.p2);
  const unsigned short* x = static_cast<const unsigned short*>(X);
  hipLaunchKernelGGL(k_train_rows, dim3(k.tiles), dim3(256), 0, s, x, labels, n, (const unsigned short*)W1, b1,
                     (const unsigned short*)W2, b2, W3, b3, wv, half_step, H1, dH2, dH1, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return RMDF_E_DEVICE;
  hipLaunchKernelGGL(k_train_wgrad, dim3(N0 / 64 + 1, k.chunks), dim3(256), 0, s, x, H1, dH2, dH1, n, k.rows, p1, p2);
  if ((e = hipGetLastError()) != hipSuccess) return RMDF_E_DEVICE;
  hipLaunchKernelGGL(k_train_reduce, dim3(NB_W + (P_N + 3) / 4), dim3(256), 0, s, p1, p2, k.chunks, part, k.tiles, dW1,
                     dW2, dW3, db1, db2, db3, loss);
  return hipGetLastError() == hipSuccess ? RMDF_OK : RMDF_E_DEVICE;
}

}  // extern "C"
