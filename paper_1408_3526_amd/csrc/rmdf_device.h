// rmdf_device.h - device-side building blocks of the recursive
// multidimensional prediction-error filter (Kennedy, arXiv:1408.3526): complex
// helpers, the row sliding-DFT chunk and the generic per-pixel work tile.
// Included by every translation unit that launches them (no relocatable
// device code is used).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "rmdf_kernels.h"
#include "rmdf_refine.h"
#include "rmdf_wave.h"

namespace rmdf {

static __device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
static __device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
static __device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
static __device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
static __device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }

// A column of N complex values in LDS at a 16-byte aligned address: 16-byte
// accesses, the last value of an odd N alone.
template <int N>
static __device__ __forceinline__ void ld_col(const lds_v2* p, float2 (&v)[N]) {
#pragma unroll
  for (int k = 0; k + 1 < N; k += 2) {
    const float4 q = ld4(p + k);
    v[k] = make_float2(q.x, q.y);
    v[k + 1] = make_float2(q.z, q.w);
  }
  if (N % 2) v[N - 1] = ld2(p + N - 1);
}
template <int N>
static __device__ __forceinline__ void st_col(lds_v2* p, const float2 (&v)[N]) {
#pragma unroll
  for (int k = 0; k + 1 < N; k += 2) st4(p + k, v[k].x, v[k].y, v[k + 1].x, v[k + 1].y);
  if (N % 2) st2(p + N - 1, v[N - 1]);
}

template <int MX>
struct RowShape {
  static constexpr int NP = (MX % 2 == 0) ? MX / 2 : (MX + 1) / 2;
  static constexpr size_t SMEM = sizeof(float) * (MX + RCX) + sizeof(float2) * (NP * RCX + MX);
};

// One (row y, chunk of RCX columns starting at x0).  Non-finite samples are
// read as 0; when `nonfinite` is given, those of the chunk's own columns are
// counted; when `copy_to` is given, the chunk's own columns are stored there
// (non-finite ones as 0): the frame's copy into the delay ring.
// DIRECT: every output is the direct Mx-term DFT sum of its window (no comb,
// no resonator): the non-recursive form of the same row spectrum.
template <int MX, bool DIRECT = false>
static __device__ void row_chunk(const float* __restrict__ f, float2* __restrict__ rs, const float2* __restrict__ twx,
                          int H, int W, int y, int x0, char* smem, unsigned long long* nonfinite,
                          float* __restrict__ copy_to = nullptr) {
  constexpr int NP = RowShape<MX>::NP;
  constexpr int NSEG = RCX / RSEG;
  constexpr bool EVEN = (MX % 2 == 0);
  float* s_in = reinterpret_cast<float*>(smem);                          // [MX + RCX]
  float2* s_out = reinterpret_cast<float2*>(smem + sizeof(float) * (MX + RCX));   // [NP][RCX]
  float2* s_tw = s_out + NP * RCX;                                       // [MX]
  const float* row = f + (size_t)y * W;
  int bad = 0;
  for (int i = threadIdx.x; i < MX + RCX; i += blockDim.x) {
    const int xx = x0 - MX + i;
    float v = (xx >= 0 && xx < W) ? row[xx] : 0.0f;
    if (!isfinite(v)) {
      v = 0.0f;
      bad += (i >= MX) ? 1 : 0;     // count the chunk's own columns only
    }
    s_in[i] = v;
    if (copy_to != nullptr && i >= MX && xx < W) copy_to[(size_t)y * W + xx] = v;
  }
  for (int i = threadIdx.x; i < MX; i += blockDim.x) s_tw[i] = twx[i];
  if (nonfinite) {
    // the wavefront's count, reduced only where it has non-finite samples
    if (__ballot(bad != 0)) {
      int tot = bad;
      for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
      if ((threadIdx.x & 63) == 0) atomicAdd(nonfinite, (unsigned long long)tot);
    }
  }
  __syncthreads();
  const float inv = rsqrtf((float)MX);
  if (DIRECT && threadIdx.x < NP * NSEG) {
    // A(kx; x) = sum_m w^(kx m) I(x - m), m = 0 .. Mx - 1, for each column
    const int p = threadIdx.x / NSEG, sg = threadIdx.x % NSEG;
    const int xs = sg * RSEG;
    for (int i = 0; i < RSEG; ++i) {
      const int xi = xs + i;
      if (p == 0) {
        float a0 = 0.f, ah = 0.f;
        for (int m = 0; m < MX; ++m) {
          const float v = s_in[MX + xi - m];
          a0 += v;
          ah += (m & 1) ? -v : v;
        }
        s_out[xi] = EVEN ? make_float2(a0 * inv, ah * inv) : make_float2(a0 * inv, 0.f);
      } else {
        float2 acc = make_float2(0.f, 0.f);
        for (int m = 0; m < MX; ++m) {
          const float v = s_in[MX + xi - m];
          const float2 w = s_tw[(p * m) % MX];
          acc.x += w.x * v;
          acc.y += w.y * v;
        }
        s_out[p * RCX + xi] = cscale(acc, inv);
      }
    }
  } else if (threadIdx.x < NP * NSEG) {
    const int p = threadIdx.x / NSEG, sg = threadIdx.x % NSEG;
    const int xs = sg * RSEG;             // segment start relative to x0
    if (p == 0) {
      // kx = 0 (pole 1) and, for even Mx, kx = Mx/2 (pole -1): real resonators
      float a0 = 0.f, ah = 0.f;
      for (int m = 0; m < MX; ++m) {
        const float v = s_in[MX + xs - 1 - m];
        a0 += v;
        ah += (m & 1) ? -v : v;
      }
      for (int i = 0; i < RSEG; ++i) {
        const int xi = xs + i;
        const float comb = s_in[MX + xi] - s_in[xi];
        a0 = a0 + comb;
        ah = -ah + comb;
        s_out[xi] = EVEN ? make_float2(a0 * inv, ah * inv) : make_float2(a0 * inv, 0.f);
      }
    } else {
      float2 acc = make_float2(0.f, 0.f);
      for (int m = 0; m < MX; ++m) {
        const float v = s_in[MX + xs - 1 - m];
        const float2 w = s_tw[(p * m) % MX];
        acc.x += w.x * v;
        acc.y += w.y * v;
      }
      const float2 w1 = s_tw[p];
      for (int i = 0; i < RSEG; ++i) {
        const int xi = xs + i;
        const float comb = s_in[MX + xi] - s_in[xi];
        acc = cmul(w1, acc);
        acc.x += comb;
        s_out[p * RCX + xi] = cscale(acc, inv);
      }
    }
  }
  __syncthreads();
  // row spectra layout [y][x][plane]: the planes of a pixel are adjacent, so
  // the per-pixel kernels read one contiguous run per row and workgroup
  for (int i = threadIdx.x; i < NP * RCX; i += blockDim.x) {
    const int xi = i / NP, p = i % NP;
    if (x0 + xi < W) rs[((size_t)y * W + x0 + xi) * NP + p] = s_out[p * RCX + xi];
  }
}

// ---------------------------------------------------------------------------
// Per-pixel kernel (generic: every compiled window shape).
//
// A wavefront owns PPW anchors (one, or two of the 8x8x4 window) and walks
// down a tile of rows; the four wavefronts of a workgroup share only the
// weight tables.  A lane holds CPL (plane, ky) columns of the Hermitian half
// of its anchor's spectrum.  Since no stage leaves its wavefront, there is no
// workgroup barrier after the tables; a row's smoothed R is loaded before the
// flow stages instead of inside the candidate loop (one memory latency a row
// instead of one per 64 candidates), and the planes beyond the half spectrum
// are stored as mirrors so that the Hann pass along kx reads fixed offsets.
// Against the form with workgroup barriers and loads in the candidate loop
// (us per frame, output and velocity read): 9x9x5 640x512 941 -> 470 (4.25 TB/s of
// cache-line traffic; the state and R alone would take 370 at the copy rate), 8x8x4
// 640x512 397 -> 217, 16x16x8 319x241 with 33x33 candidates 1243 -> 521 (3.8 TB/s,
// two wavefronts per SIMD; 391), the paper's 64x64 frames 24.4 -> 16.2 (with the
// kernel left out, launches and host calls take 12 to 13).  Of these, row spectra
// computed in the tiles give 16, 0, 10 and 1.8, the state moved in contiguous runs,
// non-temporal, 32, 22, 93 and 1.1, and the read-outs' shared launch 2 of the last.
template <int MX, int MY, int MZ>
struct Shape {
  static constexpr bool EVEN = (MX % 2 == 0);
  static constexpr int NP = EVEN ? MX / 2 : (MX + 1) / 2;   // stored kx planes
  static constexpr int NXH = MX / 2 + 1;                    // kx = 0 .. Mx/2
  static constexpr int NCOL = NP * MY;                      // (plane, ky) columns
  static constexpr int LPP = NCOL <= 32 ? 32 : 64;          // lanes per anchor
  static constexpr int CPL = (NCOL + 63) / 64;              // columns per lane
  static constexpr int PPW = 64 / LPP;                      // anchors per wavefront
  static constexpr int WAVES = 4;
  static constexpr int PPB = WAVES * PPW;                   // anchors per workgroup
  // LDS rows are padded so that neighbouring lanes' 16-byte accesses fall on
  // distinct banks (row strides of 12, 20 and 36 words over 64 banks)
  static constexpr int MZP = MZ == 8 ? 10 : 6;              // a staged column's kz values
  static constexpr int MYQ = (MY + 1) / 2 * 2;              // Q row (one kx)
  static constexpr int MYT = MY == 16 ? 18 : 10;            // weights of one l_y
  static constexpr int NXT = NXH == 9 ? 10 : 6;             // T row (one l_y); weights of one l_x
  static constexpr int S_ELEMS = (NXH + 2) * MY * MZP;      // staged planes kx = -1 .. Mx/2 + 1 (float2)
  static constexpr int QT_ELEMS = NXH * MYQ + NVY_MAX * NXT;
  static constexpr int W_ELEMS = PPW * (S_ELEMS > QT_ELEMS ? S_ELEMS : QT_ELEMS);   // per wavefront
  static constexpr int MXQ = (MX + 1) / 2 * 2;
  // one column per lane: where the operands of each candidate lie; whole rounds (and
  // whole groups of NB rounds)
  static constexpr int NB = 6;                              // candidates per lane whose smoothed R is loaded together
  static constexpr int WC = CPL > 1 ? 0 : (NVX_MAX * NVY_MAX + NB * LPP - 1) / (NB * LPP) * (NB * LPP) + LPP;
  static constexpr int TAB_ELEMS = NVY_MAX * MYT + NVX_MAX * NXT + MYQ + MXQ + (NVX_MAX + NVY_MAX + 3) / 4 * 2 + WC / 2;
  // row spectra of SR rows and the My above them for the workgroup's anchors;
  // the samples they come from (one resonator segment and the Mx before it)
  // lie in the wavefronts' staging area while it is idle
  static constexpr int SR = PPW == 2 ? 24 : 32;             // (8x8x4: four workgroups' LDS on a CU)
  static constexpr int RS_ELEMS = ((SR + MY) * PPB * NP + 1) / 2 * 2;
  static constexpr int SW = MX + RSEG + (MX % 2 ? 3 : 4);   // floats per sample row: 16-byte aligned, spread over banks
  static_assert((SR + MY) * SW <= 2 * WAVES * W_ELEMS, "samples fit the staging area");
  static constexpr size_t SMEM = sizeof(float2) * (TAB_ELEMS + WAVES * W_ELEMS);
  static constexpr size_t SMEM_ROWS = SMEM + sizeof(float2) * RS_ELEMS;   // tiles that compute their row spectra
};


// Eq. (8) at bin (kx, ky, kz) for a continuous velocity (the spatial Dirichlet
// factors select kx' = kx, ky' = ky at the bins), times sqrt(Mz) since the
// state holds S / sqrt(Mz):
//   D_Mz(kz/Mz + phi) / sqrt(Mx My) * exp(j pi [-2(kx m'x/Mx + ky m'y/My)
//   + 2 phi (m't - Dz) - 2 kz Dz/Mz]),  phi = vx kx/Mx + vy ky/My.
template <int MX, int MY, int MZ>
static __device__ __forceinline__ float2 coeff_at(int kx, int ky, int kz, float vx, float vy, int dx, int dy, int dt) {
  const float Dz = 0.5f * (MZ - 1);
  const float phi = vx * kx * (1.0f / MX) + vy * ky * (1.0f / MY);
  const float w = kz * (1.0f / MZ) + phi;
  const float rw = rintf(w);
  float D;
  if (fabsf(w - rw) < 1e-5f) D = (((int)rw * (MZ - 1)) & 1) ? -1.f : 1.f;
  else D = sinpif(MZ * w) / (MZ * sinpif(w));
  const float ph = -2.f * (kx * (float)dx / MX + ky * (float)dy / MY) + 2.f * phi * (dt - Dz) - 2.f * kz * Dz / MZ;
  float sn, cs;
  sincospif(ph, &sn, &cs);
  const float g = D * (1.0f / sqrtf((float)(MX * MY)));
  return make_float2(g * cs, g * sn);
}

// Row spectra of rows [ya, ya + rows) for the PPB columns from x0 (all in one
// resonator segment: PPB divides RSEG) into s_rs[row][column][plane]: the
// values of row_chunk, bit for bit (the segment's direct-DFT seed, then the
// comb and resonator up to each column).  Non-finite samples read as 0; those
// of rows from yc on are counted, and the columns of those rows are stored in
// the frame's delay-ring slot.  All threads of the workgroup call it; the caller
// has a barrier before (s_in idle) and gets one after.
template <int MX, int MY, int MZ>
static __device__ __forceinline__ void tile_rows(const PixArgs& a, int x0, int ya, int yc, int rows, lds_float* s_in,
                                                 const lds_v2* s_twx, lds_v2* s_rs) {
  const float* __restrict__ f = a.frame;
  float* __restrict__ slot = a.slot;
  using SH = Shape<MX, MY, MZ>;
  constexpr int NP = SH::NP, SW = SH::SW, PPB = SH::PPB;
  const int xs = x0 / RSEG * RSEG, o0 = x0 - xs;            // segment start; first own column in it
  int bad = 0;
  for (int i = threadIdx.x; i < rows * (MX + RSEG); i += 256) {
    const int row = i / (MX + RSEG), c = i - row * (MX + RSEG);
    const int yy = ya + row, xx = xs - MX + c;
    float v = (yy >= 0 && xx >= 0 && xx < a.W) ? f[(size_t)yy * a.W + xx] : 0.0f;
    const bool own = yy >= yc && c >= MX + o0 && c < MX + o0 + PPB && xx < a.W;
    if (!isfinite(v)) {
      v = 0.0f;
      bad += own ? 1 : 0;
    }
    s_in[row * SW + c] = v;
    if (own) slot[(size_t)yy * a.W + xx] = v;
  }
  // the wavefront's count, reduced only where it has non-finite samples
  if (__ballot(bad != 0)) {
    int tot = bad;
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if ((threadIdx.x & 63) == 0) atomicAdd(a.nonfinite, (unsigned long long)tot);
  }
  __syncthreads();
  const float inv = rsqrtf((float)MX);
  // one (plane, row) per thread, plane by plane; its samples and twiddles are
  // all read before the recursion, whose steps then wait for nothing
  for (int t = threadIdx.x; t < rows * NP; t += 256) {
    const int p = t / rows, row = t - p * rows;
    float in[MX + RSEG + 3];
#pragma unroll
    for (int c = 0; c < MX + RSEG; c += 4) {
      const v4f q = *reinterpret_cast<const lds_v4*>(s_in + row * SW + c);
      in[c] = q.x;
      in[c + 1] = q.y;
      in[c + 2] = q.z;
      if (c + 3 < MX + RSEG + 3) in[c + 3] = q.w;
    }
    lds_v2* out = s_rs + row * (PPB * NP) + p;
    if (p == 0) {
      float a0 = 0.f, ah = 0.f;
#pragma unroll
      for (int m = 0; m < MX; ++m) {
        const float v = in[MX - 1 - m];
        a0 += v;
        ah += (m & 1) ? -v : v;
      }
#pragma unroll
      for (int i = 0; i < RSEG; ++i) {
        if (i < o0 + PPB) {                                // uniform
          const float comb = in[MX + i] - in[i];
          a0 = a0 + comb;
          ah = -ah + comb;
          if (i >= o0) st2(out + (i - o0) * NP, SH::EVEN ? make_float2(a0 * inv, ah * inv) : make_float2(a0 * inv, 0.f));
        }
      }
    } else {
      float2 w[MX];
      int e = 0;                                           // (p m) mod Mx
#pragma unroll
      for (int m = 0; m < MX; ++m) {
        w[m] = ld2(s_twx + e);
        e += p;
        e = (e >= MX) ? e - MX : e;
      }
      float2 acc = make_float2(0.f, 0.f);
#pragma unroll
      for (int m = 0; m < MX; ++m) {
        const float v = in[MX - 1 - m];
        acc.x += w[m].x * v;
        acc.y += w[m].y * v;
      }
#pragma unroll
      for (int i = 0; i < RSEG; ++i) {
        if (i < o0 + PPB) {                                // uniform
          const float comb = in[MX + i] - in[i];
          acc = cmul(w[1], acc);
          acc.x += comb;
          if (i >= o0) st2(out + (i - o0) * NP, cscale(acc, inv));
        }
      }
    }
  }
  __syncthreads();
}

// One work tile: PPB adjacent anchor columns starting at xb*PPB, rows
// [yb*TY, yb*TY + TY).  All 256 threads of the block must call it.
// REFINED: velocity mode 3 (its eq. 8 per bin needs many registers).  OWN_ROWS:
// the tile computes its row spectra from a.frame, and stores its part of the
// frame into the delay ring; otherwise they come from the row kernel (a.rs).
template <int MX, int MY, int MZ, bool REFINED = false, bool OWN_ROWS = false>
static __device__ __forceinline__ void pixel_tile(const PixArgs& a, const float* ring_delayed, int xb, int yb, char* smem) {
  using SH = Shape<MX, MY, MZ>;
  constexpr int NP = SH::NP, NXH = SH::NXH, NCOL = SH::NCOL, LPP = SH::LPP, CPL = SH::CPL, PPW = SH::PPW;
  constexpr int MZP = SH::MZP, MYQ = SH::MYQ, MYT = SH::MYT, NXT = SH::NXT, NB = SH::NB;
  constexpr bool EVEN = SH::EVEN;
  lds_v2* s_tauy = (lds_v2*)smem;                // [nvy][MYT]
  lds_v2* s_taux = s_tauy + NVY_MAX * MYT;       // [nvx][NXT]
  lds_v2* s_twy = s_taux + NVX_MAX * NXT;        // [MY]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ps = (PPW == 1) ? 0 : lane / LPP;
  const int cl = (PPW == 1) ? lane : lane % LPP;           // lane within the anchor
  lds_v2* s_twx = s_twy + MYQ;                   // [MX]
  lds_float* s_gx = (lds_float*)(s_twx + SH::MXQ);   // [nvx], then gy [nvy]
  lds_u32* s_itC = (lds_u32*)(s_twx + SH::MXQ + (NVX_MAX + NVY_MAX + 3) / 4 * 2);   // [WC] candidates
  lds_v2* s_rs = (lds_v2*)(s_itC + SH::WC);      // [SR + MY][PPB][NP]
  lds_v2* s_w0 = s_rs + (OWN_ROWS ? SH::RS_ELEMS : 0);
  lds_v2* s_w = s_w0 + wv * SH::W_ELEMS + ps * (SH::W_ELEMS / PPW);
  const int nvx = a.nvx, nvy = a.nvy, nv = a.nv;
  for (int i = tid; i < MY; i += 256) s_twy[i] = v2f{a.twy[i].x, a.twy[i].y};
  for (int i = tid; i < nvy * MY; i += 256) s_tauy[i / MY * MYT + i % MY] = v2f{a.tauy[i].x, a.tauy[i].y};
  for (int i = tid; i < nvx * NXH; i += 256) s_taux[i / NXH * NXT + i % NXH] = v2f{a.taux[i].x, a.taux[i].y};
  for (int i = tid; i < MX; i += 256) s_twx[i] = v2f{a.twx[i].x, a.twx[i].y};
  for (int i = tid; i < nvx + nvy; i += 256) s_gx[i] = (i < nvx) ? a.gx[i] : a.gy[i - nvx];
  if (CPL == 1) {
    // byte offsets of candidate (iy, ix): T row, weight row (places past the grid
    // repeat the last one)
    const float inv_x = 1.0f / (float)nvx;
    for (int i = tid; i < (nv + LPP - 1) / LPP * LPP + LPP; i += 256) {
      const int w = min(i, nv - 1), iy = (int)(((float)w + 0.5f) * inv_x), ix = w - iy * nvx;
      s_itC[i] = (unsigned)(iy * NXT * 8) | (unsigned)(ix * NXT * 8) << 16;
    }
  }

  const int y0 = yb * a.TY;
  const int y1 = min(a.H, y0 + a.TY);
  const int xw = xb * SH::PPB + wv * PPW;         // the wavefront's first anchor
  const bool active = xw < a.W;
  if (!OWN_ROWS) {
    __syncthreads();                             // the only workgroup barrier
    if (!active) return;                         // (OWN_ROWS: an idle wavefront still stages rows)
  }
  // the second anchor of a pair past the frame's edge repeats the last column
  // without storing; lanes past the last column repeat it
  const bool px_ok = xw + ps < a.W;
  const int dxw = px_ok ? ps : max(a.W - 1 - xw, 0);
  const int x = xw + dxw;
  int p[CPL], ky[CPL], col[CPL];
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    col[j] = min(cl + 64 * j, NCOL - 1);
    p[j] = col[j] / MY;
    ky[j] = col[j] % MY;
  }
  // addresses: a base per row (the same in all lanes) and a 32-bit offset per lane
  unsigned ro[CPL];
  const lds_v2* rs_own[CPL];                     // this column's row spectrum, row 0 of s_rs
#pragma unroll
  for (int j = 0; j < CPL; ++j) {
    ro[j] = (unsigned)(dxw * NP + p[j]) * 8u;
    rs_own[j] = s_rs + (wv * PPW + dxw) * NP + p[j];
  }
  constexpr int RSR = SH::PPB * NP;              // s_rs row
  const unsigned qo = (unsigned)(dxw * nv) * 4u;
  // The state in memory is [plane][ky][kz], a column's kz values side by side: a
  // lane's own column would make accesses of 16 bytes at strides of 32 to 64, each
  // touching every line of the anchor's run (9x9x5 640x512: 119 cache write requests
  // an anchor, 61 when contiguous; 505 -> 475 us).  So the state moves between memory
  // and LDS in contiguous runs, one piece of VL values per lane, and between LDS and
  // registers by column.  Non-temporal: a stream of less than 256 MB that runs
  // alone could stay in the chip's last cache (8x8x4 320x256 with detection 63.5 us
  // cached, 70.2 this way), but streams that take turns could not (75.7 and 70.5), nor
  // larger ones (8x8x4 640x512 alone 224 and 206).
  constexpr int VL = (MZ % 2 == 0) ? 2 : 1;      // float2 per piece
  constexpr int CS = (MZ % 2 == 0) ? MZP : MZ;   // column stride in LDS (padded: distinct banks)
  constexpr int NPC = NCOL * MZ / VL, NL = (NPC + LPP - 1) / LPP;   // pieces per anchor and lane
  // (pieces past the last: the descriptors of load_row and of the stores end with
  // the anchors' states, and in LDS they lie within the staging area)
  static_assert(NL * LPP * VL <= SH::W_ELEMS / PPW && (PPW == 1 || NPC % LPP == 0), "pieces past the last");
  const unsigned po = (unsigned)((dxw * NPC + cl) * VL) * 8u;
  const int pl = (MZ % 2 == 0) ? cl * VL / MZ * CS + cl * VL % MZ : cl;
  constexpr int PLS = (MZ % 2 == 0) ? LPP * VL / MZ * CS : LPP;   // LDS distance of a lane's pieces
  const unsigned st_bytes = (unsigned)(NCOL * MZ * 8 * (PPW == 1 ? 1 : min(PPW, max(a.W - xw, 0))));

  // Staged planes: (kx in [-1, NXH], ky, kz) at s_w[((kx + 1) * MY + ky) * MZP + kz]
  auto sidx = [](int kx, int kyy) { return ((kx + 1) * MY + kyy) * MZP; };
  lds_v2* s_q = s_w;                             // [NXH][MYQ] after Hann along kx
  lds_v2* s_t = s_w + NXH * MYQ;                 // [nvy][NXT]

  // Column sliding DFT: seed with the direct DFT of the My rows above y0
  // (rows above the frame count as zero)
  float2 acol[CPL], wy[CPL];
  auto seed = [&](int j, const float2 (&v)[MY]) {
    acol[j] = make_float2(0.f, 0.f);
    int e = 0;                                   // (ky m) mod My
#pragma unroll
    for (int m = 0; m < MY; ++m) {
      acol[j] = cadd(acol[j], cmul(ld2(&s_twy[e]), v[m]));
      e += ky[j];
      e = (e >= MY) ? e - MY : e;
    }
    wy[j] = ld2(&s_twy[ky[j]]);
  };
  if (!OWN_ROWS) {
    // all My loads are issued before the sum, so a tile start costs one memory
    // latency, not My of them
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      float2 v[MY];
#pragma unroll
      for (int m = 0; m < MY; ++m) {
        const int yy = y0 - 1 - m;
        v[m] = (yy >= 0) ? at(a.rs + ((size_t)yy * a.W + xw) * NP, ro[j]) : make_float2(0.f, 0.f);
      }
      seed(j, v);
    }
  }

  // the same in every lane: held in scalar registers
  auto uni = [](float2 v) {
    return make_float2(__int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.x))),
                       __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v.y))));
  };
  float2 twz[MZ], twA[MZ];
#pragma unroll
  for (int k = 0; k < MZ; ++k) {
    twz[k] = uni(a.twz[k]);
    twA[k] = uni(a.twA[k]);
  }

  // first row's state (and row spectra); later rows' are loaded one row ahead
  float2 Xn[NL][VL], in_n[CPL], in_o[CPL];
  // (a row past the tile: an empty descriptor, and row spectra that are not used)
  auto load_row = [&](int yy) {
    const int y = CPL > 1 ? min(yy, y1 - 1) : yy;
    const auto src = buffer_of(a.st + ((size_t)y * a.W + xw) * (NCOL * MZ), CPL == 1 || yy < y1 ? st_bytes : 0u);
    const float2* rn = a.rs + ((size_t)y * a.W + xw) * NP;
    const float2* rl = a.rs + ((size_t)max(y - MY, 0) * a.W + xw) * NP;
#pragma unroll
    for (int i = 0; i < NL; ++i) buffer_ld(src, po + 8u * VL * LPP * i, Xn[i]);
    if (!OWN_ROWS) {
#pragma unroll
      for (int j = 0; j < CPL; ++j) {
        in_n[j] = at(rn, ro[j]);
        in_o[j] = at(rl, ro[j]);
      }
    }
  };
  if (active) load_row(y0);

  // Stages B (item kx * nvy + iy) and C (item iy * nvx + ix).  B: LB lanes per kx share
  // its Q row over the l_y they take (g, g + LB, ...).  C, one column per lane: items cl,
  // cl + LPP, ..., whose operands' places are read from a table (the indices carried
  // along took 15 of a candidate's 40 instructions; a lane that keeps one l_x and
  // its weights is slower, 500 against 481 us for 9x9x5 640x512: its rows wait for each
  // other).  C, two columns per lane (MX = 16): the LDS return path bounds a stage that
  // reads two rows per item, so a T row serves KX = 3 candidates of one l_y, LC =
  // ceil(nvx / 3) apart, G l_y at a time (319x241, 33x33 candidates: 733 against 890 us
  // a frame; the small windows are 8 to 10% faster in the flat order).
  constexpr bool ROWS = CPL > 1;
  constexpr int LB = LPP / NXH, KX = 3;
  const int kxB = cl / LB, iyB = cl - kxB * LB;
  const int LC = (nvx + KX - 1) / KX, G = LPP / LC;
  const int iyC0 = cl / LC, ixC0 = cl - iyC0 * LC;
  const int o_q = kxB * MYQ, o_ty = iyB * MYT, o_t = iyB * NXT + kxB;
  const float inv_nvx = 1.0f / (float)nvx;

  for (int yc = y0; yc < y1; yc += SH::SR) {      // OWN_ROWS: SR rows of row spectra at a time
   const int ye = OWN_ROWS ? min(y1, yc + SH::SR) : y1;
   if (OWN_ROWS) {
    if (yc > y0) __syncthreads();                // every wavefront is done with the previous rows
    tile_rows<MX, MY, MZ>(a, xb * SH::PPB, yc - MY, yc, ye - yc + MY, (lds_float*)s_w0, s_twx, s_rs);
    if (!active) continue;
    if (yc == y0) {
#pragma unroll
     for (int j = 0; j < CPL; ++j) {
      float2 v[MY];
#pragma unroll
      for (int m = 0; m < MY; ++m)
        v[m] = (y0 - 1 - m >= 0) ? ld2(rs_own[j] + (MY - 1 - m) * RSR) : make_float2(0.f, 0.f);
      seed(j, v);
     }
    }
   }
   for (int y = yc; y < ye; ++y) {
    const size_t pix0 = (size_t)y * a.W + xw;     // the same in all lanes
    const int r0 = (y - yc) * RSR;
    // opaque per row: what stage C derives from the lane's place is computed again each
    // row instead of being held in registers (or spilled) across the loop
    int iyC = iyC0, ixC = ixC0;
    if (ROWS) asm volatile("" : "+v"(iyC), "+v"(ixC));
    float2 X[CPL][MZ];
    float* rp = a.rsm + pix0 * nv;
    float rn[NB];
    // smoothed R, through a buffer descriptor of the anchors' values (reads past it
    // give 0, writes are dropped): every access is unconditional, so that a wait
    // counts the accesses it can leave in flight.  A lane's first candidate, or (ROWS)
    // first candidate u of KX:
    const auto rb = buffer_of(rp, 4u * (unsigned)(nv * (PPW == 1 ? 1 : min(PPW, a.W - xw))));
    const unsigned r_step = 4u * (unsigned)(ROWS ? G * nvx : LPP);   // from one round's values to the next's
    auto r_off = [&](int u) {
      if (!ROWS) return qo + 4u * (unsigned)cl;
      return iyC < G && ixC + u * LC < nvx ? qo + 4u * (unsigned)(iyC * nvx + ixC + u * LC) : BUFFER_NONE;
    };
    auto load_r = [&]() {                        // the first NB candidates'
#pragma unroll
      for (int i = 0; i < NB; ++i)
        rn[i] = ROWS ? buffer_ld(rb, r_off(i % KX) + (unsigned)(i / KX) * r_step) : buffer_ld(rb, r_off(0) + 4u * LPP * i);
    };
    wave_lds_sync();                             // the previous row's stage C reads are done
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if constexpr (VL == 2) st4(s_w + pl + i * PLS, Xn[i][0].x, Xn[i][0].y, Xn[i][1].x, Xn[i][1].y);
      else st2(s_w + pl + i * PLS, Xn[i][0]);
    }
    wave_lds_sync();
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      // ---- column sliding DFT: comb on the row spectra, resonator w_y^ky
      float2 in = OWN_ROWS ? ld2(rs_own[j] + r0 + MY * RSR) : in_n[j];
      if (y >= MY) in = csub(in, OWN_ROWS ? ld2(rs_own[j] + r0) : in_o[j]);
      acol[j] = cadd(cmul(wy[j], acol[j]), in);
      const float2 s2 = cscale(acol[j], a.inv_sqrt_my);
      // ---- temporal deadbeat observer: prior = rotate(posterior), innovation
      // e = input - sum(prior), posterior = prior + e / Mz
      float2 sum = make_float2(0.f, 0.f);
      float2 post[MZ];
      if constexpr (MZ % 2 == 0) {
        ld_col<MZ>(s_w + col[j] * CS, post);
      } else {
#pragma unroll
        for (int k = 0; k < MZ; ++k) post[k] = ld2(s_w + col[j] * CS + k);
      }
#pragma unroll
      for (int k = 0; k < MZ; ++k) {
        X[j][k] = cmul(twz[k], post[k]);
        sum = cadd(sum, X[j][k]);
      }
      const float2 e = cscale(csub(s2, sum), 1.0f / MZ);
#pragma unroll
      for (int k = 0; k < MZ; ++k) X[j][k] = cadd(X[j][k], e);
      if constexpr (MZ % 2 == 0) {
        st_col<MZ>(s_w + col[j] * CS, X[j]);
      } else {
#pragma unroll
        for (int k = 0; k < MZ; ++k) st2(s_w + col[j] * CS + k, X[j][k]);
      }
    }
    wave_lds_sync();
    {
      const auto dst = buffer_of(a.st + pix0 * (NCOL * MZ), st_bytes);
      float2 v[NL][VL];
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        if constexpr (VL == 2) {
          const float4 q = ld4(s_w + pl + i * PLS);
          v[i][0] = make_float2(q.x, q.y);
          v[i][1] = make_float2(q.z, q.w);
        } else {
          v[i][0] = ld2(s_w + pl + i * PLS);
        }
      }
#pragma unroll
      for (int i = 0; i < NL; ++i) buffer_st(dst, v[i], po + 8u * VL * LPP * i);
    }
    // this row's smoothed R (first rounds of stage C), the delayed sample and
    // the next row's state are in flight during the flow stages; stage C waits
    // for the first group only (vector memory completes in order)
    load_r();
    float idel = 0.f;
    {
      const int xs = x - a.dx, ys = y - a.dy;
      const bool ok = ring_delayed != nullptr && xs >= 0 && ys >= 0;
      if (CPL > 1) {
        const float v = *(ok ? ring_delayed + (size_t)ys * a.W + xs : a.gx);
        idel = ok ? v : 0.f;
      } else if (ok) {
        idel = ring_delayed[(size_t)ys * a.W + xs];
      }
    }
    // (unconditional where the wait for R that follows can then leave the next row's
    // state in flight: 33x33 candidates 534 -> 521 us; the small windows lose 1% by
    // the empty accesses of a tile's last row)
    if (CPL > 1 || y + 1 < y1) load_row(y + 1);

    // ---- high-pass (drop kx = ky = 0 for every kz) and Hann along kz.
    // Hann along an axis is Y(k) = (2X(k) - X(k-1) - X(k+1)) / 4; the 1/4 per
    // axis is folded into the stage-A weights.
    float2 Hy[CPL][MZ];
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      float2 V[MZ];
#pragma unroll
      for (int k = 0; k < MZ; ++k) V[k] = X[j][k];
      if (!EVEN) {
#pragma unroll
        for (int k = 0; k < MZ; ++k) V[k] = make_float2(col[j] == 0 ? 0.f : X[j][k].x, col[j] == 0 ? 0.f : X[j][k].y);
      } else if (col[j] == 0) {
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
          // the packed plane holds S(0) + j S(Mx/2); remove the S(0) part only:
          // S(0)(0, kz) = (C(kz) + conj C(-kz)) / 2
          const float2 cm = X[j][(MZ - k) % MZ];
          V[k] = make_float2(0.5f * (X[j][k].x - cm.x), 0.5f * (X[j][k].y + cm.y));
        }
      }
#pragma unroll
      for (int k = 0; k < MZ; ++k) {
        const float2 l = V[(k + MZ - 1) % MZ], r = V[(k + 1) % MZ];
        Hy[j][k] = make_float2(2.f * V[k].x - l.x - r.x, 2.f * V[k].y - l.y - r.y);
      }
    }
    // ---- Hann along ky: a plane of 16 ky is a row of 16 lanes (DPP); other
    // windows exchange through the staging rows
    if (MY == 16) {
#pragma unroll
      for (int j = 0; j < CPL; ++j)
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
          const float2 v = Hy[j][k];
          const float2 l = make_float2(dppf<ROR1>(v.x), dppf<ROR1>(v.y));
          const float2 r = make_float2(dppf<ROR15>(v.x), dppf<ROR15>(v.y));
          Hy[j][k] = make_float2(2.f * v.x - l.x - r.x, 2.f * v.y - l.y - r.y);
        }
      wave_lds_sync();                           // the state's pieces are read
    } else {
      wave_lds_sync();
      st_col<MZ>(s_w + sidx(p[0], ky[0]), Hy[0]);
      wave_lds_sync();
      float2 l[MZ], r[MZ];
      ld_col<MZ>(s_w + sidx(p[0], ky[0] == 0 ? MY - 1 : ky[0] - 1), l);
      ld_col<MZ>(s_w + sidx(p[0], ky[0] == MY - 1 ? 0 : ky[0] + 1), r);
#pragma unroll
      for (int k = 0; k < MZ; ++k) {
        const float2 v = Hy[0][k];
        Hy[0][k] = make_float2(2.f * v.x - l[k].x - r[k].x, 2.f * v.y - l[k].y - r[k].y);
      }
      wave_lds_sync();                           // every lane has read its neighbours
    }
    // ---- stage the y,z-windowed planes; even Mx: unpack plane 0 with its
    // (-ky, -kz) mirror, S(0) = (C + conj C(-k)) / 2, S(Mx/2) = (C - conj C(-k)) / 2j
#pragma unroll
    for (int j = 0; j < CPL; ++j) st_col<MZ>(s_w + sidx(p[j], ky[j]), Hy[j]);
    if (EVEN) {
      wave_lds_sync();
      if (cl < MY) {
        float2 w[MZ], s0[MZ], sh[MZ];
        ld_col<MZ>(s_w + sidx(0, ky[0] == 0 ? 0 : MY - ky[0]), w);
#pragma unroll
        for (int k = 0; k < MZ; ++k) {
          const float2 u = Hy[0][k], m = w[(MZ - k) % MZ];
          s0[k] = make_float2(0.5f * (u.x + m.x), 0.5f * (u.y - m.y));
          sh[k] = make_float2(0.5f * (u.y + m.y), -0.5f * (u.x - m.x));
        }
        wave_lds_sync();                         // every read of plane 0 precedes every write to it
        st_col<MZ>(s_w + sidx(0, ky[0]), s0);
        st_col<MZ>(s_w + sidx(MX / 2, ky[0]), sh);
      }
    }
    // planes -1 and NXH are the conjugate mirrors of planes 1 and MX - NXH:
    // S(-kx, ky, kz) = conj S(kx, -ky, -kz)
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      const bool lo = (p[j] == 1), hi = (p[j] == MX - NXH);
      if (lo | hi) {
        float2 m[MZ];
#pragma unroll
        for (int k = 0; k < MZ; ++k) m[k] = cconj(Hy[j][(MZ - k) % MZ]);
        st_col<MZ>(s_w + sidx(lo ? -1 : NXH, ky[j] == 0 ? 0 : MY - ky[j]), m);
      }
    }
    wave_lds_sync();

    // ---- Hann along kx, power spectrum (eq. 9), stage A of eq. (10):
    // Q(kx, ky) = sum_kz P(k) w_z^kz (l_z = 1), kx in [0, Mx/2]
    auto stage_a = [&](int kx, int kyy) -> float2 {
      float2 v[MZ], l[MZ], r[MZ];
      ld_col<MZ>(s_w + sidx(kx, kyy), v);
      ld_col<MZ>(s_w + sidx(kx - 1, kyy), l);
      ld_col<MZ>(s_w + sidx(kx + 1, kyy), r);
      float2 q = make_float2(0.f, 0.f);
#pragma unroll
      for (int k = 0; k < MZ; ++k) {
        const float hx = 2.f * v[k].x - l[k].x - r[k].x, hy = 2.f * v[k].y - l[k].y - r[k].y;
        const float P = hx * hx + hy * hy;
        q.x += P * twA[k].x;
        q.y += P * twA[k].y;
      }
      return q;
    };
    float2 Q[CPL], Qh = make_float2(0.f, 0.f);
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      Q[j] = stage_a(p[j], ky[j]);
      // one pass's LDS reads in flight at a time: with both in flight the 16x16x8
      // tile spilled (33x33 candidates at 319x241: 631 against 676 us a frame)
      if (CPL > 1) pass_done(Q[j]);
    }
    if (EVEN) {
      if (cl < MY) Qh = stage_a(MX / 2, ky[0]);
    }
    wave_lds_sync();                             // the staged planes are read (Q and T alias them)
#pragma unroll
    for (int j = 0; j < CPL; ++j) st2(&s_q[p[j] * MYQ + ky[j]], Q[j]);
    if (EVEN) {
      if (cl < MY) st2(&s_q[(MX / 2) * MYQ + ky[0]], Qh);
    }
    wave_lds_sync();

    // ---- stage B: T(kx, iy) = sum_ky Q(kx, ky) tau_y(ky, l_y[iy])
    {
      float2 q[MY], ty[MY];
      auto item = [&](const lds_v2* p_ty, lds_v2* p_t) {
        ld_col<MY>(p_ty, ty);
        float2 t = make_float2(0.f, 0.f);
#pragma unroll
        for (int k = 0; k < MY; ++k) t = cadd(t, cmul(q[k], ty[k]));
        st2(p_t, t);
      };
      // (LDS addresses move by additions: a 32-bit multiplication takes four
      // issue slots)
      const lds_v2 *p_q = s_q + o_q, *p_ty = s_tauy + o_ty;
      lds_v2* p_t = s_t + o_t;
      if (kxB < NXH) {
        ld_col<MY>(p_q, q);
        for (int iy = iyB; iy < nvy; iy += LB, p_ty += LB * MYT, p_t += LB * NXT) item(p_ty, p_t);
      }
    }
    wave_lds_sync();

    // ---- stage C: R(ix, iy) = sum_kx w(kx) Re[T(kx, iy) tau_x(kx, l_x[ix])],
    // first-order smoothing, running argmax
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    {
      float2 t[NXH], tx[ROWS ? KX : 1][NXH];
      auto smooth = [&](const float2 (&w_x)[NXH], float r_prev) {
        float r = 0.f;
#pragma unroll
        for (int kx = 0; kx < NXH; ++kx) r += t[kx].x * w_x[kx].x - t[kx].y * w_x[kx].y;
        return (1.f - a.alpha) * r + a.alpha * r_prev;
      };
      // A lane's candidates come in rising order, so only a larger value takes
      // over, and the round it came in is all that is kept (a grid without a value
      // above -infinity: below).
      int br = -1;
      auto keep = [&](float sm, int rnd, bool ok, unsigned off) {
        buffer_st(rb, sm, PPW == 1 || ok ? off : BUFFER_NONE);
        const bool take = (sm > bv) & ok;
        bv = take ? sm : bv;
        br = take ? rnd : br;
      };
      if constexpr (ROWS) {
        unsigned vo[KX];
#pragma unroll
        for (int u = 0; u < KX; ++u) {
          vo[u] = r_off(u);
          ld_col<NXH>(s_taux + min(ixC + u * LC, nvx - 1) * NXT, tx[u]);
        }
        int o_t = min(iyC, nvy - 1) * NXT, rnd = 0;
        // (leaving inside the group, not skipping a round of it: on the way back every
        // access has been issued)
        for (int iy0 = 0; iy0 < nvy;) {
#pragma unroll
          for (int v = 0; v < NB / KX; ++v, iy0 += G) {
            if (v > 0 && iy0 >= nvy) break;
            ld_col<NXH>(s_t + o_t, t);
            o_t = min(o_t + G * NXT, (nvy - 1) * NXT);
#pragma unroll
            for (int u = 0; u < KX; ++u, ++rnd) {
              keep(smooth(tx[u], rn[v * KX + u]), rnd, vo[u] < 4u * (unsigned)nv, vo[u]);
              rn[v * KX + u] = buffer_ld(rb, vo[u] + NB / KX * r_step);
              vo[u] += r_step;
            }
            __builtin_amdgcn_sched_barrier(0);   // one round's LDS reads in flight at a time
          }
        }
        const int rr = br / KX;
        bi = br < 0 ? 0x7fffffff : (rr * G + iyC) * nvx + ixC + (br - rr * KX) * LC;
      } else {
        unsigned vo = r_off(0);
        const lds_u32* it = s_itC + cl;
        unsigned itC = it[0];
        auto round = [&](int i, int rnd, bool ok, bool whole) {   // (whole groups have no lane past the grid)
          const unsigned o = itC;
          itC = it[(i + 1) * LPP];
          ld_col<NXH>(lds_at(s_t, o & 0xffffu), t);
          ld_col<NXH>(lds_at(s_taux, o >> 16), tx[0]);
          keep(smooth(tx[0], rn[i]), rnd, whole | ok, vo + 4u * LPP * i);
          __builtin_amdgcn_sched_barrier(0);
        };
        int w0 = 0, rnd = 0;
        for (; w0 + NB * LPP < nv; w0 += NB * LPP, rnd += NB) {
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            round(i, rnd + i, true, true);
            rn[i] = buffer_ld(rb, vo + 4u * LPP * (NB + i));
          }
          vo += 4u * LPP * NB;
          it += LPP * NB;
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
          if (w0 + i * LPP < nv) round(i, rnd + i, cl < nv - w0 - i * LPP, false);   // uniform
        bi = br < 0 ? 0x7fffffff : br * LPP + cl;
      }
    }
    group_amax<LPP>(bv, bi);
    if (__any(bv == -INFINITY)) {       // overflowed: the first candidate of -infinity, if one is
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      int first = 0x7fffffff;
      for (int w = cl; w < nv; w += LPP)
        if (at(rp, qo + 4u * (unsigned)w) == -INFINITY) first = min(first, w);
      first = group_ext<LPP, false>(first);
      if (bv == -INFINITY) bi = first;
    }
    const int istar = (bi < nv) ? bi : 0;   // no finite candidate: fall back to index 0

    // ---- velocity mode 3: refine the peak between grid points, from the
    // smoothed R this row has just stored (the fence makes the wavefront's
    // stores visible to all of its lanes)
    float2 vref = make_float2(0.f, 0.f);
    if (REFINED) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
      vref = refine_peak(a.gx, a.gy, nvx, nvy, istar, at(rp, qo + 4u * (unsigned)istar),
                         [&](int w) { return at(rp, qo + 4u * (unsigned)w); });
    }

    // ---- background estimate (eq. 4) with the coefficients of the chosen
    // velocity (eq. 8 at the bins; Hermitian weights folded into the table, or
    // evaluated here for the refined velocity)
    const int hsel = (a.vmode == 2) ? nv : istar;
    float tot = 0.f;
#pragma unroll
    for (int j = 0; j < CPL; ++j) {
      float acc = 0.f;
      const int kyc = (2 * ky[j] <= MY) ? ky[j] : ky[j] - MY;
      if ((CPL > 1 || cl < NCOL) && p[j] <= a.bx && kyc >= -a.by && kyc <= a.by) {
        if (REFINED) {
          const float wgt = (p[j] == 0) ? 1.f : 2.f;
#pragma unroll
          for (int kz = 0; kz < MZ; ++kz) {
            const float2 h = coeff_at<MX, MY, MZ>(p[j], kyc, kz, vref.x, vref.y, a.dx, a.dy, a.dt);
            acc += wgt * (h.x * X[j][kz].x - h.y * X[j][kz].y);
          }
        } else {
          // (at most (33^2 + 1) 8 17 8 entries)
          const unsigned h0 = __umul24(__umul24(hsel, a.bx + 1) + p[j], 2 * a.by + 1) * (8u * MZ) + (kyc + a.by) * (8u * MZ);
#pragma unroll
          for (int kz = 0; kz < MZ; ++kz) {
            const float2 h = (&at(a.htab, h0))[kz];
            acc += h.x * X[j][kz].x - h.y * X[j][kz].y;
          }
        }
      }
      tot += group_sum<LPP>(acc);
    }
    if (px_ok && cl == 0) {
      if (!isfinite(idel)) idel = 0.f;
      const size_t pix = pix0 + ps;
      a.out[pix] = idel - tot;
      if (a.vmode == 2) {
        a.vxy[pix] = make_float2(a.fvx, a.fvy);
        a.vidx[pix] = -1;
      } else {
        const int iy = (int)(((float)istar + 0.5f) * inv_nvx);   // istar / nvx (below 2^11, so exact)
        a.vxy[pix] = REFINED ? vref : make_float2(s_gx[istar - iy * nvx], s_gx[nvx + iy]);
        a.vidx[pix] = istar;
      }
    }
   }
   if (!OWN_ROWS) break;
  }
}

}  // namespace rmdf
