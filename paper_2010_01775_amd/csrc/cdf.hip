// pdf and marginal/conditional CDF tables of each leaf's density.
//
// One workgroup per leaf.  Every sum and prefix is formed in binary64 and only
// the stored tables are rounded to float32:
//   S = sum s;  p = s / S;  pdf = p*H*W/(4 pi)
//   row mass m_i = sum_j p_ij, marginal M_i = sum_{i'<i} m_i' (M_H = 1)
//   conditional C_ij = sum_{j'<j} p_ij' / m_i (C_iW = 1; j/W if m_i = 0)
// The quotients are taken as products with binary64 reciprocals of S and
// m_i (one more binary64 rounding, far below the float32 rounding of the
// stored values).  Maps that fit a workgroup's registers (up to 32,768 bins,
// rows of up to 256) take cdf_reg_kernel; larger ones cdf_kernel, where a row
// is scanned by one wavefront in slices of 64 consecutive bins (coalesced
// loads and stores): a wavefront scan per slice plus the running total of the
// slices before it.
#include <math.h>

#include <algorithm>

#include "npg_internal.h"

namespace {

constexpr int CDF_THREADS = 256;
constexpr double FOUR_PI = 4.0 * M_PI;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// exclusive prefix over the 64 lanes
__device__ __forceinline__ double wave_excl_scan(double v, int lane) {
  double incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  return incl - v;
}

// Output tables of leaf l: contiguous batch arrays, or per-leaf pointers.
struct BatchOut {
  float *pdf, *marg, *cond;
  double *total;
  __device__ void get(int l, int H, int W, float **p, float **m, float **c, double **t) const {
    *p = pdf + (size_t)l * H * W;
    *m = marg + (size_t)l * (H + 1);
    *c = cond + (size_t)l * H * (W + 1);
    *t = total ? total + l : nullptr;
  }
};
struct DescOut {
  const npg_leaf_desc *d;
  __device__ void get(int l, int, int, float **p, float **m, float **c, double **t) const {
    *p = d[l].pdf;
    *m = d[l].marg;
    *c = d[l].cond;
    *t = d[l].total;
  }
};

template <class OUT, int SEG>
__global__ __launch_bounds__(CDF_THREADS) void cdf_kernel(const float *__restrict__ dens, int H, int W, OUT out,
                                                          uint32_t *err) {
  extern __shared__ double rowmass[];  // [H]
  __shared__ double red[4];
  __shared__ int bad_s;
  const int leaf = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t HW = (size_t)H * W;
  const float *s = dens + leaf * HW;
  if (tid == 0) bad_s = 0;
  __syncthreads();
  // total S
  double acc = 0.0;
  int bad = 0;
  for (size_t k = tid; k < HW; k += CDF_THREADS) {
    const float v = s[k];
    if (!(v >= 0.0f) || !isfinite(v)) bad = 1;
    acc += (double)v;
  }
  acc = wave_sum(acc);
  if (lane == 0) red[wave] = acc;
  if (bad) atomicOr(&bad_s, 1);
  __syncthreads();
  const double S = red[0] + red[1] + red[2] + red[3];
  float *pl, *ml, *cl;
  double *tl;
  out.get(leaf, H, W, &pl, &ml, &cl, &tl);
  if (bad_s || !(S > 0.0) || !isfinite(S)) {
    const float qnan = __int_as_float(0x7fc00000);
    for (size_t k = tid; k < HW; k += CDF_THREADS) pl[k] = qnan;
    for (int k = tid; k <= H; k += CDF_THREADS) ml[k] = qnan;
    for (size_t k = tid; k < (size_t)H * (W + 1); k += CDF_THREADS) cl[k] = qnan;
    if (tid == 0) {
      if (tl) *tl = 0.0;
      raise_err(err, ERR_RANGE);
    }
    return;
  }
  const double invS = 1.0 / S;
  const double pdf_k = (double)HW / FOUR_PI;
  // rows: one wavefront per row, bins j = 64 t + lane of slice t
  for (int i = wave; i < H; i += 4) {
    const float *srow = s + (size_t)i * W;
    float *prow = pl + (size_t)i * W;
    double c[SEG];  // exclusive prefix of p over the row at this lane's bins
    double run = 0.0;
#pragma unroll
    for (int t = 0; t < SEG; ++t) {
      const int j = 64 * t + lane;
      const double p = j < W ? (double)srow[j] * invS : 0.0;
      if (j < W) prow[j] = (float)(p * pdf_k);
      double incl = p;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const double u = __shfl_up(incl, o);
        if (lane >= o) incl += u;
      }
      // the previous lane's inclusive sum: non-decreasing along the row
      double ex = __shfl_up(incl, 1);
      if (lane == 0) ex = 0.0;
      c[t] = run + ex;
      run += __shfl(incl, 63);
    }
    const double m = run;
    float *crow = cl + (size_t)i * (W + 1);
    if (m > 0.0) {
      const double invm = 1.0 / m;
#pragma unroll
      for (int t = 0; t < SEG; ++t) {
        const int j = 64 * t + lane;
        if (j < W) crow[j] = (float)(c[t] * invm);
      }
    } else {
#pragma unroll
      for (int t = 0; t < SEG; ++t) {
        const int j = 64 * t + lane;
        if (j < W) crow[j] = (float)((double)j / (double)W);
      }
    }
    if (lane == 0) {
      crow[W] = 1.0f;
      rowmass[i] = m;
    }
  }
  __syncthreads();
  // marginal over rows (wavefront 0)
  if (wave == 0) {
    const int rseg = (H + 63) / 64;
    const int i0 = lane * rseg;
    double part = 0.0;
    for (int t = 0; t < rseg; ++t)
      if (i0 + t < H) part += rowmass[i0 + t];
    double c = wave_excl_scan(part, lane);
    for (int t = 0; t < rseg; ++t) {
      const int i = i0 + t;
      if (i < H) {
        ml[i] = (float)c;
        c += rowmass[i];
      }
    }
    if (lane == 0) {
      ml[H] = 1.0f;
      if (tl) *tl = S;
    }
  }
}

// Lane shifts on the DPP path (one move per half instead of an LDS permute);
// lanes without a source read +0.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int2 h = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, h.x, CTRL, 0xf, 0xf, true),
                                              __builtin_amdgcn_update_dpp(0, h.y, CTRL, 0xf, 0xf, true)));
}
constexpr int DPP_ROW_SHR = 0x110, DPP_WAVE_SHR1 = 0x138, DPP_BCAST15 = 0x142, DPP_BCAST31 = 0x143;

// inclusive prefix over aligned groups of G lanes (a power of two)
__device__ __forceinline__ double group_incl_scan(double v, int lane, int G) {
  const int pos = lane & (G - 1);
  double u;
  if (G > 1) u = dpp_f64<DPP_ROW_SHR + 1>(v), v += pos >= 1 ? u : 0.0;
  if (G > 2) u = dpp_f64<DPP_ROW_SHR + 2>(v), v += pos >= 2 ? u : 0.0;
  if (G > 4) u = dpp_f64<DPP_ROW_SHR + 4>(v), v += pos >= 4 ? u : 0.0;
  if (G > 8) u = dpp_f64<DPP_ROW_SHR + 8>(v), v += pos >= 8 ? u : 0.0;
  if (G > 16) u = dpp_f64<DPP_BCAST15>(v), v += (lane & 16) ? u : 0.0;
  if (G > 32) u = dpp_f64<DPP_BCAST31>(v), v += (lane & 32) ? u : 0.0;
  return v;
}

// four floats at any 4-byte aligned address (rows of cond are W + 1 long)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// The tables of a map held in registers: NV float4 pieces per thread, a row
// of W bins in W / 4 consecutive lanes.  Bound by HBM: the density is read
// once, in 16-byte pieces that are all in flight together, and the tables are
// written in 16-byte pieces; the scans run per row on lane shifts.  (cdf_kernel
// reads the density twice and moves 4 bytes at a time: 4001 leaves of 128x128,
// 787 MB, took 307 us there and 153 us here.)  A row's prefixes and its mass
// are sums of the densities themselves, scaled once by the reciprocal of the
// row's sum.
template <class OUT, int NV>
__global__ __launch_bounds__(1024, NV <= 4 ? 8 : 4) void cdf_reg_kernel(const float *__restrict__ dens, int H, int W, OUT out,
                                                       uint32_t *err) {
  extern __shared__ double rowsum[];  // [H]
  const int leaf = blockIdx.x, tid = threadIdx.x, lane = tid & 63, NT = blockDim.x;
  const int n4 = H * W / 4, G = W >> 2, lg = __builtin_ctz((unsigned)G);
  const float *s = dens + (size_t)leaf * H * W;
  f32x4u v[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int f = k * NT + tid;
    v[k] = f < n4 ? *reinterpret_cast<const f32x4u *>(s + 4 * (size_t)f) : f32x4u{0.0f, 0.0f, 0.0f, 0.0f};
  }
  int bad = 0;
  double ex[NV];  // prefix of the row before this piece
#pragma unroll
  for (int k = 0; k < NV; ++k) {
#pragma unroll
    for (int c = 0; c < 4; ++c) bad |= !(v[k][c] >= 0.0f) || !isfinite(v[k][c]);
    const double t = ((double)v[k][0] + (double)v[k][1]) + ((double)v[k][2] + (double)v[k][3]);
    const double incl = group_incl_scan(t, lane, G);
    const double prev = dpp_f64<DPP_WAVE_SHR1>(incl);
    ex[k] = (lane & (G - 1)) ? prev : 0.0;
    const int f = k * NT + tid;
    if ((lane & (G - 1)) == G - 1 && f < n4) rowsum[f >> lg] = incl;
  }
  bad = __syncthreads_or(bad);
  // S, the same in every wavefront
  double S = 0.0;
  for (int i = lane; i < H; i += 64) S += rowsum[i];
  S = wave_sum(S);
  float *pl, *ml, *cl;
  double *tl;
  out.get(leaf, H, W, &pl, &ml, &cl, &tl);
  if (bad || !(S > 0.0) || !isfinite(S)) {
    const float qnan = __int_as_float(0x7fc00000);
    for (int k = tid; k < H * W; k += NT) pl[k] = qnan;
    for (int k = tid; k <= H; k += NT) ml[k] = qnan;
    for (int k = tid; k < H * (W + 1); k += NT) cl[k] = qnan;
    if (tid == 0) {
      if (tl) *tl = 0.0;
      raise_err(err, ERR_RANGE);
    }
    return;
  }
  const double invS = 1.0 / S;
  const double pdf_k = (double)H * (double)W / FOUR_PI;
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int f = k * NT + tid;
    if (f >= n4) break;
    f32x4u o;
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] = (float)((double)v[k][c] * invS * pdf_k);
    *reinterpret_cast<f32x4u *>(pl + 4 * (size_t)f) = o;
    const int row = f >> lg, g = f & (G - 1);
    const double m = rowsum[row];
    if (m > 0.0) {
      const double invm = 1.0 / m;
      // no entry exceeds the row's sum, whatever the order it was added in
      const double c1 = ex[k] + (double)v[k][0], c2 = c1 + (double)v[k][1], c3 = c2 + (double)v[k][2];
      o = f32x4u{(float)(fmin(ex[k], m) * invm), (float)(fmin(c1, m) * invm), (float)(fmin(c2, m) * invm),
                 (float)(fmin(c3, m) * invm)};
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) o[c] = (float)((double)(4 * g + c) / (double)W);
    }
    float *cr = cl + (size_t)row * (W + 1) + 4 * g;
    *reinterpret_cast<f32x4u *>(cr) = o;
    if (g == G - 1) cr[4] = 1.0f;
  }
  // marginal over rows (the last wavefront)
  if (tid >= NT - 64) {
    const int rseg = (H + 63) / 64, i0 = lane * rseg;
    double part = 0.0;
    for (int t = 0; t < rseg; ++t)
      if (i0 + t < H) part += rowsum[i0 + t];
    double c = wave_excl_scan(part, lane);
    for (int t = 0; t < rseg; ++t) {
      const int i = i0 + t;
      if (i < H) {
        ml[i] = (float)(fmin(c, S) * invS);
        c += rowsum[i];
      }
    }
    if (lane == 0) {
      ml[H] = 1.0f;
      if (tl) *tl = S;
    }
  }
}

template <class OUT>
hipError_t launch_cdf_t(const float *density, uint32_t L, int H, int W, const OUT &o, uint32_t *err,
                        hipStream_t s) {
  const size_t lds = sizeof(double) * H;
  // A map that 1024 threads hold in eight 16-byte pieces each, with rows
  // inside a wavefront, is read once; one piece per thread up to 1024 bins
  // (more wavefronts for the same latency), four where that needs fewer than
  // 1024 threads.  Beyond, a thread's pieces and prefixes would not fit the
  // 128 registers of such a workgroup.
  const int n4 = H * W / 4;
  if (W <= 256 && n4 <= 8192) {
    const int nv = n4 <= 256 ? 1 : n4 <= 4096 ? 4 : 8, nt = std::max(64, n4 / nv);
    if (nv == 1)
      hipLaunchKernelGGL((cdf_reg_kernel<OUT, 1>), dim3(L), dim3(nt), lds, s, density, H, W, o, err);
    else if (nv == 4)
      hipLaunchKernelGGL((cdf_reg_kernel<OUT, 4>), dim3(L), dim3(nt), lds, s, density, H, W, o, err);
    else
      hipLaunchKernelGGL((cdf_reg_kernel<OUT, 8>), dim3(L), dim3(nt), lds, s, density, H, W, o, err);
    return hipGetLastError();
  }
  const int seg = (W + 63) / 64;  // W is a power of two in [4, 1024]
  switch (seg) {
    case 1: hipLaunchKernelGGL((cdf_kernel<OUT, 1>), dim3(L), dim3(CDF_THREADS), lds, s, density, H, W, o, err); break;
    case 2: hipLaunchKernelGGL((cdf_kernel<OUT, 2>), dim3(L), dim3(CDF_THREADS), lds, s, density, H, W, o, err); break;
    case 4: hipLaunchKernelGGL((cdf_kernel<OUT, 4>), dim3(L), dim3(CDF_THREADS), lds, s, density, H, W, o, err); break;
    case 8: hipLaunchKernelGGL((cdf_kernel<OUT, 8>), dim3(L), dim3(CDF_THREADS), lds, s, density, H, W, o, err); break;
    default: hipLaunchKernelGGL((cdf_kernel<OUT, 16>), dim3(L), dim3(CDF_THREADS), lds, s, density, H, W, o, err);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_build_cdf(const float *density, uint32_t L, int H, int W, float *pdf, float *marg,
                            float *cond, double *total, uint32_t *err, hipStream_t s) {
  return launch_cdf_t(density, L, H, W, BatchOut{pdf, marg, cond, total}, err, s);
}

hipError_t launch_build_cdf_desc(const float *density, const npg_leaf_desc *d, uint32_t L, int H, int W,
                                 uint32_t *err, hipStream_t s) {
  return launch_cdf_t(density, L, H, W, DescOut{d}, err, s);
}
