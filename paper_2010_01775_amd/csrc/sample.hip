// Guided direction sampling by table inversion, and pdf evaluation.
//
// One lane per query.  Row and column are found by searches over the
// monotone float32 tables with exact comparisons, so a query selects exactly
// the bin the definition names: the last entry <= u.
#include <math.h>

#include "npg_internal.h"

namespace {

// Orders this wavefront's LDS accesses before and after it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int X>
__device__ __forceinline__ int quad_xor(int v) {  // the value of lane ^ X, X = 1 or 2
  return __builtin_amdgcn_mov_dpp(v, X == 1 ? 0xB1 : 0x4E, 0xF, 0xF, true);
}

// A row of n + 1 entries holds 16 of them from the first 16-byte boundary on
// (at most three entries in) once n >= 18.
constexpr int WIN_MIN = 18;

// Eight table entries t[a .. a+m] (m = 7, or fewer on short rows) around
// entry g, loaded in one memory round trip.  Rows of at least 16 entries load
// a 16-byte aligned window as two 16-byte pieces (it starts 3 to 6 entries
// below g and is moved by 4 entries to stay inside the row); shorter rows
// load eight clamped single entries.  A load instruction whose 64 lanes hit
// 64 different lines costs the same at any width, so the wide loads quarter
// that cost.
__device__ __forceinline__ void load_window(const float *__restrict__ t, int n, int g, int *a_out, int *m_out,
                                            float (&w)[8]) {
  int a, m;
  if (n >= 15) {
    const uintptr_t t0 = reinterpret_cast<uintptr_t>(t);
    a = (int)(((intptr_t)((t0 + 4 * (uintptr_t)(g - 3)) & ~(uintptr_t)15) - (intptr_t)t0) / 4);
    a = a < 0 ? a + 4 : a;
    a = a < 0 ? a + 4 : a;
    a = a + 7 > n ? a - 4 : a;
    m = 7;
    const float4 *p = reinterpret_cast<const float4 *>(t + a);
    const float4 v0 = p[0], v1 = p[1];
    w[0] = v0.x, w[1] = v0.y, w[2] = v0.z, w[3] = v0.w, w[4] = v1.x, w[5] = v1.y, w[6] = v1.z, w[7] = v1.w;
  } else {
    a = g - 3;
    a = a > n - 7 ? n - 7 : a;
    a = a < 0 ? 0 : a;
    m = n - a < 7 ? n - a : 7;
#pragma unroll
    for (int k = 0; k < 8; ++k) w[k] = t[a + (k < m ? k : m)];
  }
  *a_out = a;
  *m_out = m;
}

// largest i in [0, n-1] with t[i] <= u, for t non-decreasing with t[0] = 0
// <= u < t[n] = 1 (as build_cdf writes every row); *tl = t[i], *th =
// t[i+1].  The first window is placed where a linear table would hold u,
// up to three more (while none brackets u) by linear interpolation inside
// the bracket [lo, hi] the previous ones left, with its end values; each
// window settles the search when it brackets u, else narrows the bracket,
// which bisection finishes.  (On the clustered workload's tables the first
// window brackets about a third of the searches and the second most of the
// rest, where galloping outwards from the first window took several
// dependent loads: 1e8 samples 10.4 -> 7.6 ms.)  The answer is that of
// plain bisection.  Each lane by itself: for rows shorter than WIN_MIN, and in
// calls that wide_search leaves to it.
__device__ __forceinline__ int last_le(const float *__restrict__ t, int n, float u, float *tl, float *th) {
  int lo = 0, hi = n;           // t[lo] <= u < t[hi]
  float tlo = 0.0f, thi = 1.0f;  // t[lo], t[hi]
  int g = (int)(u * (float)n);
  g = g < n - 1 ? g : n - 1;
#pragma unroll 1
  for (int attempt = 0; attempt < 4 && hi - lo > 1; ++attempt) {
    int a, m;
    float w[8];
    load_window(t, n, g, &a, &m, w);
    if (w[0] <= u && u < w[m]) {
      int c = 0;  // entries t[a+1 .. a+m-1] that are <= u
#pragma unroll
      for (int k = 1; k < 7; ++k) c += (k < m && w[k] <= u) ? 1 : 0;
      float lo_v = w[0], hi_v = w[1];
#pragma unroll
      for (int k = 1; k < 7; ++k)
        if (k == c) {
          lo_v = w[k];
          hi_v = w[k + 1];
        }
      *tl = lo_v;
      *th = hi_v;
      return a + c;
    }
    if (w[m] <= u) {  // the bracket lies right of the window
      if (a + m > lo) {
        lo = a + m;
        tlo = w[m];
      }
    } else if (a < hi) {  // left of it: u < t[a]
      hi = a;
      thi = w[0];
    }
    // next guess: linear inside the bracket
    const float f = thi > tlo ? (u - tlo) / (thi - tlo) : 0.0f;
    g = lo + (int)(f * (float)(hi - lo));
    g = g < lo ? lo : g;
    g = g > hi - 1 ? hi - 1 : g;
  }
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    const float v = t[mid];
    if (v <= u) {
      lo = mid;
      tlo = v;
    } else {
      hi = mid;
      thi = v;
    }
  }
  *tl = tlo;
  *th = thi;
  return lo;
}

// last_le for the 64 searches of a wavefront at once (every lane calls it;
// `act`: the lane has a search).  A window is the 64-byte sector that holds
// the guessed entry, moved by whole 16-byte pieces where it would leave the
// row; four lanes read it, 16 bytes each, so one load instruction covers 16
// searches.  The searches still open are packed into the first slots of `slot`
// (64 of them, this wavefront's own), so a round costs one instruction per 16
// open searches, not per search left in the slowest lane.
//
// What bounds it: random 64-byte sectors (about 2 for a row of the marginal
// and 2.6 for one of the conditional table at 128 entries, one for the pdf).
// A lane that reads its own window of 32 bytes as two pieces asks L2 for a
// sector twice when the other 63 lanes have pushed the line out of the
// 32 KiB L1 in between, and each instruction looks up 64 lines.  20 million
// samples of 4000 maps of 128x128: requests to L2 184 -> 126 million, 1754 ->
// 1377 us; 10 million MIS samples of 12000 maps of 64x64: 555 -> 493 us.
// Windows of 32 entries, more rounds before bisection and guesses nearer the
// middle of the bracket measured within 2 % of this, or slower.
__device__ __forceinline__ int wave_last_le(const float *__restrict__ t, int n, float u, bool act,
                                            uint4 *__restrict__ slot, float *tl, float *th) {
  if (n < WIN_MIN) return act ? last_le(t, n, u, tl, th) : 0;
  const int lane = (int)threadIdx.x & 63, piece = lane & 3, quad = lane >> 2;
  const int r4 = (int)(-(reinterpret_cast<intptr_t>(t) >> 2) & 3);    // 16-byte aligned entries: r4 + 4k
  const int r16 = (int)(-(reinterpret_cast<intptr_t>(t) >> 2) & 15);  // 64-byte aligned entries: r16 + 16k
  int lo = 0, hi = n;            // t[lo] <= u < t[hi]
  float tlo = 0.0f, thi = 1.0f;  // t[lo], t[hi]
  int g = (int)(u * (float)n);
  g = g < n - 1 ? g : n - 1;
  bool open = act;
#pragma unroll 1
  for (int attempt = 0; attempt < 4; ++attempt) {
    int a = g - ((g - r16) & 15);
    a = a < 0 ? r4 : a;
    a = a + 15 > n ? a - ((a + 18 - n) & ~3) : a;
    const bool ask = open && a + 15 > lo && a < hi;
    const uint64_t asks = __ballot(ask);
    if (!asks) break;
    const int cnt = __popcll(asks);
    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(asks >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)asks, 0u));
    if (ask) {
      const uint64_t at = reinterpret_cast<uint64_t>(t + a);
      slot[rank] = make_uint4((uint32_t)at, (uint32_t)(at >> 32), __float_as_uint(u), 0u);
    }
    wave_sync();
    float4 w[4];
    float uq[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (16 * k < cnt) {  // the last searches of a ragged round are read twice
        const int sl = 16 * k + quad;
        const uint4 q = slot[sl < cnt ? sl : cnt - 1];
        uq[k] = __uint_as_float(q.z);
        w[k] = reinterpret_cast<const float4 *>((uint64_t)q.y << 32 | q.x)[piece];
      }
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (16 * k < cnt) {
        const float4 v = w[k];
        const bool b0 = v.x <= uq[k], b1 = v.y <= uq[k], b2 = v.z <= uq[k], b3 = v.w <= uq[k];
        int c = (int)b0 + (int)b1 + (int)b2 + (int)b3;
        // the last entry <= u and the first one above it
        float l = b3 ? v.w : b2 ? v.z : b1 ? v.y : b0 ? v.x : -INFINITY;
        float h = !b0 ? v.x : !b1 ? v.y : !b2 ? v.z : !b3 ? v.w : INFINITY;
        c += quad_xor<1>(c);
        l = fmaxf(l, __int_as_float(quad_xor<1>(__float_as_int(l))));
        h = fminf(h, __int_as_float(quad_xor<1>(__float_as_int(h))));
        c += quad_xor<2>(c);
        l = fmaxf(l, __int_as_float(quad_xor<2>(__float_as_int(l))));
        h = fminf(h, __int_as_float(quad_xor<2>(__float_as_int(h))));
        const int sl = 16 * k + quad;
        if (piece == 0 && sl < cnt) slot[sl] = make_uint4((uint32_t)c, __float_as_uint(l), __float_as_uint(h), 0u);
      }
    wave_sync();
    if (ask) {
      const uint4 q = slot[rank];
      const int c = (int)q.x;
      if (c > 0 && a + c - 1 >= lo) {
        lo = a + c - 1;
        tlo = __uint_as_float(q.y);
      }
      if (c < 16 && a + c <= hi) {
        hi = a + c;
        thi = __uint_as_float(q.z);
      }
      // next guess: linear inside the bracket, outside this window
      const float f = fminf((u - tlo) * __builtin_amdgcn_rcpf(thi - tlo), 1.0f);
      g = lo + (int)(f * (float)(hi - lo));
      g = g < lo + 1 ? lo + 1 : g;
      g = g > hi - 1 ? hi - 1 : g;
      open = hi - lo > 1;
    }
    wave_sync();
  }
  if (act)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      const float v = t[mid];
      if (v <= u) {
        lo = mid;
        tlo = v;
      } else {
        hi = mid;
        thi = v;
      }
    }
  *tl = tlo;
  *th = thi;
  return lo < n ? lo : n - 1;
}

// The guided sample of leaf l from (u1, u2): direction, the table pdf of the
// sampled bin and the bin, for the lanes with `act` (their leaf and uniforms
// are valid); every lane of the wavefront calls it.
template <bool WIDE>
__device__ __forceinline__ void guided_sample(const float *__restrict__ pdf, const float *__restrict__ marg,
                                              const float *__restrict__ cond, uint32_t l, int H, int W,
                                              float u1, float u2, bool act, uint4 *slot, float *d, float *p,
                                              uint32_t *bin) {
  if (!act) l = 0;
  const float below1 = __int_as_float(0x3f7fffff);
  const float two_over_h = 2.0f / (float)H;
  const float dphi = 6.283185307179586f / (float)W;
  const float *M = marg + (size_t)l * (H + 1);
  float m0, m1, c0, c1;
  const int i = WIDE ? wave_last_le(M, H, u1, act, slot, &m0, &m1) : act ? last_le(M, H, u1, &m0, &m1) : 0;
  const float *C = cond + ((size_t)l * H + i) * (W + 1);
  const int j = WIDE ? wave_last_le(C, W, u2, act, slot, &c0, &c1) : act ? last_le(C, W, u2, &c0, &c1) : 0;
  if (!act) return;
  float t1 = (u1 - m0) / (m1 - m0);
  float t2 = (u2 - c0) / (c1 - c0);
  t1 = fminf(fmaxf(t1, 0.0f), below1);
  t2 = fminf(fmaxf(t2, 0.0f), below1);
  // -1 + 2i/H, 2i/H and 2(H-i)/H are exact; each of z, 1+z, 1-z takes
  // one rounding, so sin(theta) = sqrt((1-z)(1+z)) stays accurate at the
  // poles where 1 - z*z would cancel.
  const float z = fmaf(t1, two_over_h, fmaf((float)i, two_over_h, -1.0f));
  const float opz = fmaf(t1, two_over_h, (float)i * two_over_h);
  const float omz = fmaf(-t1, two_over_h, (float)(H - i) * two_over_h);
  const float phi = fmaf(t2, dphi, (float)j * dphi);
  float sp, cp;
  sincosf(phi, &sp, &cp);
  const float r = sqrtf(fmaxf(0.0f, omz * opz));
  d[0] = r * cp;
  d[1] = r * sp;
  d[2] = z;
  *p = pdf[(size_t)l * H * W + (size_t)i * W + j];
  *bin = (uint32_t)(i * W + j);
}

// One query per lane, 64 consecutive queries per wavefront and iteration.
// The wavefront's directions (768 bytes, contiguous in dir) are staged in its
// own part of LDS and written as 16-byte pieces; pdf and bin are written one
// lane each (coalesced 4-byte pieces).  No workgroup barrier: the searches of
// the four wavefronts take different numbers of rounds, and none waits for
// the slowest.
template <bool WIDE>
__global__ __launch_bounds__(256) void sample_kernel(
    const float *__restrict__ pdf, const float *__restrict__ marg, const float *__restrict__ cond,
    uint32_t L, int H, int W, const uint32_t *__restrict__ leaf, const float2 *__restrict__ u, uint64_t n,
    float *__restrict__ dir, float *__restrict__ pdf_out, uint32_t *__restrict__ bin_out, uint32_t *err) {
  __shared__ float4 sdir[4][48];  // 64 directions of 3 floats for each wavefront
  __shared__ uint4 slot[WIDE ? 4 : 1][WIDE ? 64 : 1];
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  float *sd = reinterpret_cast<float *>(sdir[wave]);
  const bool dir16 = (reinterpret_cast<uintptr_t>(dir) & 15) == 0;
  for (uint64_t base = (uint64_t)blockIdx.x * 256 + wave * 64; base < n; base += (uint64_t)gridDim.x * 256) {
    const uint64_t q = base + (uint64_t)lane;
    float d[3] = {0.0f, 0.0f, 0.0f}, p = 0.0f;
    uint32_t b = 0, l = 0;
    float2 uu{0.0f, 0.0f};
    bool act = false;
    if (q < n) {
      l = leaf[q];
      uu = u[q];
      if (l >= L || !(uu.x >= 0.0f && uu.x < 1.0f) || !(uu.y >= 0.0f && uu.y < 1.0f)) {
        const float qnan = __int_as_float(0x7fc00000);
        d[0] = d[1] = d[2] = p = qnan;
        b = 0xffffffffu;
        raise_err(err, ERR_RANGE);
      } else {
        act = true;
      }
    }
    guided_sample<WIDE>(pdf, marg, cond, l, H, W, uu.x, uu.y, act, slot[WIDE ? wave : 0], d, &p, &b);
    if (q < n) {
      pdf_out[q] = p;
      if (bin_out) bin_out[q] = b;
    }
    sd[3 * lane] = d[0];
    sd[3 * lane + 1] = d[1];
    sd[3 * lane + 2] = d[2];
    wave_sync();
    const uint64_t nb = n - base < 64 ? n - base : 64;
    float *dst = dir + 3 * base;  // 16-byte aligned when dir is (3 * 64 * 4 bytes per wavefront)
    if (nb == 64 && dir16) {
      if (lane < 48) reinterpret_cast<float4 *>(dst)[lane] = sdir[wave][lane];
    } else {
      for (int k = lane; k < 3 * (int)nb; k += 64) dst[k] = sd[k];
    }
    wave_sync();
  }
}

// ------------------------------------------------------- one-sample MIS
constexpr float INV_PI = 0.3183098861837907f;

// alpha_j from the path statistics: FP64 quotient of the two averages once
// both strategies have MIS_MIN bounces, clamped to [0.2, 0.8]
constexpr uint32_t MIS_MIN = 50;
__global__ void mis_alpha_kernel(const float *__restrict__ nu_b, const float *__restrict__ nu_g,
                                 const uint32_t *__restrict__ q_b, const uint32_t *__restrict__ q_g, uint32_t L,
                                 float *__restrict__ alpha, uint32_t *err) {
  for (uint32_t l = blockIdx.x * blockDim.x + threadIdx.x; l < L; l += gridDim.x * blockDim.x) {
    const double nb = nu_b[l], ng = nu_g[l];
    const uint32_t qb = q_b[l], qg = q_g[l];
    if (!(nb >= 0.0 && ng >= 0.0 && isfinite(nb) && isfinite(ng))) {
      alpha[l] = 0.5f;
      raise_err(err, ERR_RANGE);
      continue;
    }
    double a = 0.5;
    if (qb >= MIS_MIN && qg >= MIS_MIN) {
      const double mb = nb / (double)qb, mg = ng / (double)qg;
      if (mb + mg > 0.0) a = mb / (mb + mg);
    }
    alpha[l] = (float)fmin(fmax(a, 0.2), 0.8);
  }
}

// Cosine-lobe direction about the unit normal (nx, ny, nz) from (u1, u2):
// disk point (sqrt(u1), 2 pi u2) lifted to the hemisphere, in the frame of
// Duff et al. 2017 (sign of nz with +0 counted as positive)
__device__ __forceinline__ void cosine_sample(float nx, float ny, float nz, float u1, float u2, float *w) {
  const float sg = nz >= 0.0f ? 1.0f : -1.0f;
  const float a = -1.0f / (sg + nz);
  const float b = nx * ny * a;
  const float tx = 1.0f + sg * nx * nx * a, ty = sg * b, tz = -sg * nx;
  const float bx = b, by = sg + ny * ny * a, bz = -ny;
  const float r = sqrtf(u1);
  float sp, cp;
  sincosf(6.283185307179586f * u2, &sp, &cp);
  const float h = sqrtf(fmaxf(0.0f, 1.0f - u1));
  const float x = r * cp, y = r * sp;
  w[0] = x * tx + y * bx + h * nx;
  w[1] = x * ty + y * by + h * ny;
  w[2] = x * tz + y * bz + h * nz;
}

// The mixture a p_BSDF(w) + (1 - a) g, spelled out with explicit fused
// multiply-adds so that sampling and evaluation round it identically
// (contraction left to the compiler could differ between the two kernels).
__device__ __forceinline__ float mis_mixture(float a, float nx, float ny, float nz, const float *w, float g) {
  const float c = fmaf(nz, w[2], fmaf(ny, w[1], nx * w[0]));
  const float pb = fmaxf(0.0f, c) * INV_PI;
  return fmaf(a, pb, (1.0f - a) * g);
}

template <bool WIDE>
__global__ __launch_bounds__(256) void sample_mis_kernel(
    const float2 *__restrict__ bnd, const float *__restrict__ pdf, const float *__restrict__ marg,
    const float *__restrict__ cond, uint32_t L, int H, int W, const float *__restrict__ alpha,
    const uint32_t *__restrict__ leaf, const float *__restrict__ normal, const float *__restrict__ u, uint64_t n,
    float *__restrict__ dir, float *__restrict__ pdf_out, uint8_t *__restrict__ strat, uint32_t *err) {
  __shared__ float2 q4[256];
  __shared__ uint4 slot[WIDE ? 4 : 1][WIDE ? 64 : 1];
  load_quarter(bnd, W, q4);
  __syncthreads();
  const int lane = (int)threadIdx.x & 63, wave = (int)threadIdx.x >> 6;
  for (uint64_t base = (uint64_t)blockIdx.x * 256 + wave * 64; base < n; base += (uint64_t)gridDim.x * 256) {
    const uint64_t q = base + (uint64_t)lane;
    uint32_t l = 0;
    float u0 = 0.0f, u1 = 0.0f, u2 = 0.0f, nx = 0.0f, ny = 0.0f, nz = 0.0f, a = 0.0f;
    bool ok = false, bsdf = false;
    if (q < n) {
      l = leaf[q];
      u0 = u[3 * q], u1 = u[3 * q + 1], u2 = u[3 * q + 2];
      nx = normal[3 * q], ny = normal[3 * q + 1], nz = normal[3 * q + 2];
      ok = !(l >= L || !(u0 >= 0.0f && u0 < 1.0f) || !(u1 >= 0.0f && u1 < 1.0f) || !(u2 >= 0.0f && u2 < 1.0f) ||
             !finite3(nx, ny, nz));
      if (ok) {
        a = alpha[l];
        bsdf = u0 < a;
      }
    }
    float w[3], g;
    uint32_t b;
    guided_sample<WIDE>(pdf, marg, cond, l, H, W, u1, u2, ok && !bsdf, slot[WIDE ? wave : 0], w, &g, &b);
    if (q >= n) continue;
    if (!ok) {
      const float qnan = __int_as_float(0x7fc00000);
      dir[3 * q] = qnan;
      dir[3 * q + 1] = qnan;
      dir[3 * q + 2] = qnan;
      pdf_out[q] = qnan;
      if (strat) strat[q] = 0;
      raise_err(err, ERR_RANGE);
      continue;
    }
    if (bsdf) {
      cosine_sample(nx, ny, nz, u1, u2, w);
      const int k = z_row(w[2], H) * W + phi_sector(q4, w[0], w[1], W);
      g = pdf[(size_t)l * H * W + k];
    }
    dir[3 * q] = w[0];
    dir[3 * q + 1] = w[1];
    dir[3 * q + 2] = w[2];
    pdf_out[q] = mis_mixture(a, nx, ny, nz, w, g);
    if (strat) strat[q] = bsdf ? 1 : 0;
  }
}

__global__ __launch_bounds__(256) void eval_mis_kernel(const float2 *__restrict__ bnd, const float *__restrict__ pdf,
                                                       uint32_t L, int H, int W, const float *__restrict__ alpha,
                                                       const uint32_t *__restrict__ leaf,
                                                       const float *__restrict__ normal,
                                                       const float *__restrict__ dir, uint64_t n,
                                                       float *__restrict__ out, uint32_t *err) {
  __shared__ float2 q4[256];
  load_quarter(bnd, W, q4);
  __syncthreads();
  for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < n;
       q += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t l = leaf[q];
    const float w[3] = {dir[3 * q], dir[3 * q + 1], dir[3 * q + 2]};
    const float nx = normal[3 * q], ny = normal[3 * q + 1], nz = normal[3 * q + 2];
    if (l >= L || !finite3(w[0], w[1], w[2]) || !finite3(nx, ny, nz)) {
      out[q] = 0.0f;
      raise_err(err, ERR_RANGE);
      continue;
    }
    const float a = alpha[l];
    const int k = z_row(w[2], H) * W + phi_sector(q4, w[0], w[1], W);
    out[q] = mis_mixture(a, nx, ny, nz, w, pdf[(size_t)l * H * W + k]);
  }
}

__global__ __launch_bounds__(256) void eval_kernel(const float2 *__restrict__ bnd, const float *__restrict__ pdf, uint32_t L, int H, int W,
                                                   const uint32_t *__restrict__ leaf,
                                                   const float *__restrict__ dir, uint64_t n,
                                                   float *__restrict__ out, uint32_t *err) {
  __shared__ float2 q4[256];
  load_quarter(bnd, W, q4);
  __syncthreads();
  for (uint64_t q = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; q < n;
       q += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t l = leaf[q];
    const float x = dir[3 * q], y = dir[3 * q + 1], z = dir[3 * q + 2];
    if (l >= L || !finite3(x, y, z)) {
      out[q] = 0.0f;
      raise_err(err, ERR_RANGE);
      continue;
    }
    const int k = z_row(z, H) * W + phi_sector(q4, x, y, W);
    out[q] = pdf[(size_t)l * H * W + k];
  }
}

size_t grid_for(uint64_t n) {
  const uint64_t b = (n + 255) / 256;
  return (size_t)(b < 262144 ? b : 262144);
}

// Whether a wavefront's searches are done together.  The wide search asks L2
// for less, but a round of it takes longer (queries, sums and results go
// through LDS), so on rows that take several rounds it pays only where the
// memory is what the others wait for: enough queries to fill the chip, and
// tables that do not stay in an XCD's 4 MiB L2.  128x128 maps, lane by lane
// against together: 220 thousand queries on 178 leaves 23.0 / 23.5 us, 400
// thousand 38.0 / 35.2; 3 million on 15 leaves (1 MB) 138 / 147, on 178 209 /
// 174, on 2851 323 / 263.  Rows of up to 64 bins take one or two rounds, and
// together is faster or the same for any number of queries (200 leaves, one call
// and the wait for it): 32x32 maps 1 query 23.0 / 22.7, 1000 28.0 / 25.8, 80
// thousand 27.9 / 27.0, 200 thousand 29.9 / 28.9; 64x64 23.2 / 22.7, 27.3 / 25.7,
// 28.0 / 27.3, 31.7 / 30.4; MIS on 64x64 23.2 / 23.7, 27.6 / 26.5, 28.6 / 27.5,
// 32.8 / 31.4.
// A mixture sample searches only half the time and waits for memory less, so there
// the tables have to be further past the L2, and for many queries further still.
// Lane by lane against together, 300 and 600 thousand queries: one leaf of
// 1024x1024 (4 MiB) 14.4 / 14.8 and 21.7 / 24.1 us, 5 of 512x512 (5 MiB) 14.8 / 14.3
// and 23.2 / 23.4, 100 of 128x128 (6 MiB) 15.2 / 14.3 and 25.0 / 24.1; 1 and 10
// million: 1024x1024 30.9 / 34.8 and 262 / 299, 8 of 512x512 35.3 / 36.9 and 289 /
// 303, 200 of 128x128 (13 MiB) 37.8 / 38.8 and 314 / 316, 8 of 1024x1024 (32 MiB)
// 39.7 / 42.0 and 333 / 331, 4000 of 128x128 47.5 / 47.7 and 424 / 409.
bool wide_search(const npg_tables &t, uint64_t n, bool mis) {
  const uint64_t fits = (!mis ? 4u : n < 900000 ? 6u : 16u) << 20;
  return (t.H <= 64 && t.W <= 64) || (n >= (1u << 18) && 4ull * t.L * t.H * (t.W + 1) > fits);
}

}  // namespace

hipError_t launch_sample(const npg_tables &t, const uint32_t *leaf, const float *u, uint64_t n,
                         float *dir, float *pdf, uint32_t *bin, uint32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(wide_search(t, n, false) ? sample_kernel<true> : sample_kernel<false>, dim3(grid_for(n)),
                     dim3(256), 0, s, t.pdf_dev, t.marg_dev, t.cond_dev, t.L, t.H, t.W, leaf,
                     reinterpret_cast<const float2 *>(u), n, dir, pdf, bin, err);
  return hipGetLastError();
}

hipError_t launch_mis_alpha(const float *nu_b, const float *nu_g, const uint32_t *q_b, const uint32_t *q_g,
                            uint32_t L, float *alpha, uint32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(mis_alpha_kernel, dim3(grid_for(L)), dim3(256), 0, s, nu_b, nu_g, q_b, q_g, L, alpha, err);
  return hipGetLastError();
}

hipError_t launch_sample_mis(const float2 *bnd, const npg_tables &t, const float *alpha, const uint32_t *leaf,
                             const float *normal, const float *u, uint64_t n, float *dir, float *pdf,
                             uint8_t *strat, uint32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(wide_search(t, n, true) ? sample_mis_kernel<true> : sample_mis_kernel<false>, dim3(grid_for(n)),
                     dim3(256), 0, s, bnd, t.pdf_dev, t.marg_dev, t.cond_dev, t.L, t.H, t.W, alpha, leaf, normal, u, n,
                     dir, pdf, strat, err);
  return hipGetLastError();
}

hipError_t launch_eval_mis(const float2 *bnd, const npg_tables &t, const float *alpha, const uint32_t *leaf,
                           const float *normal, const float *dir, uint64_t n, float *pdf, uint32_t *err,
                           hipStream_t s) {
  hipLaunchKernelGGL(eval_mis_kernel, dim3(grid_for(n)), dim3(256), 0, s, bnd, t.pdf_dev, t.L, t.H, t.W, alpha, leaf,
                     normal, dir, n, pdf, err);
  return hipGetLastError();
}

hipError_t launch_eval(const float2 *bnd, const npg_tables &t, const uint32_t *leaf, const float *dir, uint64_t n, float *pdf,
                       uint32_t *err, hipStream_t s) {
  hipLaunchKernelGGL(eval_kernel, dim3(grid_for(n)), dim3(256), 0, s, bnd, t.pdf_dev, t.L, t.H, t.W, leaf, dir,
                     n, pdf, err);
  return hipGetLastError();
}
