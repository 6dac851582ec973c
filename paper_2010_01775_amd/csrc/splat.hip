// Photon binning into per-leaf energy/count maps, and the mean-1 input
// normalisation of the energy map.
//
// Splat: one workgroup per (leaf, band of rows), or several per band that each
// take a slice of a large leaf's photons when there are few leaves.  The band's bins live in LDS
// as packed 64-bit words: bits 0..46 accumulate energy, bits 47..63 the
// photon count.  A photon adds (1 << 47) + w with one LDS atomic.  Packing is
// exact as long as a round covers at most 2^15 photons (energy < 2^47, count
// <= 2^15 < 2^17); after each round the words are drained into per-thread
// 64-bit registers, so leaves of any size are exact.  Integer sums make the
// result independent of the order photons are processed in.
#include <algorithm>

#include "npg_internal.h"

namespace {

constexpr int SPLAT_THREADS = 1024;
constexpr int SPLAT_MAX_BINS = 16384;           // 128 KiB of packed words
constexpr uint32_t SPLAT_ROUND = 1u << 15;     // photons per drain round
constexpr int PACK_SHIFT = 47;
constexpr unsigned long long PACK_MASK = (1ull << PACK_SHIFT) - 1;

// Where a workgroup finds its leaf's photons: a CSR batch (one direction and
// weight array, offsets, optional permutation) or per-leaf descriptors
// (serving batches mix leaves of several requests).
struct CsrLeaves {
  const float *dir;
  const uint32_t *w;
  const uint32_t *perm;
  const uint32_t *off;
  __device__ void range(int leaf, uint32_t *b, uint32_t *e) const {
    *b = off[leaf];
    *e = off[leaf + 1];
  }
  __device__ uint32_t idx(int, uint32_t i) const { return perm ? perm[i] : i; }
  __device__ const float *dirs(int) const { return dir; }
  __device__ const uint32_t *ws(int) const { return w; }
};

struct DescLeaves {
  const npg_leaf_desc *d;
  __device__ void range(int leaf, uint32_t *b, uint32_t *e) const {
    *b = d[leaf].begin;
    *e = d[leaf].begin + d[leaf].count;
  }
  __device__ uint32_t idx(int, uint32_t i) const { return i; }
  __device__ const float *dirs(int leaf) const { return d[leaf].dir; }
  __device__ const uint32_t *ws(int leaf) const { return d[leaf].w; }
};

// How the leaves of a batch are cut into slices (smax 1: no leaf is): a leaf of P
// photons into min(smax, P / slice, sqrt(P / unit)), given the reciprocals.
struct SplatCut {
  uint32_t smax;
  float per_slice, per_unit;
};
__device__ __forceinline__ uint32_t splat_slices(uint32_t beg, uint32_t end, SplatCut cut) {
  const float p = end > beg ? (float)(end - beg) : 0.0f;
  return max(1u, min(cut.smax, (uint32_t)fminf(p * cut.per_slice, sqrtf(p * cut.per_unit))));
}

// Zeroes the maps of the leaves whose slices will be added up in memory.
template <class LS>
__global__ __launch_bounds__(256) void splat_zero_kernel(LS src, int HW, SplatCut cut,
                                                         uint64_t *__restrict__ energy,
                                                         uint32_t *__restrict__ count) {
  const int leaf = blockIdx.x;
  uint32_t beg, end;
  src.range(leaf, &beg, &end);
  if (splat_slices(beg, end, cut) == 1) return;
  const size_t base = (size_t)leaf * HW;
  for (int k = blockIdx.y * 256 + threadIdx.x; k < HW; k += gridDim.y * 256) {
    energy[base + k] = 0;
    if (count) count[base + k] = 0;
  }
}

// CUT: a leaf of many photons is shared by several workgroups per band
// (blockIdx.z), whose exact sums meet in global integer atomics (the maps hold
// zeros or the sums to accumulate onto).
template <int BPT, int NT, bool CUT, class LS>
__global__ __launch_bounds__(NT) void splat_kernel(
    const float2 *__restrict__ bnd, LS src, int H, int W, int band_rows, SplatCut cut, uint64_t *__restrict__ energy,
    uint32_t *__restrict__ count, int accumulate, uint32_t *err) {
  extern __shared__ unsigned long long acc[];
  __shared__ float2 q4[256];
  const int leaf = blockIdx.x;
  uint32_t beg, end, ns = 1;
  if constexpr (CUT) {
    src.range(leaf, &beg, &end);
    ns = splat_slices(beg, end, cut);
    if (blockIdx.z >= ns) return;
    if (ns > 1) {
      const uint32_t per = (end - beg) / ns;
      const uint32_t b0 = beg + blockIdx.z * per;
      end = blockIdx.z + 1 == ns ? end : b0 + per;
      beg = b0;
    }
  }
  const int row0 = blockIdx.y * band_rows;
  const int nb = band_rows * W;
  const int tid = threadIdx.x;
  for (int k = tid; k < nb; k += NT) acc[k] = 0ull;
  load_quarter(bnd, W, q4);
  unsigned long long e[BPT];
  uint32_t c[BPT];
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    e[j] = 0ull;
    c[j] = 0u;
  }
  if constexpr (!CUT) src.range(leaf, &beg, &end);
  const float *dir = src.dirs(leaf);
  const uint32_t *w = src.ws(leaf);
  bool bad = false;
  __syncthreads();
  for (uint64_t r0 = beg; r0 < end; r0 += SPLAT_ROUND) {
    const uint32_t r1 = (uint32_t)min((uint64_t)end, r0 + SPLAT_ROUND);
    // PB photons per thread and step: all their loads are issued before
    // the first bin is computed
    constexpr int PB = 2;
    for (uint32_t i0 = (uint32_t)r0 + tid; i0 < r1; i0 += PB * NT) {
      float x[PB], y[PB], z[PB];
      uint32_t wp[PB];
#pragma unroll
      for (int j = 0; j < PB; ++j) {
        const uint32_t i = i0 + j * NT;
        const uint32_t p = src.idx(leaf, i < r1 ? i : i0);
        x[j] = dir[3 * (size_t)p];
        y[j] = dir[3 * (size_t)p + 1];
        z[j] = dir[3 * (size_t)p + 2];
        wp[j] = w[p];
      }
#pragma unroll
      for (int j = 0; j < PB; ++j) {
        if (i0 + j * NT >= r1) continue;
        if (!finite3(x[j], y[j], z[j])) {
          bad = true;
          continue;
        }
        const int iz = z_row(z[j], H) - row0;
        if (iz < 0 || iz >= band_rows) continue;
        const int k = iz * W + phi_sector(q4, x[j], y[j], W);
        atomicAdd(&acc[k], (1ull << PACK_SHIFT) + (unsigned long long)wp[j]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
      const int k = tid + j * NT;
      if (k < nb) {
        const unsigned long long v = acc[k];
        acc[k] = 0ull;
        e[j] += v & PACK_MASK;
        c[j] += (uint32_t)(v >> PACK_SHIFT);
      }
    }
    __syncthreads();
  }
  if (bad && blockIdx.y == 0) raise_err(err, ERR_RANGE);
  const size_t base = ((size_t)leaf * H + row0) * W;
#pragma unroll
  for (int j = 0; j < BPT; ++j) {
    const int k = tid + j * NT;
    if (k < nb) {
      if (CUT && ns > 1) {
        if (c[j]) {
          atomicAdd(reinterpret_cast<unsigned long long *>(energy + base + k), e[j]);
          if (count) atomicAdd(count + base + k, c[j]);
        }
      } else if (accumulate) {
        energy[base + k] += e[j];
        if (count) count[base + k] += c[j];
      } else {
        energy[base + k] = e[j];
        if (count) count[base + k] = c[j];
      }
    }
  }
}

// Whether and how a batch's leaves are cut.  One workgroup takes 1.1 ns per
// photon of its leaf, and on few leaves the rest of the chip is idle.  The slices
// of a leaf add their sums in memory: n slices of all L leaves touch n L HW / 16
// lines of 128 bytes, 12 G lines/s, half as many again with counts.  The two
// together are least at n^2 = P / unit with unit = L HW / 200; a sixth of that
// here, as the leaves of a batch differ in size and only the large ones are cut:
// requests of 11 to 100 leaves of lognormal sizes about 10 to 30 thousand take
// within 1 % of what they take with 2048 photons a slice, whatever L HW.  A leaf is
// not cut below two slices of L HW / 192, so that leaves of one size are not cut
// for nothing.
// Whole and cut, us: 64x64 maps, 11 leaves of 30,000 photons 42 / 12.5, 64 leaves
// 45 / 25; 128x128 maps, 11 leaves 32 / 19; lognormal sizes about 3000 on 200
// 64x64 maps 77 / 25.  Leaves of 8000 on 128 128x128 maps stay whole (15.5; 39 in
// slices of 2048: the fused call 357 -> 333).
// The zeroing pass costs 2.5 us whatever the photons, which the host does not
// know.  A splat on its own leaves it out where only leaves of more than the
// octree's 8192 photons would be cut (64x64 maps: from 193 leaves on; 200 of 300
// photons 8.9 us queued, 11.5 with the pass).  In front of a network (`chain`)
// it is 1.5 % of the call at such sizes, and stays for the few large leaves up to
// 512 leaf bands, from where on the bands fill the chip by themselves.
SplatCut splat_cut(uint32_t L, int H, int W, int band_rows, bool count, bool chain) {
  const uint64_t bands = (uint64_t)(H / band_rows);
  // four photons per thread of a 512-thread workgroup: on fewer, the loads of
  // one step already cover the slice
  const float slice = std::max(2048.0f, (float)L * H * W / (count ? 128 : 192));
  if (L * bands > 512 || (!chain && 2 * slice > 8192)) return {1, 0.0f, 0.0f};
  return {(uint32_t)std::min<uint64_t>(64, 1024 / (L * bands)), 1.0f / slice, (count ? 768.0f : 1152.0f) / ((float)L * H * W)};
}

template <int BPT, int NT, bool CUT, class LS>
hipError_t launch_splat_k(const float2 *bnd, const LS &src, uint32_t L, int H, int W, int band_rows, SplatCut cut,
                          uint64_t *energy, uint32_t *count, int accumulate, uint32_t *err, hipStream_t s) {
  const size_t lds = sizeof(unsigned long long) * (size_t)band_rows * W;
  static std::atomic<uint64_t> attr{0};
  if (npg_first_on_device(attr)) {
    hipError_t e = hipFuncSetAttribute((const void *)splat_kernel<BPT, NT, CUT, LS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       SPLAT_MAX_BINS * sizeof(unsigned long long));
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((splat_kernel<BPT, NT, CUT, LS>), dim3(L, (unsigned)(H / band_rows), cut.smax), dim3(NT), lds, s,
                     bnd, src, H, W, band_rows, cut, energy, count, accumulate, err);
  return hipGetLastError();
}

template <int BPT, int NT, class LS>
hipError_t launch_splat_t(const float2 *bnd, const LS &src, uint32_t L, int H, int W, int band_rows,
                          uint64_t *energy, uint32_t *count, int accumulate, bool chain, uint32_t *err,
                          hipStream_t s) {
  const SplatCut cut = splat_cut(L, H, W, band_rows, count != nullptr, chain);
  if (cut.smax == 1)
    return launch_splat_k<BPT, NT, false>(bnd, src, L, H, W, band_rows, cut, energy, count, accumulate, err, s);
  if (!accumulate) {
    hipLaunchKernelGGL(splat_zero_kernel<LS>, dim3(L, (unsigned)(H * W + 4095) / 4096), dim3(256), 0, s, src, H * W,
                       cut, energy, count);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_splat_k<BPT, NT, true>(bnd, src, L, H, W, band_rows, cut, energy, count, accumulate, err, s);
}

// Maps of up to 4096 bins take 512-thread workgroups (four fit a CU, so a
// 1024-leaf batch is resident at once); larger bands 1024 threads.
template <class LS>
hipError_t launch_splat_any(const float2 *bnd, const LS &src, uint32_t L, int H, int W, uint64_t *energy,
                            uint32_t *count, int accumulate, bool chain, uint32_t *err, hipStream_t s) {
  int band_rows = H;
  while (band_rows * W > SPLAT_MAX_BINS) band_rows >>= 1;
  const int nb = band_rows * W;
  if (nb <= 4096) {
    switch ((nb + 511) / 512) {
      case 1: return launch_splat_t<1, 512>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
      case 2: return launch_splat_t<2, 512>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
      case 4: return launch_splat_t<4, 512>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
      default: return launch_splat_t<8, 512>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
    }
  }
  switch ((nb + SPLAT_THREADS - 1) / SPLAT_THREADS) {
    case 8: return launch_splat_t<8, SPLAT_THREADS>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
    default: return launch_splat_t<16, SPLAT_THREADS>(bnd, src, L, H, W, band_rows, energy, count, accumulate, chain, err, s);
  }
}

// Per-leaf energy total (exact u64 sum), stored as binary64.
__global__ __launch_bounds__(256) void leaf_total_kernel(const uint64_t *__restrict__ energy, int HW,
                                                         double *__restrict__ tot) {
  __shared__ unsigned long long part[4];
  const int leaf = blockIdx.x;
  const uint64_t *e = energy + (size_t)leaf * HW;
  unsigned long long s = 0;
  for (int k = threadIdx.x; k < HW; k += 256) s += e[k];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) tot[leaf] = (double)(part[0] + part[1] + part[2] + part[3]);
}

// x = H*W*E / total in binary64, rounded to float32; zero map for total 0.
__global__ void apply_scale_kernel(const uint64_t *__restrict__ energy, const double *__restrict__ tot,
                                   int HW, int log2HW, size_t n, float *__restrict__ x) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x) {
    const double t = tot[i >> log2HW];
    x[i] = t > 0.0 ? (float)((double)HW * (double)energy[i] / t) : 0.0f;
  }
}

}  // namespace

hipError_t launch_splat(const float2 *bnd, const float *dir, const uint32_t *w, const uint32_t *perm,
                        const uint32_t *off, uint32_t L, int H, int W, uint64_t *energy,
                        uint32_t *count, int accumulate, bool chain, uint32_t *err, hipStream_t s) {
  return launch_splat_any(bnd, CsrLeaves{dir, w, perm, off}, L, H, W, energy, count, accumulate, chain, err, s);
}

hipError_t launch_splat_desc(const float2 *bnd, const npg_leaf_desc *d, uint32_t L, int H, int W,
                             uint64_t *energy, uint32_t *err, hipStream_t s) {
  return launch_splat_any(bnd, DescLeaves{d}, L, H, W, energy, nullptr, 0, true, err, s);
}

hipError_t launch_leaf_scale(const uint64_t *energy, uint32_t L, int HW, double *tot, hipStream_t s) {
  hipLaunchKernelGGL(leaf_total_kernel, dim3(L), dim3(256), 0, s, energy, HW, tot);
  return hipGetLastError();
}

hipError_t launch_apply_scale(const uint64_t *energy, const double *tot, uint32_t L, int HW,
                              float *x, hipStream_t s) {
  const size_t n = (size_t)L * HW;
  int log2HW = 0;
  while ((1 << log2HW) < HW) ++log2HW;
  const size_t blocks = std::min<size_t>((n + 255) / 256, 65536);
  hipLaunchKernelGGL(apply_scale_kernel, dim3(blocks), dim3(256), 0, s, energy, tot, HW, log2HW, n, x);
  return hipGetLastError();
}
