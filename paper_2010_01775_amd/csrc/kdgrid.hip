// The paper's hierarchical grid: a regular grid of res^3 voxels, valid
// voxels marked by camera-path bounce points, and every valid voxel split
// into a local binary KD tree (Sec. 7.1 "Voxel subdivision"; Sec. 8,
// path-guiding details).
//
// Build, level by level (every node of a level is independent):
//   1. voxel id of each photon (FP64 rule; invalid voxels get a sentinel
//      key), stable radix sort of (voxel, photon index): the photons of a
//      voxel become one contiguous segment, in ascending photon index;
//   2. segment starts = the roots, in ascending voxel id: a bit per photon
//      marks the first of its segment, and the rank of a root is a scan over
//      the words of that bitmap;
//   3. per level: the split test of each node (count, and the normal
//      variance from exact integer sums) and, for a splitting node, the
//      median coordinate on the longest axis by an exact radix select over
//      its segment (from the highest bit where the node's keys differ), one
//      wavefront per node of up to 2048 photons and one workgroup per larger
//      node; then a stable partition of each
//      splitting node's segment into its two child segments, in place
//      (child slots from a scan of the split flags, so node ids do not
//      depend on scheduling); a node that does not split keeps its segment
//      where it is and becomes a leaf;
//   4. leaves ranked by segment start, with a bitmap again: depth-first
//      order inside a voxel, voxels ascending, since every split keeps its
//      children inside the parent's segment, first child first.
// The number of nodes of a level stays on the device (LevelState): the kernels of
// a level are queued with grids that stride over however many nodes there are,
// KD_AHEAD levels before the host knows whether the first of them has any.
// Waiting for each level's count cost 60 us a level, as much as a level's work from
// the fourth on.  20 million photons in 100^3 voxels, depth 8, with 2 million
// locations: 3.3 to 3.75 -> 2.3 to 2.65 ms by the photons, together with the
// bitmaps (250 us of flags and scans over the photons -> 60), wavefronts instead
// of workgroups for small nodes in the partition (250 -> 100 us a level where 300
// thousand nodes hold the photons), 1024 threads for large ones, and photons
// copied into voxel order by the first level (the others' selections 150 -> 90
// us).
// Point location: voxel id, then down the tree by the split comparisons.
#include "npg_internal.h"

namespace {

constexpr int KD_THREADS = 256;
constexpr int KD_BIG = 1024;  // workgroups that take one large node
constexpr uint32_t KD_NONE = 0xFFFFFFFFu;
constexpr double KD_QSCALE = 1048576.0;  // normals quantised to multiples of 2^-20

struct GridDev {
  int res;
  float lo[3];
  double invr[3];  // res / (hi - lo)
  double step[3];  // (hi - lo) / res
};

// Monotone map of float32 to uint32 (-0 read as +0): a < b iff key(a) < key(b).
__device__ __forceinline__ uint32_t okey(float x) {
  const uint32_t b = __float_as_uint(x == 0.0f ? 0.0f : x);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float okey_inv(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// Voxel coordinate on one axis: floor((p - lo) * invr) in FP64 (no
// contraction), clamped to [0, res-1].
__device__ __forceinline__ int vox_axis(float p, float lo, double invr, int res) {
  const double t = __dmul_rn(__dsub_rn((double)p, (double)lo), invr);
  const double f = floor(t);
  return f < 0.0 ? 0 : (f > (double)(res - 1) ? res - 1 : (int)f);
}

__device__ __forceinline__ bool finite3(float x, float y, float z) {
  return isfinite(x) && isfinite(y) && isfinite(z);
}

__device__ __forceinline__ uint32_t vox_id(const GridDev &g, float x, float y, float z) {
  const uint32_t r = (uint32_t)g.res;
  return (uint32_t)vox_axis(x, g.lo[0], g.invr[0], g.res) +
         r * ((uint32_t)vox_axis(y, g.lo[1], g.invr[1], g.res) + r * (uint32_t)vox_axis(z, g.lo[2], g.invr[2], g.res));
}

__global__ __launch_bounds__(256) void kd_mark_kernel(GridDev g, const float *__restrict__ p, uint64_t n,
                                                      uint8_t *__restrict__ valid, uint32_t *err) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const float x = p[3 * i], y = p[3 * i + 1], z = p[3 * i + 2];
    if (!finite3(x, y, z)) {
      raise_err(err, ERR_RANGE);
      continue;
    }
    valid[vox_id(g, x, y, z)] = 1;
  }
}

// key = voxel id, or `sent` (sorts last) for an invalid voxel or a bad
// position; a non-finite position, or normal of a photon in a valid voxel,
// raises the range error
__global__ __launch_bounds__(256) void kd_keys_kernel(GridDev g, const float *__restrict__ p,
                                                      const float *__restrict__ nrm, uint64_t n,
                                                      const uint8_t *__restrict__ valid, uint32_t sent,
                                                      uint32_t *__restrict__ key, uint32_t *err) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const float x = p[3 * i], y = p[3 * i + 1], z = p[3 * i + 2];
    uint32_t k = sent;
    if (!finite3(x, y, z)) {
      raise_err(err, ERR_RANGE);
    } else {
      const uint32_t v = vox_id(g, x, y, z);
      if (!valid || valid[v]) {
        k = v;
        if (nrm && !finite3(nrm[3 * i], nrm[3 * i + 1], nrm[3 * i + 2])) raise_err(err, ERR_RANGE);
      }
    }
    key[i] = k;
  }
}

// What a build keeps on the device about a level, and about the whole.
struct LevelState {
  uint32_t active;     // nodes
  uint32_t leaf_base;  // leaves of the levels above
  uint32_t nodes;      // node ids given out up to and including this level
  uint32_t nbig;       // nodes of more than KD_WAVE_MAX photons
  uint32_t nsplit;     // nodes that split
};
constexpr int KD_LEVELS = 18;  // max_depth <= 16, and one more
struct BuildState {
  uint32_t nvalid;  // photons in valid voxels
  uint32_t roots;
  uint32_t over;  // a level did not fit max_leaves
  uint32_t err;   // the error word when the build ended
  LevelState lv[KD_LEVELS];  // the one after the last level queued holds the totals
};

// bits: 1 at the first photon of each valid voxel's segment; cnt[w] = number
// of bits of word w; *nvalid = number of photons in valid voxels (the
// sentinel keys sort last); iota (or null) receives 0, 1, ...  A wavefront takes
// SEG_G groups of 64 keys.
constexpr int SEG_G = 8;
__global__ __launch_bounds__(256) void kd_seg_kernel(const uint32_t *__restrict__ ks, uint64_t n, uint32_t sent,
                                                     uint32_t *__restrict__ bits, uint32_t *__restrict__ cnt,
                                                     uint32_t *__restrict__ iota, BuildState *st) {
  const int lane = threadIdx.x & 63;
  const uint64_t nw = (n + 31) / 32, span = 64 * SEG_G;
  for (uint64_t i0 = (blockIdx.x * 4ull + (threadIdx.x >> 6)) * span; i0 < n; i0 += (uint64_t)gridDim.x * 4 * span) {
    uint32_t k[SEG_G];
#pragma unroll
    for (int g = 0; g < SEG_G; ++g) {
      const uint64_t i = i0 + 64 * g + lane;
      k[g] = i < n ? ks[i] : sent;
    }
    uint32_t before = i0 ? ks[i0 - 1] : KD_NONE;  // KD_NONE: no voxel id and not the sentinel
    uint32_t word = 0;
#pragma unroll
    for (int g = 0; g < SEG_G; ++g) {
      const uint64_t i = i0 + 64 * g + lane;
      const uint32_t up = __shfl_up(k[g], 1), prev = lane ? up : before;
      before = __shfl(k[g], 63);
      const uint64_t m = __ballot(i < n && k[g] != sent && k[g] != prev);
      if ((lane >> 1) == g) word = (uint32_t)(lane & 1 ? m >> 32 : m);
      if (i < n) {
        if (iota) iota[i] = (uint32_t)i;
        if (k[g] == sent && prev != sent && i) st->nvalid = (uint32_t)i;
        if (k[g] != sent && i + 1 == n) st->nvalid = (uint32_t)n;
      }
    }
    const uint64_t w = i0 / 32 + lane;
    if (lane < 2 * SEG_G && w < nw) {
      bits[w] = word;
      cnt[w] = (uint32_t)__popc(word);
    }
  }
}

__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t *__restrict__ a, uint64_t n, int32_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    a[i] = v;
}

// Per-level node records (structure of arrays).
struct Level {
  uint32_t *start, *count, *id;
  double *box;  // [6] per node: lo xyz, hi xyz
};

// roots: node j = j-th valid non-empty voxel; rank[w] = set bits before word
// w, rank[nw] = all of them.  More roots than max_leaves: none is written.
__global__ __launch_bounds__(256) void kd_roots_kernel(GridDev g, const uint32_t *__restrict__ ks,
                                                       const uint32_t *__restrict__ bits,
                                                       const uint32_t *__restrict__ rank, uint64_t nw, uint32_t cap,
                                                       Level lv, int32_t *__restrict__ cell_root, BuildState *st) {
  const uint32_t n0 = rank[nw];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->roots = n0;
    st->over = n0 > cap ? 1u : 0u;
    st->lv[0].active = n0 > cap ? 0u : n0;
    st->lv[0].nodes = n0;
  }
  if (n0 > cap) return;
  for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < nw; w += (uint64_t)gridDim.x * blockDim.x) {
    uint32_t b = bits[w], j = b ? rank[w] : 0;
    for (; b; b &= b - 1, ++j) {
      const uint32_t i = (uint32_t)(32 * w) + (uint32_t)__builtin_ctz(b), v = ks[i];
      lv.start[j] = i;
      lv.id[j] = j;
      cell_root[v] = (int32_t)j;
      const uint32_t r = (uint32_t)g.res;
      const uint32_t c[3] = {v % r, (v / r) % r, v / (r * r)};
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        lv.box[6 * (size_t)j + a] = __dadd_rn((double)g.lo[a], __dmul_rn((double)c[a], g.step[a]));
        lv.box[6 * (size_t)j + 3 + a] = __dadd_rn((double)g.lo[a], __dmul_rn((double)(c[a] + 1), g.step[a]));
      }
    }
  }
}

// Nodes of more than KD_WAVE_MAX photons take a whole workgroup in the
// selection (those of a level are listed in `big`); smaller ones one wavefront
// each.
constexpr uint32_t KD_WAVE_MAX = 2048;

__device__ __forceinline__ void note_big(uint32_t count, uint32_t j, LevelState *ls, uint32_t *big) {
  if (count > KD_WAVE_MAX) big[atomicAdd(&ls->nbig, 1u)] = j;
}

__global__ __launch_bounds__(256) void kd_root_counts_kernel(Level lv, BuildState *st, uint32_t *__restrict__ big) {
  const uint32_t n0 = st->lv[0].active, nvalid = st->nvalid;
  for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n0; j += gridDim.x * blockDim.x) {
    const uint32_t c = (j + 1 < n0 ? lv.start[j + 1] : nvalid) - lv.start[j];
    lv.count[j] = c;
    note_big(c, j, &st->lv[0], big);
  }
}

// perm: from places in voxel order to the photons there
__global__ __launch_bounds__(256) void kd_final_kernel(const uint32_t *__restrict__ order, uint64_t n,
                                                       const BuildState *st, uint32_t *__restrict__ perm) {
  const uint32_t nvalid = st->nvalid;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
    perm[i] = order[i < nvalid ? perm[i] : (uint32_t)i];
}

// Workgroup-wide sums of three int64 values (exact, so the order is free).
__device__ __forceinline__ void wg_sum3_i64(long long v[3], long long (*red)[KD_BIG / 64]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v[a] += __shfl_xor(v[a], o);
    if (lane == 0) red[a][wave] = v[a];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    long long t = 0;
#pragma unroll
    for (int w = 0; w < KD_BIG / 64; ++w) t += red[a][w];
    v[a] = t;
  }
}

// Split test of one node from its photons' normals: V > split_var, with V
// from exact integer sums (the order of the sums does not matter).
__device__ __forceinline__ bool variance_exceeds(long long sx_, long long sy_, long long sz_, uint32_t M,
                                                 double split_var) {
  const double sx = (double)sx_, sy = (double)sy_, sz = (double)sz_;
  const double num = __dadd_rn(__dadd_rn(__dmul_rn(sx, sx), __dmul_rn(sy, sy)), __dmul_rn(sz, sz));
  const double den = __dmul_rn(__dmul_rn((double)M, (double)M), KD_QSCALE * KD_QSCALE);
  return __dsub_rn(1.0, __ddiv_rn(num, den)) > split_var;
}

// three floats in one access, at any 4-byte boundary
typedef float f32x3 __attribute__((ext_vector_type(3), aligned(4)));
__device__ __forceinline__ f32x3 load3(const float *p, uint32_t i) {
  return *reinterpret_cast<const f32x3 *>(p + 3 * (size_t)i);
}
__device__ __forceinline__ void store3(float *p, uint32_t i, f32x3 v) {
  *reinterpret_cast<f32x3 *>(p + 3 * (size_t)i) = v;
}

// One photon's quantised normal added to s[3]; a non-finite component counts
// as 0 and sets *bad.
__device__ __forceinline__ void add_qnormal(f32x3 n, long long s[3], bool *bad) {
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float v = n[a];
    if (!isfinite(v)) *bad = true;
    const double c = isfinite(v) ? fmin(fmax((double)v, -1.0), 1.0) : 0.0;
    s[a] += (long long)rint(c * KD_QSCALE);
  }
}

// Longest axis of a node's box (ties: the lower axis).
__device__ __forceinline__ uint32_t longest_axis(const double *b) {
  double ext[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) ext[a] = __dsub_rn(b[3 + a], b[a]);
  uint32_t axis = 0;
  if (ext[1] > ext[axis]) axis = 1;
  if (ext[2] > ext[axis]) axis = 2;
  return axis;
}

// Split test and median selection of node j, one workgroup.  Outputs per
// node: sflag (1: splits, also counted in the node's chunk of ccnt), axis,
// the split key and the number of photons below it.  tkey receives the node's
// photon keys on the split axis (aligned with perm) for the partition.
struct SelArgs {
  const float *pos, *nrm;
  const uint32_t *perm;
  Level lv;
  int split_allowed;  // the level lies above max_depth
  double split_count, split_var;
  uint32_t *tkey, *sflag, *sel, *ccnt;
  uint32_t *err;
  // First level, if the later ones are to read the photons in voxel order: what
  // they will read.  The first level gathers photon i of the order from the
  // caller's arrays (a line of memory each, 53 G lines/s) and leaves it here;
  // the others find a node's photons within its voxel's few kilobytes.
  float *pos_s, *nrm_s;
};
constexpr f32x3 NO3 = {0.0f, 0.0f, 0.0f};

__device__ __forceinline__ float axis_of(f32x3 p, uint32_t axis) { return axis == 0 ? p[0] : axis == 1 ? p[1] : p[2]; }
// Nodes that share a counter of splits, and the distance of the counters in
// words: atomics on one 128-byte line are done one after the other (10 ns
// each: 18 counters side by side made 9000 splits take 80 us).
constexpr int KD_CHUNK = 1024, KD_CSTEP = 32;

__device__ __forceinline__ void put_selection(const SelArgs &a, uint32_t j, bool split, uint32_t axis, uint32_t key,
                                              uint32_t less) {
  a.sflag[j] = split ? 1u : 0u;
  a.sel[3 * (size_t)j] = axis;
  a.sel[3 * (size_t)j + 1] = key;
  a.sel[3 * (size_t)j + 2] = less;
  if (split) atomicAdd(&a.ccnt[(size_t)(j / KD_CHUNK) * KD_CSTEP], 1u);
}

__device__ __forceinline__ void select_group(const SelArgs &a, uint32_t j, uint32_t *hist,
                                             long long (*red)[KD_BIG / 64], uint32_t *wsum, uint32_t *pick) {
  const float *pos = a.pos, *nrm = a.nrm;
  const uint32_t *perm = a.perm;
  uint32_t *tkey = a.tkey;
  const uint32_t start = a.lv.start[j], M = a.lv.count[j];
  bool split = false, tested = false;
  if (a.split_allowed && M >= 2) {
    split = (double)M > a.split_count;
    if (!split && nrm) {
      long long s[3] = {0, 0, 0};
      bool bad = false;
      for (uint64_t i = threadIdx.x; i < M; i += KD_BIG) {
        const f32x3 v = load3(nrm, perm[start + i]);
        if (a.nrm_s) store3(a.nrm_s, start + (uint32_t)i, v);
        add_qnormal(v, s, &bad);
      }
      tested = true;
      if (bad) raise_err(a.err, ERR_RANGE);
      wg_sum3_i64(s, red);
      split = variance_exceeds(s[0], s[1], s[2], M, a.split_var);
    }
  }
  uint32_t axis = 0, key = 0, less = 0;
  if (split) {
    axis = longest_axis(a.lv.box + 6 * (size_t)j);
    const bool copy_n = a.nrm_s && !tested;
    // exact selection of the (M/2)-th smallest key, 8 bits per pass
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // keys of the split axis, and their range: bits above the highest one
    // where min and max differ are common to every key (and to the median)
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
    for (uint64_t i0 = threadIdx.x; i0 < M; i0 += 4 * KD_BIG) {  // four keys in flight per lane
      uint32_t ph[4];
      f32x3 x[4] = {NO3, NO3, NO3, NO3}, v[4] = {NO3, NO3, NO3, NO3};
#pragma unroll
      for (int q = 0; q < 4; ++q) ph[q] = i0 + q * KD_BIG < M ? perm[start + i0 + q * KD_BIG] : KD_NONE;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ph[q] == KD_NONE) continue;
        x[q] = load3(pos, ph[q]);
        if (copy_n) v[q] = load3(nrm, ph[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ph[q] == KD_NONE) continue;
        const uint32_t at = start + (uint32_t)i0 + q * KD_BIG, k = okey(axis_of(x[q], axis));
        tkey[at] = k;
        if (a.pos_s) store3(a.pos_s, at, x[q]);
        if (copy_n) store3(a.nrm_s, at, v[q]);
        kmin = min(kmin, k);
        kmax = max(kmax, k);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmin = min(kmin, (uint32_t)__shfl_xor(kmin, o));
      kmax = max(kmax, (uint32_t)__shfl_xor(kmax, o));
    }
    if (lane == 0) {
      wsum[wave] = kmin;
      hist[wave] = kmax;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < KD_BIG / 64; ++w) {
      kmin = min(kmin, wsum[w]);
      kmax = max(kmax, hist[w]);
    }
    __syncthreads();
    // exact selection of the (M/2)-th smallest key, 8 bits per pass from the
    // highest differing bit down
    uint32_t m = M / 2;
    const int h = kmin == kmax ? -1 : 31 - __clz(kmin ^ kmax);
    uint32_t pmask = h < 0 ? 0xFFFFFFFFu : (h >= 31 ? 0u : ~((2u << h) - 1u));
    uint32_t prefix = kmin & pmask;
    for (int hi = h; hi >= 0; hi -= 8) {
      const int sh = hi >= 7 ? hi - 7 : 0;
      const uint32_t dmask = (2u << (hi - sh)) - 1u;
      if (threadIdx.x < 256) hist[threadIdx.x] = 0;
      __syncthreads();
      for (uint64_t i0 = threadIdx.x; i0 < M; i0 += 4 * KD_BIG) {
        uint32_t k[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) k[q] = i0 + q * KD_BIG < M ? tkey[start + i0 + q * KD_BIG] : 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (i0 + q * KD_BIG < M && ((k[q] ^ prefix) & pmask) == 0) atomicAdd(&hist[(k[q] >> sh) & dmask], 1u);
      }
      __syncthreads();
      // inclusive scan of the 256 digit counts (one per thread, the rest idle)
      const uint32_t c = threadIdx.x < 256 ? hist[threadIdx.x] : 0u;
      uint32_t inc = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      if (lane == 63) wsum[wave] = inc;
      __syncthreads();
      for (int w = 0; w < wave && w < 4; ++w) inc += wsum[w];
      const uint32_t exc = inc - c;
      if (exc <= m && m < inc) {  // exactly one digit holds rank m
        pick[0] = threadIdx.x;
        pick[1] = exc;
      }
      __syncthreads();
      const uint32_t d = pick[0], below = pick[1];
      m -= below;
      less += below;
      prefix |= d << sh;
      pmask |= dmask << sh;
      __syncthreads();
    }
    key = prefix;  // all keys equal (h < 0): the common key, nothing below it
    split = less > 0;
  }
  if (threadIdx.x == 0) put_selection(a, j, split, axis, key, less);
}

// Orders this wavefront's LDS accesses before and after it (the lanes of a
// wavefront read what other lanes wrote).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The same with one wavefront for a node of at most REG_MAX photons, its keys in
// registers: the bits of the median from the highest differing one down, each
// from the ballots of the keys that still match (no LDS, no second read of
// the keys; deep levels hold hundreds of thousands of nodes of a few dozen
// photons.  In 4 x 64 registers the bits cost more than the histograms).
constexpr uint32_t REG_MAX = 128;
template <int Q>
__device__ __forceinline__ void select_regs(const SelArgs &a, uint32_t j, uint32_t start, uint32_t M) {
  static_assert(64 * Q <= 1024, "the sums of quantised normals fit 32 bits");
  const int lane = threadIdx.x & 63;
  uint32_t ph[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) ph[q] = 64 * q + lane < M ? a.perm[start + 64 * q + lane] : KD_NONE;
  bool split = false, tested = false;
  if (a.split_allowed && M >= 2) {
    split = (double)M > a.split_count;
    if (!split && a.nrm) {
      long long s64[3] = {0, 0, 0};
      bool bad = false;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        if (ph[q] == KD_NONE) continue;
        const f32x3 v = load3(a.nrm, ph[q]);
        if (a.nrm_s) store3(a.nrm_s, start + 64 * q + lane, v);
        add_qnormal(v, s64, &bad);
      }
      tested = true;
      if (bad) raise_err(a.err, ERR_RANGE);
      int s[3] = {(int)s64[0], (int)s64[1], (int)s64[2]};
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s[c] += __shfl_xor(s[c], o);
      split = variance_exceeds(s[0], s[1], s[2], M, a.split_var);
    }
  }
  uint32_t axis = 0, key = 0, less = 0;
  if (split) {
    axis = longest_axis(a.lv.box + 6 * (size_t)j);
    const bool copy_n = a.nrm_s && !tested;
    float x[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      x[q] = 0.0f;
      if (ph[q] == KD_NONE) continue;
      const f32x3 p = load3(a.pos, ph[q]);
      x[q] = axis_of(p, axis);
      if (a.pos_s) store3(a.pos_s, start + 64 * q + lane, p);
      if (copy_n) store3(a.nrm_s, start + 64 * q + lane, load3(a.nrm, ph[q]));
    }
    uint32_t k[Q], kmin = 0xFFFFFFFFu, kmax = 0;
    uint64_t cand[Q];  // keys that agree with the median so far
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      k[q] = okey(x[q]);
      cand[q] = __ballot(ph[q] != KD_NONE);
      if (ph[q] == KD_NONE) continue;
      a.tkey[start + 64 * q + lane] = k[q];
      kmin = min(kmin, k[q]);
      kmax = max(kmax, k[q]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmin = min(kmin, (uint32_t)__shfl_xor(kmin, o));
      kmax = max(kmax, (uint32_t)__shfl_xor(kmax, o));
    }
    kmin = __builtin_amdgcn_readfirstlane(kmin);
    kmax = __builtin_amdgcn_readfirstlane(kmax);
    uint32_t m = M / 2;
    const int h = kmin == kmax ? -1 : 31 - __clz(kmin ^ kmax);
    key = h < 0 ? kmin : (h >= 31 ? 0u : kmin & ~((2u << h) - 1u));
    for (int b = h; b >= 0; --b) {
      uint64_t z[Q];
      uint32_t c = 0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        z[q] = cand[q] & ~__ballot((k[q] >> b) & 1u);
        c += (uint32_t)__popcll(z[q]);
      }
      const bool low = m < c;
      if (!low) {
        m -= c;
        less += c;
        key |= 1u << b;
      }
#pragma unroll
      for (int q = 0; q < Q; ++q) cand[q] = low ? z[q] : cand[q] & ~z[q];
    }
    split = less > 0;
  }
  if (lane == 0) put_selection(a, j, split, axis, key, less);
}

// The same with one wavefront for a node of at most KD_WAVE_MAX photons; it
// works alone (its own LDS histogram, no workgroup barrier).
__device__ __forceinline__ void select_wave(const SelArgs &a, uint32_t j, uint32_t *hist) {
  const float *pos = a.pos, *nrm = a.nrm;
  const uint32_t *perm = a.perm;
  uint32_t *tkey = a.tkey;
  const int lane = threadIdx.x & 63;
  const uint32_t start = a.lv.start[j], M = a.lv.count[j];
  if (M > KD_WAVE_MAX) return;
  if (M <= 64) return select_regs<1>(a, j, start, M);
  if (M <= REG_MAX) return select_regs<REG_MAX / 64>(a, j, start, M);
  bool split = false, tested = false;
  if (a.split_allowed && M >= 2) {
    split = (double)M > a.split_count;
    if (!split && nrm) {
      long long s[3] = {0, 0, 0};
      bool bad = false;
      for (uint32_t i0 = 0; i0 < M; i0 += 4 * 64) {  // four photons in flight per lane
        uint32_t ph[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t i = i0 + 64 * q + lane;
          ph[q] = i < M ? perm[start + i] : KD_NONE;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (ph[q] == KD_NONE) continue;
          const f32x3 v = load3(nrm, ph[q]);
          if (a.nrm_s) store3(a.nrm_s, start + i0 + 64 * q + lane, v);
          add_qnormal(v, s, &bad);
        }
      }
      tested = true;
      if (bad) raise_err(a.err, ERR_RANGE);
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s[c] += __shfl_xor(s[c], o);
      split = variance_exceeds(s[0], s[1], s[2], M, a.split_var);
    }
  }
  uint32_t axis = 0, key = 0, less = 0;
  if (split) {
    axis = longest_axis(a.lv.box + 6 * (size_t)j);
    const bool copy_n = a.nrm_s && !tested;
    // keys of the split axis and their range (as in select_group)
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
    for (uint32_t i0 = 0; i0 < M; i0 += 4 * 64) {  // four keys in flight per lane
      uint32_t ph[4];
      f32x3 x[4] = {NO3, NO3, NO3, NO3}, v[4] = {NO3, NO3, NO3, NO3};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = i0 + 64 * q + lane;
        ph[q] = i < M ? perm[start + i] : KD_NONE;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ph[q] == KD_NONE) continue;
        x[q] = load3(pos, ph[q]);
        if (copy_n) v[q] = load3(nrm, ph[q]);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (ph[q] == KD_NONE) continue;
        const uint32_t at = start + i0 + 64 * q + lane, k = okey(axis_of(x[q], axis));
        tkey[at] = k;
        if (a.pos_s) store3(a.pos_s, at, x[q]);
        if (copy_n) store3(a.nrm_s, at, v[q]);
        kmin = min(kmin, k);
        kmax = max(kmax, k);
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      kmin = min(kmin, (uint32_t)__shfl_xor(kmin, o));
      kmax = max(kmax, (uint32_t)__shfl_xor(kmax, o));
    }
    uint32_t m = M / 2;
    const int h = kmin == kmax ? -1 : 31 - __clz(kmin ^ kmax);
    uint32_t pmask = h < 0 ? 0xFFFFFFFFu : (h >= 31 ? 0u : ~((2u << h) - 1u));
    uint32_t prefix = kmin & pmask;
    for (int hi = h; hi >= 0; hi -= 8) {
      const int sh = hi >= 7 ? hi - 7 : 0;
      const uint32_t dmask = (2u << (hi - sh)) - 1u;
#pragma unroll
      for (int q = 0; q < 4; ++q) hist[4 * lane + q] = 0;
      wave_sync();
      for (uint32_t i0 = 0; i0 < M; i0 += 4 * 64) {
        uint32_t k[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t i = i0 + 64 * q + lane;
          k[q] = i < M ? tkey[start + i] : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t i = i0 + 64 * q + lane;
          if (i < M && ((k[q] ^ prefix) & pmask) == 0) atomicAdd(&hist[(k[q] >> sh) & dmask], 1u);
        }
      }
      wave_sync();
      // lane l holds digits 4l..4l+3: their counts, the lane total and the
      // exclusive prefix over lanes
      uint32_t c[4], tot = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        c[q] = hist[4 * lane + q];
        tot += c[q];
      }
      uint32_t inc = tot;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      uint32_t exc = inc - tot, dsel = 0, bsel = 0;
      bool hit = false;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (!hit && exc <= m && m < exc + c[q]) {
          hit = true;
          dsel = 4 * lane + q;
          bsel = exc;
        }
        exc += c[q];
      }
      const uint64_t hb = __ballot(hit);  // exactly one lane holds rank m
      const int src = __ffsll((long long)hb) - 1;
      const uint32_t d = __shfl(dsel, src), below = __shfl(bsel, src);
      m -= below;
      less += below;
      prefix |= d << sh;
      pmask |= dmask << sh;
      wave_sync();
    }
    key = prefix;  // all keys equal (h < 0): the common key, nothing below it
    split = less > 0;
  }
  if (lane == 0) put_selection(a, j, split, axis, key, less);
}

// One level's selections: the nodes of `big`, a workgroup of 1024 each, and
// the small ones.  A level lasts as long as its largest node, whose photons go
// through one workgroup: with 256 threads the levels of 20 million photons
// with one voxel of 170 thousand took 200 us each, whatever the others held.
__global__ __launch_bounds__(KD_BIG) void kd_select_big_kernel(SelArgs a, const LevelState *ls,
                                                               const uint32_t *__restrict__ big) {
  __shared__ uint32_t hist[256];
  __shared__ long long red[3][KD_BIG / 64];
  __shared__ uint32_t wsum[KD_BIG / 64];
  __shared__ uint32_t pick[2];
  const uint32_t nb = ls->nbig;
  for (uint32_t bi = blockIdx.x; bi < nb; bi += gridDim.x) {
    __syncthreads();  // shared arrays of the previous node are no longer read
    select_group(a, big[bi], hist, red, wsum, pick);
  }
}

__global__ __launch_bounds__(KD_THREADS) void kd_select_kernel(SelArgs a, const LevelState *ls) {
  __shared__ uint32_t hist[KD_THREADS / 64][256];
  const uint32_t active = ls->active, wave = threadIdx.x >> 6;
  for (uint32_t j = blockIdx.x * (KD_THREADS / 64) + wave; j < active; j += gridDim.x * (KD_THREADS / 64)) {
    wave_sync();
    select_wave(a, j, hist[wave]);
  }
}

// From the split flags of a level: the list of splitting nodes, the leaf
// record of every other node (slot leaf_base + number of non-splitting nodes
// before it) with the bit of its segment start, and the next level's state (its
// number of nodes in the host's memory too, where the host asks for it).
// Every workgroup takes a range of chunks and sums the counters before it.
__global__ __launch_bounds__(256) void kd_lists_kernel(Level lv, BuildState *st, int depth, uint32_t cap,
                                                       uint32_t *__restrict__ sflag,
                                                       const uint32_t *__restrict__ ccnt,
                                                       uint32_t *__restrict__ ccnt_next,
                                                       uint32_t *__restrict__ split_list,
                                                       uint32_t *__restrict__ leaf_start,
                                                       uint32_t *__restrict__ leaf_node,
                                                       uint32_t *__restrict__ leaf_bits, uint32_t *host_active) {
  __shared__ uint32_t wa[4], wb[4];
  const LevelState cur = st->lv[depth];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // the counters of the next level were last used one level ago
  const uint32_t old = depth ? (st->lv[depth - 1].active + KD_CHUNK - 1) / KD_CHUNK : 0;
  for (uint32_t c = blockIdx.x * 256 + threadIdx.x; c < old; c += gridDim.x * 256) ccnt_next[(size_t)c * KD_CSTEP] = 0;
  const uint32_t chunks = (cur.active + KD_CHUNK - 1) / KD_CHUNK;
  const uint32_t per = (chunks + gridDim.x - 1) / gridDim.x;
  const uint32_t c0 = min(chunks, blockIdx.x * per), c1 = min(chunks, c0 + per);
  if (c0 == c1 && blockIdx.x) return;
  uint32_t before = 0, total = 0;
  for (uint32_t c = threadIdx.x; c < chunks; c += 256) {
    const uint32_t v = ccnt[(size_t)c * KD_CSTEP];
    total += v;
    if (c < c0) before += v;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    before += __shfl_xor(before, o);
    total += __shfl_xor(total, o);
  }
  if (lane == 0) {
    wa[wave] = before;
    wb[wave] = total;
  }
  __syncthreads();
  before = wa[0] + wa[1] + wa[2] + wa[3];
  total = wb[0] + wb[1] + wb[2] + wb[3];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    // leaves so far + this level's + at least one per child: the bound keeps
    // the next level's records and every leaf slot within max_leaves
    const uint32_t emitted = cur.leaf_base + (cur.active - total);
    const bool fits = (uint64_t)emitted + 2ull * total <= cap;
    if (!fits) st->over = 1;
    st->lv[depth].nsplit = fits ? total : 0;
    st->lv[depth + 1].active = fits ? 2 * total : 0;
    if (host_active)
      __hip_atomic_store(host_active + depth + 1, fits ? 2 * total : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    st->lv[depth + 1].leaf_base = emitted;
    st->lv[depth + 1].nodes = cur.nodes + 2 * total;
  }
  for (uint32_t c = c0; c < c1; ++c) {
    const uint32_t j0 = c * KD_CHUNK + 4 * threadIdx.x;
    uint32_t f[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f[q] = j0 + q < cur.active ? sflag[j0 + q] : 0u;
      sum += f[q];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t t = __shfl_up(inc, o);
      if (lane >= o) inc += t;
    }
    __syncthreads();
    if (lane == 63) wa[wave] = inc;
    __syncthreads();
    uint32_t r = before + inc - sum;
    for (int w = 0; w < wave; ++w) r += wa[w];
    before += wa[0] + wa[1] + wa[2] + wa[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t j = j0 + q;
      if (j >= cur.active) continue;
      if (f[q]) {
        split_list[r] = j;
        sflag[j] = ++r;  // its place in the list, plus one
      } else {
        const uint32_t slot = cur.leaf_base + (j - r), s0 = lv.start[j];
        leaf_start[slot] = s0;
        leaf_node[slot] = lv.id[j];
        atomicOr(&leaf_bits[s0 >> 5], 1u << (s0 & 31));
      }
    }
  }
}

// What a partition writes besides the photons: the node's record and its two
// children, nodes 2k and 2k + 1 of the next level (k: place in the split list).
__device__ __forceinline__ void put_children(Level lv, Level nx, uint32_t j, uint32_t k, uint32_t base, uint32_t axis,
                                             uint32_t key, uint32_t less, LevelState *next, uint32_t *big,
                                             npg_kd_node *nodes) {
  const uint32_t start = lv.start[j], M = lv.count[j], id = lv.id[j], c0 = base + 2 * k, q0 = 2 * k;
  const float s = okey_inv(key);
  nodes[id].split = s;
  nodes[id].info = (c0 << 2) | axis;
  nx.start[q0] = start;
  nx.count[q0] = less;
  nx.id[q0] = c0;
  nx.start[q0 + 1] = start + less;
  nx.count[q0 + 1] = M - less;
  nx.id[q0 + 1] = c0 + 1;
  note_big(less, q0, next, big);
  note_big(M - less, q0 + 1, next, big);
  const double *b = lv.box + 6 * (size_t)j;
  double *bl0 = nx.box + 6 * (size_t)q0, *br0 = nx.box + 6 * (size_t)(q0 + 1);
  for (int q = 0; q < 6; ++q) {
    bl0[q] = b[q];
    br0[q] = b[q];
  }
  bl0[3 + axis] = (double)s;
  br0[axis] = (double)s;
}

// Stable partition of one node's segment by one workgroup of NT threads, in
// rounds of PART_G * NT photons, through tmp: a photon's slot follows from the
// number of left photons before it.
constexpr int PART_G = 8;
template <int NT>
__device__ __forceinline__ void partition_node(uint32_t *__restrict__ perm, uint32_t *__restrict__ tmp,
                                               const uint32_t *__restrict__ tkey, uint32_t start, uint32_t M,
                                               uint32_t key, uint32_t less, uint32_t *wl) {
  constexpr uint32_t ROUND = PART_G * NT;
  constexpr int NW = NT / 64, PER = (PART_G * NW + 63) / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  uint32_t lbase = 0;  // left photons of the rounds before
  for (uint64_t r0 = 0; r0 < M; r0 += ROUND) {
    const int groups = (int)((min(M - (uint32_t)r0, ROUND) + NT - 1) / NT);
    uint32_t ph[PART_G], tk[PART_G];
    uint64_t bl[PART_G];
#pragma unroll
    for (int g = 0; g < PART_G; ++g)
      if (g < groups) {
        const uint64_t i = r0 + g * NT + threadIdx.x;
        tk[g] = i < M ? tkey[start + i] : 0xFFFFFFFFu;
        ph[g] = i < M ? perm[start + i] : 0u;
      }
#pragma unroll
    for (int g = 0; g < PART_G; ++g) {
      const uint64_t i = r0 + g * NT + threadIdx.x;
      bl[g] = g < groups ? __ballot(i < M && tk[g] < key) : 0ull;
      if (lane == 0) wl[g * NW + wave] = (uint32_t)__popcll(bl[g]);
    }
    __syncthreads();
    if (wave == 0) {  // left photons before each group of 64, and in all of them
      uint32_t c[PER], sum = 0;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int w = PER * lane + q;
        c[q] = w < PART_G * NW ? wl[w] : 0u;
        sum += c[q];
      }
      uint32_t inc = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(inc, o);
        if (lane >= o) inc += t;
      }
      uint32_t exc = inc - sum;
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int w = PER * lane + q;
        if (w < PART_G * NW) wl[w] = exc;
        exc += c[q];
      }
      if (lane == 63) wl[PART_G * NW] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int g = 0; g < PART_G; ++g)
      if (g < groups) {
        const uint64_t i = r0 + g * NT + threadIdx.x;
        const uint32_t l = lbase + wl[g * NW + wave] + (uint32_t)__popcll(bl[g] & below);
        if (i < M) {
          const uint32_t dst = tk[g] < key ? l : less + ((uint32_t)i - l);
          tmp[start + dst] = ph[g];
        }
      }
    lbase += wl[PART_G * NW];
    __syncthreads();
  }
  // every read of the segment is done (barrier above): write it in place
  for (uint64_t i = threadIdx.x; i < M; i += NT) perm[start + i] = tmp[start + i];
  __syncthreads();  // wl is free for the next node
}

// The same by one wavefront for a node of at most KD_WAVE_MAX photons: one
// round is kept in registers and written straight to its places, more go
// through buf (LDS).
__device__ __forceinline__ void partition_wave(uint32_t *__restrict__ perm, const uint32_t *__restrict__ tkey,
                                               uint32_t start, uint32_t M, uint32_t key, uint32_t less,
                                               uint32_t *buf) {
  constexpr uint32_t ROUND = PART_G * 64;
  const int lane = threadIdx.x & 63;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  const bool one = M <= ROUND;
  uint32_t lbase = 0;
  for (uint32_t r0 = 0; r0 < M; r0 += ROUND) {
    const int groups = (int)((min(M - r0, ROUND) + 63) / 64);
    uint32_t ph[PART_G], tk[PART_G];
#pragma unroll
    for (int g = 0; g < PART_G; ++g)
      if (g < groups) {
        const uint32_t i = r0 + g * 64 + lane;
        tk[g] = i < M ? tkey[start + i] : 0xFFFFFFFFu;
        ph[g] = i < M ? perm[start + i] : 0u;
      }
    // the photons are read before any is written
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int g = 0; g < PART_G; ++g)
      if (g < groups) {
        const uint32_t i = r0 + g * 64 + lane;
        const uint64_t bl = __ballot(i < M && tk[g] < key);
        const uint32_t l = lbase + (uint32_t)__popcll(bl & below);
        lbase += (uint32_t)__popcll(bl);
        if (i < M) {
          const uint32_t dst = tk[g] < key ? l : less + (i - l);
          if (one)
            perm[start + dst] = ph[g];
          else
            buf[dst] = ph[g];
        }
      }
  }
  if (one) return;
  wave_sync();
  for (uint32_t i = lane; i < M; i += 64) perm[start + i] = buf[i];
  wave_sync();  // buf is free for the next node
}

// Partitions of a level: the nodes of the split list of at most KD_WAVE_MAX
// photons, one wavefront each (a workgroup each took 250 us a level where
// hundreds of thousands of nodes hold a few dozen photons), and those of `big`
// that split (sflag: place in the split list plus one).  big_next receives the
// large children.
__global__ __launch_bounds__(KD_THREADS) void kd_partition_kernel(
    uint32_t *__restrict__ perm, const uint32_t *__restrict__ tkey, Level lv, Level nx,
    const uint32_t *__restrict__ split_list, const uint32_t *__restrict__ sel, BuildState *st, int depth,
    uint32_t *__restrict__ big_next, npg_kd_node *__restrict__ nodes) {
  __shared__ uint32_t buf[KD_THREADS / 64][KD_WAVE_MAX];
  const uint32_t nsplit = st->lv[depth].nsplit, base = st->lv[depth].nodes, wave = threadIdx.x >> 6;
  for (uint32_t k = blockIdx.x * (KD_THREADS / 64) + wave; k < nsplit; k += gridDim.x * (KD_THREADS / 64)) {
    const uint32_t j = split_list[k], M = lv.count[j];
    if (M > KD_WAVE_MAX) continue;
    const uint32_t axis = sel[3 * (size_t)j], key = sel[3 * (size_t)j + 1], less = sel[3 * (size_t)j + 2];
    if ((threadIdx.x & 63) == 0)
      put_children(lv, nx, j, k, base, axis, key, less, &st->lv[depth + 1], big_next, nodes);
    partition_wave(perm, tkey, lv.start[j], M, key, less, buf[wave]);
  }
}

__global__ __launch_bounds__(KD_BIG) void kd_partition_big_kernel(
    uint32_t *__restrict__ perm, uint32_t *__restrict__ tmp, const uint32_t *__restrict__ tkey, Level lv, Level nx,
    const uint32_t *__restrict__ big, const uint32_t *__restrict__ sflag, const uint32_t *__restrict__ sel,
    BuildState *st, int depth, uint32_t *__restrict__ big_next, npg_kd_node *__restrict__ nodes) {
  __shared__ uint32_t wl[PART_G * KD_BIG / 64 + 1];
  const uint32_t nb = st->lv[depth].nsplit ? st->lv[depth].nbig : 0, base = st->lv[depth].nodes;
  for (uint32_t bi = blockIdx.x; bi < nb; bi += gridDim.x) {
    const uint32_t j = big[bi], k1 = sflag[j];
    if (!k1) continue;
    const uint32_t axis = sel[3 * (size_t)j], key = sel[3 * (size_t)j + 1], less = sel[3 * (size_t)j + 2];
    if (threadIdx.x == 0) put_children(lv, nx, j, k1 - 1, base, axis, key, less, &st->lv[depth + 1], big_next, nodes);
    partition_node<KD_BIG>(perm, tmp, tkey, lv.start[j], lv.count[j], key, less, wl);
  }
}

__global__ __launch_bounds__(256) void kd_popc_kernel(const uint32_t *__restrict__ bits, uint64_t nw,
                                                      uint32_t *__restrict__ cnt) {
  for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < nw; w += (uint64_t)gridDim.x * blockDim.x)
    cnt[w] = (uint32_t)__popc(bits[w]);
}

// leaf k = k-th leaf start in ascending order (starts are distinct: no node
// is empty)
__global__ __launch_bounds__(256) void kd_leaves_kernel(const uint32_t *__restrict__ leaf_start,
                                                        const uint32_t *__restrict__ leaf_node,
                                                        const uint32_t *__restrict__ bits,
                                                        const uint32_t *__restrict__ rank, int last,
                                                        BuildState *st, uint32_t *__restrict__ leaf_off,
                                                        npg_kd_node *__restrict__ nodes, const uint32_t *err) {
  const uint32_t t0 = blockIdx.x * blockDim.x + threadIdx.x;
  if (t0 == 0) st->err = *err;
  if (st->over) return;
  const uint32_t L = st->lv[last].leaf_base;
  for (uint32_t q = t0; q < L; q += gridDim.x * blockDim.x) {
    const uint32_t s0 = leaf_start[q], w = s0 >> 5;
    const uint32_t k = rank[w] + (uint32_t)__popc(bits[w] & ((1u << (s0 & 31)) - 1u));
    leaf_off[k] = s0;
    nodes[leaf_node[q]].split = 0.0f;
    nodes[leaf_node[q]].info = (k << 2) | 3u;
  }
  if (t0 == 0) leaf_off[L] = st->nvalid;
}

__global__ __launch_bounds__(256) void kd_locate_kernel(GridDev g, const int32_t *__restrict__ root,
                                                        const npg_kd_node *__restrict__ nodes, uint32_t n_nodes,
                                                        const float *__restrict__ q, uint64_t n,
                                                        uint32_t *__restrict__ out, uint32_t *err) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x) {
    const float p[3] = {q[3 * i], q[3 * i + 1], q[3 * i + 2]};
    uint32_t res = KD_NONE;
    if (!finite3(p[0], p[1], p[2])) {
      raise_err(err, ERR_RANGE);
    } else {
      const int32_t r = root[vox_id(g, p[0], p[1], p[2])];
      if (r >= 0) {
        uint32_t node = (uint32_t)r;
        for (int step = 0; step < 64; ++step) {  // depth <= 16: ends long before
          if (node >= n_nodes) {
            raise_err(err, ERR_RANGE);
            break;
          }
          const npg_kd_node nd = nodes[node];
          const uint32_t a = nd.info & 3u;
          if (a == 3u) {
            res = nd.info >> 2;
            break;
          }
          const float x = p[a] == 0.0f ? 0.0f : p[a];
          node = (nd.info >> 2) + (x < nd.split ? 0u : 1u);
        }
      }
    }
    out[i] = res;
  }
}

unsigned grid_for(uint64_t n) {
  const uint64_t b = (n + 255) / 256;
  return (unsigned)(b ? (b < 65536 ? b : 65536) : 1);
}

int grid_params(npg_ctx *ctx, const npg_kdgrid_params *p, GridDev *g) {
  if (!p) return npg_fail(ctx, NPG_E_ARG, "kdgrid: null params");
  if (p->res < 1 || p->res > 1024) return npg_fail(ctx, NPG_E_ARG, "kdgrid: res %d outside [1,1024]", p->res);
  g->res = p->res;
  for (int a = 0; a < 3; ++a) {
    if (!std::isfinite(p->lo[a]) || !std::isfinite(p->hi[a]) || !(p->hi[a] > p->lo[a]))
      return npg_fail(ctx, NPG_E_ARG, "kdgrid: box axis %d is empty or not finite", a);
    const double ext = (double)p->hi[a] - (double)p->lo[a];
    g->lo[a] = p->lo[a];
    g->invr[a] = (double)p->res / ext;
    g->step[a] = ext / (double)p->res;
  }
  return NPG_OK;
}

// Workgroups of a level's kernels, which stride over the nodes there are: more
// than fit the chip at once (2048), so that nodes of unequal size even out,
// and few enough that a kernel without nodes costs 5 us, a level 15 to 24.
constexpr uint64_t KD_GRID = 8192;

// Levels queued before the host looks whether the first of them has nodes: the
// chip does not wait for the host, and a tree that ends early pays for two levels
// without nodes.  One level of 100 thousand photons, max_depth 16: 182 us; 377 with
// all levels queued at once, 305 with a wait for every level's count.  Two ahead
// leaves gaps on small builds (2000 photons, 5 levels: 10 us more), four cost 10
// to 20 us more behind the tree's end.
constexpr int KD_AHEAD = 3;

// The nodes of a level, once kd_lists_kernel of the level above has told.  A
// value from the device's memory costs a wait and a copy, an event per level
// 1.5 us on the stream; a word in the host's memory neither.  The wait ends with
// the stream's work, or its error, at the latest (asked for every few
// milliseconds: asking holds up the stream).
int level_nodes(npg_ctx *ctx, int depth, hipStream_t s, uint32_t *nodes) {
  for (uint32_t spins = 1;; ++spins) {
    *nodes = __atomic_load_n(ctx->kd_active + depth, __ATOMIC_ACQUIRE);
    if (*nodes != KD_NONE) return NPG_OK;
    __builtin_ia32_pause();
    if (spins % (1u << 18)) continue;
    const hipError_t e = hipStreamQuery(s);
    if (e == hipErrorNotReady) continue;
    NPG_HIP_CHECK(ctx, e);
    *nodes = __atomic_load_n(ctx->kd_active + depth, __ATOMIC_ACQUIRE);
    return *nodes != KD_NONE ? NPG_OK : npg_fail(ctx, NPG_E_HIP, "build_kdgrid: level %d was not counted", depth);
  }
}

}  // namespace

extern "C" int npg_mark_valid(npg_ctx *ctx, const npg_kdgrid_params *params, const float *pts_dev, uint64_t n,
                              uint8_t *valid_dev, void *stream) {
  if (!ctx) return NPG_E_ARG;
  GridDev g;
  int rc = grid_params(ctx, params, &g);
  if (rc) return rc;
  if (!valid_dev || (n && !pts_dev)) return npg_fail(ctx, NPG_E_ARG, "mark_valid: null pointer");
  rc = npg_set_device(ctx);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint64_t nv = (uint64_t)g.res * g.res * g.res;
  NPG_HIP_CHECK(ctx, hipMemsetAsync(valid_dev, 0, nv, s));
  if (n) hipLaunchKernelGGL(kd_mark_kernel, dim3(grid_for(n)), dim3(256), 0, s, g, pts_dev, n, valid_dev, ctx->err_dev);
  NPG_HIP_CHECK(ctx, hipGetLastError());
  return NPG_OK;
}

extern "C" int npg_build_kdgrid(npg_ctx *ctx, const npg_kdgrid_params *params, const float *pos_dev,
                                const float *normal_dev, uint64_t n, const uint8_t *valid_dev, uint32_t *perm_dev,
                                uint32_t *leaf_off_dev, int32_t *cell_root_dev, npg_kd_node *nodes_dev,
                                uint32_t max_leaves, uint32_t *n_leaves_out, uint32_t *n_nodes_out, void *stream) {
  if (!ctx) return NPG_E_ARG;
  GridDev g;
  int rc = grid_params(ctx, params, &g);
  if (rc) return rc;
  if (!n_leaves_out || !n_nodes_out) return npg_fail(ctx, NPG_E_ARG, "build_kdgrid: null count output");
  *n_leaves_out = 0;
  *n_nodes_out = 0;
  if (params->max_depth < 0 || params->max_depth > 16)
    return npg_fail(ctx, NPG_E_ARG, "build_kdgrid: max_depth %d outside [0,16]", params->max_depth);
  if (n > 0xffffffffull) return npg_fail(ctx, NPG_E_ARG, "build_kdgrid: n > 2^32-1");
  if (max_leaves == 0 || max_leaves >= (1u << 29))
    return npg_fail(ctx, NPG_E_ARG, "build_kdgrid: max_leaves %u outside [1, 2^29)", max_leaves);
  if (!leaf_off_dev || !cell_root_dev || !nodes_dev || (n && (!pos_dev || !perm_dev)))
    return npg_fail(ctx, NPG_E_ARG, "build_kdgrid: null pointer");
  rc = npg_set_device(ctx);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const uint64_t nvox = (uint64_t)g.res * g.res * g.res;
  const uint32_t sent = (uint32_t)nvox;
  const uint64_t m = n ? n : 1;
  const uint64_t cap = max_leaves;
  // scratch
  const uint64_t nw = (m + 31) / 32;         // words of a bitmap over the photons
  const uint64_t nch = (cap / KD_CHUNK + 1) * KD_CSTEP;  // split counters of a level
  const size_t sort_work = npg_radix_work_bytes(m);
  // keys, sorted keys and the sort's memory, and then the copies in their place
  // (six arrays of words and more against 24 bytes a photon)
  const size_t sort_bytes = 2 * npg_align(4 * m) + sort_work;
  size_t bytes = 2 * npg_align(4 * m) + sort_bytes;
  bytes += 3 * npg_align(4 * (nw + 1)) + npg_align(4 * npg_scan_tmp_words(nw));
  bytes += 2 * (3 * npg_align(4 * cap) + npg_align(48 * cap));        // two levels
  bytes += 2 * npg_align(4 * cap) + npg_align(12 * cap);              // sflag, split list, sel
  bytes += 2 * npg_align(4 * cap) + 2 * npg_align(4 * nch);           // leaves, split counters
  bytes += 2 * npg_align(4 * (m / KD_WAVE_MAX + 1)) + npg_align(sizeof(BuildState));
  // Photons are copied into voxel order for trees of more than one level (one
  // level reads each photon once anyway).  That takes one more array of words
  // (`order`): 37 bytes a photon, where every level gathering from the caller's
  // arrays takes 33.  Left out where the device has no room for it, and under a
  // budget unless the scratch is that large already: what fitted it before a
  // build, or fits it after, does not depend on the copies.
  const size_t with_order = npg_align(bytes + npg_align(4 * m), 1 << 20);
  bool voxel_order = params->max_depth >= 2 &&
                     (with_order <= ctx->scratch_bytes || (!ctx->budget && with_order < ctx->kd_no_room));
  void *scr = nullptr;
  rc = npg_scratch(ctx, voxel_order ? with_order : bytes, s, &scr);
  if (rc && voxel_order && hipGetLastError() == hipErrorOutOfMemory) {
    ctx->kd_no_room = with_order;  // not tried again by later builds
    voxel_order = false;
    rc = npg_scratch(ctx, bytes, s, &scr);
  }
  if (rc) return rc;
  Carver cv(scr);
  uint32_t *pa = cv.take<uint32_t>(m);  // partition staging
  uint32_t *tkey = cv.take<uint32_t>(m);
  uint32_t *order = voxel_order ? cv.take<uint32_t>(m) : perm_dev;  // photons by voxel
  Carver sorting(cv.take<char>(sort_bytes)), copies(sorting.base);
  uint32_t *key = sorting.take<uint32_t>(m), *ks = sorting.take<uint32_t>(m);
  void *work = sorting.take<char>(sort_work);
  // written by the first level, when the keys have been read
  float *pos_s = voxel_order ? copies.take<float>(3 * m) : nullptr;
  float *nrm_s = voxel_order && normal_dev ? copies.take<float>(3 * m) : nullptr;
  uint32_t *bits = cv.take<uint32_t>(nw + 1), *cnt = cv.take<uint32_t>(nw + 1), *rank = cv.take<uint32_t>(nw + 1);
  uint32_t *stmp = cv.take<uint32_t>(npg_scan_tmp_words(nw));
  Level lv[2];
  for (auto &l : lv) {
    l.start = cv.take<uint32_t>(cap);
    l.count = cv.take<uint32_t>(cap);
    l.id = cv.take<uint32_t>(cap);
    l.box = cv.take<double>(6 * cap);
  }
  uint32_t *sflag = cv.take<uint32_t>(cap), *slist = cv.take<uint32_t>(cap);
  uint32_t *sel = cv.take<uint32_t>(3 * cap);
  uint32_t *lstart = cv.take<uint32_t>(cap), *lnode = cv.take<uint32_t>(cap);
  uint32_t *ccnt[2];
  for (auto &c : ccnt) c = cv.take<uint32_t>(nch);
  uint32_t *big[2];  // large nodes of a level and of the next
  for (auto &b : big) b = cv.take<uint32_t>(m / KD_WAVE_MAX + 1);
  BuildState *st = cv.take<BuildState>(1);

  if (!ctx->kd_active)
    NPG_HIP_CHECK(ctx, hipHostMalloc(reinterpret_cast<void **>(&ctx->kd_active), sizeof(uint32_t) * KD_LEVELS,
                                     hipHostMallocCoherent));
  std::fill_n(ctx->kd_active, KD_LEVELS, KD_NONE);
  NPG_HIP_CHECK(ctx, hipMemsetAsync(st, 0, sizeof(BuildState), s));
  hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(nvox)), dim3(256), 0, s, cell_root_dev, nvox, -1);
  NPG_HIP_CHECK(ctx, hipGetLastError());
  int last = 0;  // levels queued: lv[last] has the totals
  if (n) {
    NPG_HIP_CHECK(ctx, hipMemsetAsync(ccnt[0], 0, 4 * nch, s));
    NPG_HIP_CHECK(ctx, hipMemsetAsync(ccnt[1], 0, 4 * nch, s));
    hipLaunchKernelGGL(kd_keys_kernel, dim3(grid_for(n)), dim3(256), 0, s, g, pos_dev, normal_dev, n, valid_dev,
                       sent, key, ctx->err_dev);
    NPG_HIP_CHECK(ctx, hipGetLastError());
    int vbits = 1;
    while (vbits < 32 && (1ull << vbits) <= (uint64_t)sent) ++vbits;
    NPG_HIP_CHECK(ctx, npg_radix_sort(key, nullptr, n, vbits, ks, order, work, s));
    hipLaunchKernelGGL(kd_seg_kernel, dim3(grid_for((n + SEG_G - 1) / SEG_G)), dim3(256), 0, s, ks, n, sent, bits, cnt,
                       voxel_order ? perm_dev : nullptr, st);
    NPG_HIP_CHECK(ctx, hipGetLastError());
    NPG_HIP_CHECK(ctx, npg_scan_u32(cnt, nw, rank, stmp, s));
    hipLaunchKernelGGL(kd_roots_kernel, dim3(grid_for(nw)), dim3(256), 0, s, g, ks, bits, rank, nw, max_leaves, lv[0],
                       cell_root_dev, st);
    NPG_HIP_CHECK(ctx, hipMemsetAsync(bits, 0, 4 * nw, s));  // from here on: the leaf starts
    // most nodes a level can have: one photon each, and twice the level above
    uint64_t bound = std::min(std::min<uint64_t>(n, cap), nvox);
    hipLaunchKernelGGL(kd_root_counts_kernel, dim3((unsigned)std::min<uint64_t>((bound + 255) / 256, 1024)), dim3(256),
                       0, s, lv[0], st, big[0]);
    NPG_HIP_CHECK(ctx, hipGetLastError());
    const uint32_t big_blocks = (uint32_t)std::min<uint64_t>(n / KD_WAVE_MAX, 512);  // 2 per CU
    for (last = 0; last <= params->max_depth; ++last) {
      const int depth = last;
      if (depth >= KD_AHEAD) {
        uint32_t nodes = 0;
        rc = level_nodes(ctx, depth - KD_AHEAD + 1, s, &nodes);
        if (rc) return rc;
        if (!nodes) break;  // nor has any level after it
      }
      Level &cur = lv[depth & 1], &nxt = lv[(depth + 1) & 1];
      uint32_t *bg = big[depth & 1], *bg_next = big[(depth + 1) & 1];
      const bool copied = voxel_order && depth > 0;  // the first level has left them
      const SelArgs sa{copied ? pos_s : pos_dev, copied ? nrm_s : normal_dev, copied ? perm_dev : order, cur,
                       depth < params->max_depth, params->split_count, params->split_var, tkey, sflag, sel,
                       ccnt[depth & 1], ctx->err_dev, depth ? nullptr : pos_s, depth ? nullptr : nrm_s};
      if (big_blocks)
        hipLaunchKernelGGL(kd_select_big_kernel, dim3(big_blocks), dim3(KD_BIG), 0, s, sa, &st->lv[depth], bg);
      hipLaunchKernelGGL(kd_select_kernel, dim3((unsigned)std::min<uint64_t>((bound + 3) / 4, KD_GRID)),
                         dim3(KD_THREADS), 0, s, sa, &st->lv[depth]);
      hipLaunchKernelGGL(kd_lists_kernel, dim3((unsigned)std::min<uint64_t>((bound + KD_CHUNK - 1) / KD_CHUNK, 256)),
                         dim3(256), 0, s, cur, st, depth, max_leaves, sflag, ccnt[depth & 1], ccnt[(depth + 1) & 1],
                         slist, lstart, lnode, bits, depth + KD_AHEAD <= params->max_depth ? ctx->kd_active : nullptr);
      if (depth < params->max_depth) {
        if (big_blocks)
          hipLaunchKernelGGL(kd_partition_big_kernel, dim3(big_blocks), dim3(KD_BIG), 0, s, perm_dev, pa, tkey, cur,
                             nxt, bg, sflag, sel, st, depth, bg_next, nodes_dev);
        hipLaunchKernelGGL(kd_partition_kernel, dim3((unsigned)std::min<uint64_t>((bound + 3) / 4, KD_GRID)),
                           dim3(KD_THREADS), 0, s, perm_dev, tkey, cur, nxt, slist, sel, st, depth, bg_next, nodes_dev);
      }
      NPG_HIP_CHECK(ctx, hipGetLastError());
      bound = std::min<uint64_t>(2 * bound, std::min<uint64_t>(n, cap));
    }
    if (voxel_order)
      hipLaunchKernelGGL(kd_final_kernel, dim3(grid_for(n)), dim3(256), 0, s, order, n, st, perm_dev);
    hipLaunchKernelGGL(kd_popc_kernel, dim3(grid_for(nw)), dim3(256), 0, s, bits, nw, cnt);
    NPG_HIP_CHECK(ctx, hipGetLastError());
    NPG_HIP_CHECK(ctx, npg_scan_u32(cnt, nw, rank, stmp, s));
  }
  hipLaunchKernelGGL(kd_leaves_kernel, dim3((unsigned)std::min<uint64_t>((std::min<uint64_t>(m, cap) + 255) / 256, 1024)),
                     dim3(256), 0, s, lstart, lnode, bits, rank, last, st, leaf_off_dev, nodes_dev, ctx->err_dev);
  NPG_HIP_CHECK(ctx, hipGetLastError());
  BuildState h;
  NPG_HIP_CHECK(ctx, hipMemcpyAsync(&h, st, sizeof h, hipMemcpyDeviceToHost, s));
  NPG_HIP_CHECK(ctx, hipStreamSynchronize(s));
  if (h.err) NPG_HIP_CHECK(ctx, hipMemsetAsync(ctx->err_dev, 0, 4, s));
  if (h.err & ERR_RANGE) return npg_fail(ctx, NPG_E_RANGE, "build_kdgrid: a position or normal is not finite");
  if (h.roots > max_leaves)
    return npg_fail(ctx, NPG_E_CAPACITY, "build_kdgrid: %u voxel roots exceed max_leaves %u", h.roots, max_leaves);
  if (h.over) return npg_fail(ctx, NPG_E_CAPACITY, "build_kdgrid: more than max_leaves %u leaves", max_leaves);
  *n_leaves_out = h.lv[last].leaf_base;
  *n_nodes_out = h.lv[last].nodes;
  return NPG_OK;
}

extern "C" int npg_locate(npg_ctx *ctx, const npg_kdgrid_params *params, const int32_t *cell_root_dev,
                          const npg_kd_node *nodes_dev, uint32_t n_nodes, const float *q_dev, uint64_t n,
                          uint32_t *leaf_dev, void *stream) {
  if (!ctx) return NPG_E_ARG;
  GridDev g;
  int rc = grid_params(ctx, params, &g);
  if (rc) return rc;
  if (n == 0) return NPG_OK;
  if (!cell_root_dev || !q_dev || !leaf_dev || (n_nodes && !nodes_dev))
    return npg_fail(ctx, NPG_E_ARG, "locate: null pointer");
  rc = npg_set_device(ctx);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  hipLaunchKernelGGL(kd_locate_kernel, dim3(grid_for(n)), dim3(256), 0, s, g, cell_root_dev, nodes_dev, n_nodes,
                     q_dev, n, leaf_dev, ctx->err_dev);
  NPG_HIP_CHECK(ctx, hipGetLastError());
  return NPG_OK;
}
