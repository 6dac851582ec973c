// 8/16-bit 3x3 convolution tiles: implicit GEMM on the matrix cores with the
// tile geometry fixed at compile time.
//
// A workgroup (4 wavefronts) computes 64 * MW output pixels x 16 * NW output
// channels.  What bounds these layers is not the matrix cores (10 to 55 % busy in
// BF16; 16 cycles of work per product) but, where little is multiplied per
// pixel, the vector instructions beside them: on full-resolution maps with 16
// channels the vector ALUs are 80 to 87 % busy in the tile that computes the first
// layer and in the one with the head; the one behind an upsampling runs at 5.3
// TB/s in BF16.  So everything that does not depend on the chunk is computed
// once per tile or at compile time:
//  - a thread's staging offsets (input patch and weights) are computed once;
//    a chunk of KC input channels only moves the buffers' base addresses;
//  - the nine taps are unrolled, and every LDS fragment read is one of three
//    registers (one per tap column) plus an immediate: the 16-byte pieces of
//    a patch pixel are stored in an order that depends on its column only;
//  - on tiles 16 pixels wide the fragment of tile row r serves the three tap
//    rows of output rows r, r - 1 and r - 2 (MW + 2 reads per tap column
//    instead of 3 MW);
//  - outputs go from the accumulators to memory: lane (lr, lg) holds four
//    consecutive channels of pixel lr, and row swaps between the lanes of two
//    channel blocks make that 16 bytes, whole pixels per instruction; the 2x2
//    means of the next level are formed from the same registers.
// BF16 network on 1501 leaves of 128x128: 3770 -> 2865 us, FP8 on 1024 of 64x64:
// 545 -> 398 us, against the tiles with run-time geometry.
//
// Every output sums its terms in the same order whatever the tile: chunks in
// order, then taps in order (for 16-channel chunks pairs of taps, one product
// covering two taps of 16 channels).
#pragma once

#include <type_traits>

#include "conv_common.h"

// One layer's launch (pointers are device pointers).
struct TileArgs {
  const void *s0 = nullptr, *s1 = nullptr;  // input, or the half-resolution input read through nearest
                                            // upsampling (s0) and the skip tensor (s1)
  int C0 = 0, C1 = 0;                       // their channels
  int H = 0, W = 0, Lc = 0;                 // output map, leaves in this launch
  int Cout = 0, nchunk = 0;
  size_t lds_budget = 0;                    // LDS for chunks staged together; 0: one at a time
  int cstage = 1;                           // chunks staged per barrier (set by the launch)
  int TR = 0, TL = 1;                       // rows per leaf and leaves of a tile
  int lw = 0, ltx = 0, ltpl = 0;            // log2 of W, of the tiles in a row and of those in a leaf
  const void *w = nullptr;                  // packed weights [chunk][tap][Cout][KC]
  const float *bias = nullptr;
  const float *head_w = nullptr;            // non-null: fuse the 1x1 head + softplus (Cout == 16)
  float head_b = 0.0f;
  const float *wsc = nullptr;               // FP8: weight scale per output channel
  float oinv = 1.0f, asc = 1.0f;            // FP8: output quantisation multiplier and unit value
  int act = ACT_RELU;                       // BF16: ACT_RELU or ACT_ELU
  const void *res = nullptr;                // BF16: residual added after the activation (layout of out)
  void *out = nullptr;
  void *pool_out = nullptr;                 // also store the 2x2 means of the stored output
  // the first layer computed into the patch: energies, totals, weights [16][9], biases
  const uint64_t *energy = nullptr;
  const double *tot = nullptr;
  const float *w0 = nullptr, *b0 = nullptr;
  float oinv0 = 1.0f;
};
enum TileIn : int { TILE_PLAIN = 0, TILE_UPCAT = 1, TILE_FIRST = 2 };
struct TileShape {
  int MW, NW, TWL;  // 64 * MW pixels, 16 * NW channels, 1 << TWL columns
};

// Launches the layer; kc: 32 or 16 input channels per chunk.
hipError_t launch_tile_bf16(TileArgs a, TileShape t, int kc, TileIn in, hipStream_t s);
hipError_t launch_tile_fp8(TileArgs a, TileShape t, int kc, TileIn in, hipStream_t s);

// Element types: a lane's fragment is 8 consecutive channels of one pixel (or
// output channel).  swz orders the 16-byte pieces of a 32-channel pixel by
// its column, and of a weight row by its index, so that the lanes of a
// fragment read fall into different LDS banks.
struct TileBF16 {
  using T = uint16_t;
  using Frag = bf16x8;
  static constexpr bool Q8 = false;
  __device__ static int swz(int p) { return (p >> 1) & 3; }
  __device__ static f32x4 mma(Frag a, Frag b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
};
struct TileFP8 {
  using T = uint8_t;
  using Frag = fp8x8;
  static constexpr bool Q8 = true;
  __device__ static int swz(int p) { return (p >> 2) & 1; }
  __device__ static f32x4 mma(Frag a, Frag b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, c, 0, 0, 0);
  }
};

template <class P, int KC, int MW, int NW, int TWL>
struct TileGeom {
  static constexpr int ESZ = (int)sizeof(typename P::T);
  static constexpr int TW = 1 << TWL, FR = 16 >> TWL;  // columns, rows of a 16-pixel fragment
  static constexpr int ROWS = 64 * MW / TW, PW = TW + 2;
  static constexpr int TLMAX = TWL == 4 ? 1 : 4;       // leaves of a tile
  static constexpr int PXB = KC * ESZ, SPP = PXB / 16; // bytes and 16-byte slots of a pixel's chunk
  static constexpr int BN = 16 * NW;
  static constexpr int NTAPW = KC == 16 ? 10 : 9;      // weight taps in LDS (the tenth zeros)
  static constexpr int WSLOTS = NTAPW * BN * SPP;
  __host__ __device__ static constexpr int npx(int TL) { return (ROWS + 2 * TL) * PW; }
  __host__ __device__ static constexpr int blocks(int slots) { return (slots + 63) / 64; }
  __host__ __device__ static constexpr int patch_bytes(int TL) { return blocks(npx(TL) * SPP) * 1024; }
  __host__ __device__ static constexpr int chunk_bytes(int TL) { return patch_bytes(TL) + blocks(WSLOTS) * 1024; }
};

constexpr uint32_t OOB = 0x80000000u;  // past the end of every buffer: loads give zeros

// e4m3_pack4_d of values that are not negative (or NaN): only the upper clamp
__device__ __forceinline__ uint32_t pack4_pos(float a, float b, float c, float d) {
  auto top = [](float x) { return x > E4M3_MAX ? E4M3_MAX : x; };
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(top(a), top(b), 0, false);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(top(c), top(d), lo, true);
}

// value of the lane N away (N a power of two below 16): N = 1 and 8 on the
// DPP path
template <int N>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
  if constexpr (N == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);
  if constexpr (N == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);
  return (uint32_t)__shfl_xor((int)v, N);
}

// 2x2 mean of four 32-bit words of stored elements, in binary64 for BF16 and
// in float for e4m3 (exact sums), rounded to storage
template <class P>
__device__ __forceinline__ uint32_t pool_word(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
  if constexpr (P::Q8) {
    const auto la = __builtin_amdgcn_cvt_pk_f32_fp8((int)a, false), lb = __builtin_amdgcn_cvt_pk_f32_fp8((int)b, false);
    const auto lc = __builtin_amdgcn_cvt_pk_f32_fp8((int)c, false), ld = __builtin_amdgcn_cvt_pk_f32_fp8((int)d, false);
    const auto ha = __builtin_amdgcn_cvt_pk_f32_fp8((int)a, true), hb = __builtin_amdgcn_cvt_pk_f32_fp8((int)b, true);
    const auto hc = __builtin_amdgcn_cvt_pk_f32_fp8((int)c, true), hd = __builtin_amdgcn_cvt_pk_f32_fp8((int)d, true);
    int o = __builtin_amdgcn_cvt_pk_fp8_f32((la[0] + lb[0] + lc[0] + ld[0]) * 0.25f,
                                            (la[1] + lb[1] + lc[1] + ld[1]) * 0.25f, 0, false);
    o = __builtin_amdgcn_cvt_pk_fp8_f32((ha[0] + hb[0] + hc[0] + hd[0]) * 0.25f,
                                        (ha[1] + hb[1] + hc[1] + hd[1]) * 0.25f, o, true);
    return (uint32_t)o;
  } else {
    auto lo = [](uint32_t v) { return (double)__uint_as_float(v << 16); };
    auto hi = [](uint32_t v) { return (double)__uint_as_float(v & 0xffff0000u); };
    const uint16_t l = from_d<uint16_t>((lo(a) + lo(b) + lo(c) + lo(d)) * 0.25);
    const uint16_t h = from_d<uint16_t>((hi(a) + hi(b) + hi(c) + hi(d)) * 0.25);
    return (uint32_t)l | ((uint32_t)h << 16);
  }
}

// stored bf16 pair plus the residual's, each sum rounded once
__device__ __forceinline__ uint32_t add_res_word(uint32_t v, uint32_t r) {
  const float l = __uint_as_float(v << 16) + __uint_as_float(r << 16);
  const float h = __uint_as_float(v & 0xffff0000u) + __uint_as_float(r & 0xffff0000u);
  return (uint32_t)f2bf(l) | ((uint32_t)f2bf(h) << 16);
}

// X: the extended form (BF16: ELU, residual); without it a plain conv + ReLU
template <class P, int KC, int MW, int NW, int TWL, TileIn IN, bool X>
__global__ __launch_bounds__(256, MW * NW >= 16 ? 2 : MW * NW >= 8 ? 3 : 4) void conv_tile_kernel(TileArgs a) {
  using G = TileGeom<P, KC, MW, NW, TWL>;
  using Frag = typename P::Frag;
  constexpr int ESZ = G::ESZ, TW = G::TW, FR = G::FR, ROWS = G::ROWS, PW = G::PW, PXB = G::PXB, SPP = G::SPP, BN = G::BN;
  constexpr bool TWO = KC == 16;  // a product covers two taps of 16 channels
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int H = a.H, W = a.W, TL = G::TLMAX == 1 ? 1 : a.TL, TR = G::TLMAX == 1 ? ROWS : a.TR;
  const int Cout = a.Cout, n0 = blockIdx.y * BN;
  // maps are powers of two on both sides, and so are the tiles in them
  const int lw = a.lw, grp = blockIdx.x >> a.ltpl, t = blockIdx.x & ((1 << a.ltpl) - 1);
  const int leaf0 = grp * TL;
  const int ty0 = (t >> a.ltx) * TR, tx0 = (t & ((1 << a.ltx) - 1)) * TW;
  const int nl = min(TL, a.Lc - leaf0);

  // leaf of patch row r (blocks of TR + 2 rows), at most three compares
  auto leaf_of = [&](int r, int rows) {
    int l = 0;
    if constexpr (G::TLMAX > 1) l = (r >= rows) + (r >= 2 * rows) + (r >= 3 * rows);
    return l;
  };

  // ---- staging offsets of this lane's 16-byte slots: slot 64 k + lane of
  // the patch (and of the weights) is written by instruction k of the chunk,
  // issued by wavefront k % 4
  constexpr int NP = (G::blocks(G::npx(G::TLMAX) * SPP) + 3) / 4, NQ = (G::blocks(G::WSLOTS) + 3) / 4;
  const int npx = G::npx(TL), np = G::blocks(npx * SPP);
  uint32_t po[IN == TILE_FIRST ? 1 : NP], pu[IN == TILE_UPCAT ? NP : 1], wo[NQ];
  if constexpr (IN != TILE_FIRST) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      // (products of 24-bit numbers: pixels of a tile's leaves < 2^22, bytes
      // of a pixel <= 2^14)
      const uint32_t s = ((uint32_t)wave * 64 + (uint32_t)lane) + 256u * i;
      __builtin_assume(s < 8192);
      const uint32_t pp = s / SPP, g = s - pp * SPP;
      const uint32_t pr = pp / PW, pc = pp - pr * PW;
      const int ls = leaf_of((int)pr, TR + 2);
      const int y = ty0 - 1 + (int)pr - ls * (TR + 2), x = tx0 - 1 + (int)pc;
      const uint32_t gs = 16u * (uint32_t)(TWO ? (int)g : (int)g ^ P::swz((int)pc));
      const bool in = (int)pp < npx && (uint32_t)y < (uint32_t)H && (uint32_t)x < (uint32_t)W;
      const uint32_t px = (uint32_t)(((ls * H + y) << lw) + x);
      if constexpr (IN == TILE_UPCAT) {
        const uint32_t pxu = (uint32_t)(((ls * (H >> 1) + (y >> 1)) << (lw - 1)) + (x >> 1));
        const uint32_t ou = __umul24(pxu, (uint32_t)(a.C0 * ESZ)) + gs, o = __umul24(px, (uint32_t)(a.C1 * ESZ)) + gs;
        pu[i] = in ? ou : OOB;
        po[i] = in ? o : OOB;
      } else {
        const uint32_t o = __umul24(px, (uint32_t)(a.C0 * ESZ)) + gs;
        po[i] = in ? o : OOB;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const uint32_t s = ((uint32_t)wave * 64 + (uint32_t)lane) + 256u * i;
    const uint32_t row = s / SPP, g = s - row * SPP, tap = row / BN, n = row - tap * BN;
    const uint32_t o = (__umul24(tap, (uint32_t)Cout) + n) * PXB + 16u * (uint32_t)(TWO ? (int)g : (int)g ^ P::swz((int)row));
    wo[i] = tap < 9 ? o : OOB;
  }
  const int wbytes = 9 * Cout * PXB;  // of one chunk
  const int cbytes = G::chunk_bytes(TL), pbytes = G::patch_bytes(TL);
  auto load_slots = [&](__amdgpu_buffer_rsrc_t rs, int at, int k, uint32_t o) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void *)(smem + at + k * (int)DMA_BLOCK), 16, o, 0, 0, 0);
  };
  auto stage_w = [&](int ch, int at) {
    const char *wb = static_cast<const char *>(a.w) + (size_t)ch * wbytes + n0 * PXB;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(wb), (short)0, wbytes - n0 * PXB, BUF_WORD3);
#pragma unroll
    for (int i = 0; i < NQ; ++i)
      if (wave + 4 * i < G::blocks(G::WSLOTS)) load_slots(rs, at + pbytes, wave + 4 * i, wo[i]);
  };
  auto stage_p = [&](int ch, int at) {
    const int c0 = ch * KC;
    const bool up = IN == TILE_UPCAT && c0 < a.C0;
    const int C = IN == TILE_UPCAT && !up ? a.C1 : a.C0, off = IN == TILE_UPCAT && !up ? c0 - a.C0 : c0;
    const int plane = (up ? (H >> 1) * (W >> 1) : H * W) * C * ESZ;
    const char *b = static_cast<const char *>(IN == TILE_UPCAT && !up ? a.s1 : a.s0) + (size_t)leaf0 * plane + off * ESZ;
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(b), (short)0, nl * plane - off * ESZ, BUF_WORD3);
    // a last chunk of 8 channels (BF16 only): its second piece is zeros
    const bool part = TWO && ESZ == 2 && C - off < KC;
#pragma unroll
    for (int i = 0; i < NP; ++i)
      if (wave + 4 * i < np) {
        uint32_t o = po[i];
        if constexpr (IN == TILE_UPCAT)
          if (up) o = pu[i];
        if (part && (lane & 1)) o = OOB;
        load_slots(rs, at, wave + 4 * i, o);
      }
  };

  // ---- fragment addresses: this wavefront's first pixel row and column
  const int wrow = wave * MW * FR;
  const int ls_w = G::TLMAX == 1 ? 0 : wrow / TR;  // the wavefront's leaf (its rows lie in one)
  const int prow = wrow + 2 * ls_w + (lr >> TWL), col = lr & (TW - 1);
  const int pbase = prow * PW + col;
  int fa[TWO ? 4 : 3], fb;
  if constexpr (!TWO) {
#pragma unroll
    for (int tx = 0; tx < 3; ++tx) {
      const int sw = P::swz(col + tx);
      fa[tx] = (pbase + tx) * PXB + (ESZ == 2 ? (lg ^ sw) * 16 : ((lg >> 1) ^ sw) * 16 + (lg & 1) * 8);
    }
    const int sw = P::swz(lr);
    fb = pbytes + lr * PXB + (ESZ == 2 ? (lg ^ sw) * 16 : ((lg >> 1) ^ sw) * 16 + (lg & 1) * 8);
  } else {
    // pairs (0,1), (2,3), (4,5) and (8,-): lanes 32..63 hold the second tap
    // (the tenth has zero weights; they read the first tap's pixel again).
    // Pair (6,7) is pair (0,1) two rows down.
    const int hi = lg >> 1, c = (lg & 1) * 8 * ESZ;
    fa[0] = (pbase + hi) * PXB + c;
    fa[1] = (pbase + (hi ? PW : 2)) * PXB + c;
    fa[2] = (pbase + PW + 1 + hi) * PXB + c;
    fa[3] = (pbase + (hi ? 0 : 2 * PW + 2)) * PXB + c;
    fb = pbytes + (hi * BN + lr) * PXB + c;
  }
  f32x4 acc[MW][NW];
#pragma unroll
  for (int mi = 0; mi < MW; ++mi)
#pragma unroll
    for (int ni = 0; ni < NW; ++ni) acc[mi][ni] = f32x4{0, 0, 0, 0};

  // the taps of the chunk staged at LDS offset `at`
  auto frag = [&](int o) { return *reinterpret_cast<const Frag *>(smem + o); };
  auto taps = [&](int at) {
    if constexpr (!TWO) {
      constexpr bool SHARE = FR == 1 && MW <= 4;
      int ra[3];
#pragma unroll
      for (int tx = 0; tx < 3; ++tx) ra[tx] = fa[tx] + at;
      const int rb = fb + at;
      Frag f[SHARE ? MW + 2 : MW][3];
      if constexpr (SHARE) {
#pragma unroll
        for (int r = 0; r < MW; ++r)
#pragma unroll
          for (int tx = 0; tx < 3; ++tx) f[r][tx] = frag(ra[tx] + r * PW * PXB);
      }
#pragma unroll
      for (int ty = 0; ty < 3; ++ty) {
        if constexpr (SHARE) {
          if (ty > 0)
#pragma unroll
            for (int tx = 0; tx < 3; ++tx) f[MW - 1 + ty][tx] = frag(ra[tx] + (MW - 1 + ty) * PW * PXB);
        }
#pragma unroll
        for (int tx = 0; tx < 3; ++tx) {
          Frag b[NW];
#pragma unroll
          for (int ni = 0; ni < NW; ++ni) b[ni] = frag(rb + ((3 * ty + tx) * BN + 16 * ni) * PXB);
#pragma unroll
          for (int mi = 0; mi < MW; ++mi) {
            Frag av;
            if constexpr (SHARE) av = f[mi + ty][tx];
            else av = frag(ra[tx] + (mi * FR + ty) * PW * PXB);
#pragma unroll
            for (int ni = 0; ni < NW; ++ni) acc[mi][ni] = P::mma(b[ni], av, acc[mi][ni]);
          }
        }
      }
    } else {
      int ra[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) ra[j] = fa[j] + at;
      const int rb = fb + at;
#pragma unroll
      for (int j = 0; j < 5; ++j) {
        Frag b[NW];
#pragma unroll
        for (int ni = 0; ni < NW; ++ni) b[ni] = frag(rb + (2 * j * BN + 16 * ni) * PXB);
#pragma unroll
        for (int mi = 0; mi < MW; ++mi) {
          const int o = mi * FR * PW * PXB;
          const Frag av = frag(j == 3 ? ra[0] + o + 2 * PW * PXB : ra[j == 4 ? 3 : j] + o);
#pragma unroll
          for (int ni = 0; ni < NW; ++ni) acc[mi][ni] = P::mma(b[ni], av, acc[mi][ni]);
        }
      }
    }
  };

  if constexpr (IN == TILE_FIRST) {
    static_assert(TWO && NW == 1, "the first layer feeds 16 channels into 16");
    stage_w(0, 0);
    // the first layer's weights read as constant memory: scalar loads,
    // although the LDS loads issued above are in flight
    using CF = const __attribute__((address_space(4))) float;
    CF *w0 = (CF *)a.w0, *b0 = (CF *)a.b0;
    // the normalised energy x = HW*E/total, rounded to float32 (zero outside
    // the map), on the patch plus one more pixel of border.  The quotient of
    // a = HW*E by the total t: q = a (1/t), corrected twice by fma(r, 1/t, q)
    // with the exact remainder r = a - q t, which gives the correctly rounded
    // quotient (Markstein 1990) in six operations instead of a division per
    // element.
    constexpr int EW = TW + 4;
    const int ERL = TR + 4, ne = (ROWS + 4 * TL) * EW;
    float *xt = reinterpret_cast<float *>(smem + cbytes);
    const double hw = (double)H * (double)W;
    double tl = 0.0, inv = 0.0;
    if constexpr (G::TLMAX == 1) {
      tl = a.tot[leaf0];
      inv = tl > 0.0 ? 1.0 / tl : 0.0;
    }
    for (int i = tid; i < ne; i += 256) {
      const int er = i / EW, ex = i - er * EW;
      const int ls = leaf_of(er, ERL);
      const int y = ty0 - 2 + er - ls * ERL, x = tx0 - 2 + ex;
      float v = 0.0f;
      if (ls < nl && (uint32_t)y < (uint32_t)H && (uint32_t)x < (uint32_t)W) {
        if constexpr (G::TLMAX > 1) {
          tl = a.tot[leaf0 + ls];
          inv = tl > 0.0 ? 1.0 / tl : 0.0;
        }
        const double e = hw * (double)(a.energy + (size_t)leaf0 * H * W)[(uint32_t)(((ls * H + y) << lw) + x)];
        double q = e * inv;
        q = fma(fma(-q, tl, e), inv, q);
        q = fma(fma(-q, tl, e), inv, q);
        v = (float)q;
      }
      xt[i] = v;
    }
    __syncthreads();
    // the biases in vector registers (a product takes one scalar operand,
    // its weight)
    float bv[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) {
      bv[c] = b0[c];
      asm("" : "+v"(bv[c]));
    }
    for (int pp = tid; pp < npx; pp += 256) {
      const int pr = pp / PW, pc = pp - pr * PW;
      const int ls = leaf_of(pr, TR + 2);
      const int y = ty0 - 1 + pr - ls * (TR + 2), x = tx0 - 1 + pc;
      uint32_t o[4 * ESZ];
#pragma unroll
      for (int k = 0; k < 4 * ESZ; ++k) o[k] = 0;
      if (ls < nl && (uint32_t)y < (uint32_t)H && (uint32_t)x < (uint32_t)W) {
        const float *xp = xt + (pr + 2 * ls) * EW + pc;
        float xv[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) xv[k] = xp[(k / 3) * EW + k % 3];
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
          float r[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = 4 * c4 + q;
            float s = bv[c];
#pragma unroll
            for (int k = 0; k < 9; ++k) s = fmaf(w0[c * 9 + k], xv[k], s);
            s = fmaxf(s, 0.0f);
            r[q] = P::Q8 ? s * a.oinv0 : s;
          }
          if constexpr (P::Q8) {
            o[c4] = pack4_pos(r[0], r[1], r[2], r[3]);
          } else {
            o[2 * c4] = (uint32_t)f2bf(r[0]) | ((uint32_t)f2bf(r[1]) << 16);
            o[2 * c4 + 1] = (uint32_t)f2bf(r[2]) | ((uint32_t)f2bf(r[3]) << 16);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < ESZ; ++k)
        *reinterpret_cast<uint4 *>(smem + pp * PXB + 16 * k) = make_uint4(o[4 * k], o[4 * k + 1], o[4 * k + 2], o[4 * k + 3]);
    }
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    taps(0);
  } else {
    for (int ch = 0; ch < a.nchunk; ch += a.cstage) {
      const int nc = min(a.cstage, a.nchunk - ch);
      if (ch) __syncthreads();  // the taps before have read their chunks
      for (int c = 0; c < nc; ++c) {
        stage_w(ch + c, c * cbytes);
        stage_p(ch + c, c * cbytes);
      }
      // the LDS loads of this wavefront have landed; the barrier covers the others'
      __builtin_amdgcn_s_waitcnt(0);
      __syncthreads();
      for (int c = 0; c < nc; ++c) taps(c * cbytes);
    }
  }

  // ---- epilogue
  if (G::TLMAX > 1 && ls_w >= nl) return;  // rows past the last leaf
  // output pixel (mi, lr): row y0 + mi FR, relative to the first map of the tile
  const int y0 = ls_w * H + ty0 + wrow - ls_w * TR + (lr >> TWL);
  const size_t map0 = (size_t)leaf0 * H * W;
  if (NW == 1 && !X && IN != TILE_FIRST && a.head_w) {
    float bn[4], hw[4], ws[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bn[r] = a.bias[4 * lg + r];
      hw[r] = a.head_w[4 * lg + r];
      ws[r] = 1.0f;
      if constexpr (P::Q8) ws[r] = a.wsc[4 * lg + r];
    }
    float mine[(MW + 3) / 4] = {};
#pragma unroll
    for (int mi = 0; mi < MW; ++mi) {
      float v = 0.0f;
      // the values the unfused path would store (type T) feed the head
      if constexpr (P::Q8) {
        float q[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v0 = acc[mi][0][r] * ws[r] + bn[r];
          q[r] = fmaxf(v0, 0.0f) * a.oinv;
        }
        const int pk = (int)pack4_pos(q[0], q[1], q[2], q[3]);
        const auto d01 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, false), d23 = __builtin_amdgcn_cvt_pk_f32_fp8(pk, true);
        const float dq[4] = {d01[0], d01[1], d23[0], d23[1]};
#pragma unroll
        for (int r = 0; r < 4; ++r) v += (dq[r] * a.asc) * hw[r];
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v0 = acc[mi][0][r] + bn[r];
          v += bf2f(f2bf(fmaxf(v0, 0.0f))) * hw[r];
        }
      }
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lg == (mi & 3)) mine[mi >> 2] = v;
    }
    float *out = static_cast<float *>(a.out) + map0;
#pragma unroll
    for (int h = 0; h < (MW + 3) / 4; ++h)
      if (4 * h + lg < MW)
        out[(uint32_t)(((y0 + (4 * h + lg) * FR) << lw) + tx0 + col)] = softplus_f(mine[h] + a.head_b);
    return;
  }
  // packed outputs: NWD words (16 bytes where the tile has the channels) of
  // NPC pieces per pixel, piece p from channel chb + 32 p on
  constexpr int NPC = ESZ == 2 && NW == 4 ? 2 : 1, NWD = NW * ESZ / NPC;
  uint32_t v[MW][NPC][NWD];
  const int chb = NW == 1 ? 4 * lg : ESZ == 1 && NW == 4 ? 16 * lg : (lg & 1) * 16 + (lg >> 1) * 8;
  {
    float bn[NW][4], ws[NW][4];
#pragma unroll
    for (int ni = 0; ni < NW; ++ni)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        bn[ni][r] = a.bias[n0 + 16 * ni + 4 * lg + r];
        ws[ni][r] = 1.0f;
        if constexpr (P::Q8) ws[ni][r] = a.wsc[n0 + 16 * ni + 4 * lg + r];
      }
#pragma unroll
    for (int mi = 0; mi < MW; ++mi) {
      uint32_t pk[NW][ESZ];
#pragma unroll
      for (int ni = 0; ni < NW; ++ni) {
        float q[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if constexpr (P::Q8) {
            const float x = acc[mi][ni][r] * ws[ni][r] + bn[ni][r];
            q[r] = fmaxf(x, 0.0f) * a.oinv;
          } else {
            const float x = acc[mi][ni][r] + bn[ni][r];
            q[r] = X ? act_fn(x, a.act) : fmaxf(x, 0.0f);
          }
        }
        if constexpr (P::Q8) {
          pk[ni][0] = pack4_pos(q[0], q[1], q[2], q[3]);
        } else {
          pk[ni][0] = (uint32_t)f2bf(q[0]) | ((uint32_t)f2bf(q[1]) << 16);
          pk[ni][1] = (uint32_t)f2bf(q[2]) | ((uint32_t)f2bf(q[3]) << 16);
        }
      }
      // swapping the odd lane rows (16 lanes) of block ni with the even rows
      // of block ni + 1 leaves eight consecutive channels in a lane's pair
      if constexpr (NW >= 2) {
#pragma unroll
        for (int ni = 0; ni < NW; ni += 2)
#pragma unroll
          for (int k = 0; k < ESZ; ++k) {
            const auto r = __builtin_amdgcn_permlane16_swap(pk[ni][k], pk[ni + 1][k], false, false);
            pk[ni][k] = r[0];
            pk[ni + 1][k] = r[1];
          }
      }
      if constexpr (ESZ == 1 && NW == 4) {  // and swapping halves sixteen
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          const auto r = __builtin_amdgcn_permlane32_swap(pk[k][0], pk[k + 2][0], false, false);
          pk[k][0] = r[0];
          pk[k + 2][0] = r[1];
        }
      }
#pragma unroll
      for (int p = 0; p < NPC; ++p)
#pragma unroll
        for (int k = 0; k < NWD; ++k) v[mi][p][k] = pk[p * (NW / NPC) + k / ESZ][k % ESZ];
    }
  }
  char *out = static_cast<char *>(a.out) + map0 * Cout * ESZ;
  const char *res = X && a.res ? static_cast<const char *>(a.res) + map0 * Cout * ESZ : nullptr;
  using Piece = uint32_t __attribute__((ext_vector_type(NWD == 1 ? 2 : NWD)));  // (NWD == 1: see put)
  auto put = [&](char *p, const uint32_t *x) {
    if constexpr (NWD == 1) {
      *reinterpret_cast<uint32_t *>(p) = x[0];
    } else {
      Piece q;
#pragma unroll
      for (int k = 0; k < NWD; ++k) q[k] = x[k];
      *reinterpret_cast<Piece *>(p) = q;
    }
  };
#pragma unroll
  for (int mi = 0; mi < MW; ++mi) {
    const uint32_t o = __umul24((uint32_t)(((y0 + mi * FR) << lw) + tx0 + col), (uint32_t)(Cout * ESZ)) + (uint32_t)(n0 + chb) * ESZ;
#pragma unroll
    for (int p = 0; p < NPC; ++p) {
      if constexpr (X) {
        if (res) {
          const Piece r = *reinterpret_cast<const Piece *>(res + o + 64 * p);
#pragma unroll
          for (int k = 0; k < NWD; ++k) v[mi][p][k] = add_res_word(v[mi][p][k], r[k]);
        }
      }
      put(out + o + 32 * ESZ * p, v[mi][p]);
    }
  }
  if (a.pool_out && (TWL != 4 || MW > 1)) {
    // the 2x2 means, stored [leaf][H/2][W/2][Cout]: the neighbouring column
    // is the lane next door, the row below another lane (fragments of
    // several rows) or this lane's next fragment.  The two lanes of a window
    // form half of its words each: the even lane the first half.
    char *po2 = static_cast<char *>(a.pool_out) + (size_t)leaf0 * (H >> 1) * (W >> 1) * Cout * ESZ;
    constexpr int ST = FR == 1 ? 2 : 1, NH = NWD == 1 ? 1 : NWD / 2;
    const bool odd = lr & 1;
#pragma unroll
    for (int mi = 0; mi < MW; mi += ST)
#pragma unroll
      for (int p = 0; p < NPC; ++p) {
        uint32_t m[NH];
#pragma unroll
        for (int k = 0; k < NH; ++k) {
          auto row_below = [&](uint32_t x, int w) { return FR == 1 ? v[mi + ST - 1][p][w] : xor_lane<FR == 2 ? 8 : 4>(x); };
          const uint32_t x0 = v[mi][p][k], z0 = row_below(x0, k);
          if constexpr (NWD == 1) {
            m[k] = pool_word<P>(x0, xor_lane<1>(x0), z0, xor_lane<1>(z0));
          } else {
            const uint32_t x1 = v[mi][p][k + NH], z1 = row_below(x1, k + NH);
            const uint32_t xo = odd ? x1 : x0, zo = odd ? z1 : z0;  // this lane's half of the words ...
            const uint32_t xn = xor_lane<1>(odd ? x0 : x1), zn = xor_lane<1>(odd ? z0 : z1);  // ... from next door
            m[k] = pool_word<P>(odd ? xn : xo, odd ? xo : xn, odd ? zn : zo, odd ? zo : zn);
          }
        }
        const int y = y0 + mi * FR;  // even in the lanes that store
        if ((NWD > 1 || !odd) && (FR == 1 || !((lr >> TWL) & 1))) {
          char *d = po2 + __umul24((uint32_t)(((y >> 1) << (lw - 1)) + ((tx0 + col) >> 1)), (uint32_t)(Cout * ESZ)) +
                    (uint32_t)(n0 + chb) * ESZ + 32 * ESZ * p + (odd ? 4 * NH : 0);
          if constexpr (NH == 1) {
            *reinterpret_cast<uint32_t *>(d) = m[0];
          } else {
            *reinterpret_cast<uint2 *>(d) = make_uint2(m[0], m[1]);
          }
        }
      }
  }
}

template <class P, int KC, int MW, int NW, int TWL, TileIn IN, bool X>
hipError_t launch_tile_kx(TileArgs &a, hipStream_t s) {
  using G = TileGeom<P, KC, MW, NW, TWL>;
  a.TR = G::ROWS < a.H ? G::ROWS : a.H;
  a.TL = G::ROWS / a.TR;
  // what the kernel assumes: whole tiles, a wavefront's rows in one leaf
  if (a.W % G::TW || a.H % a.TR || a.TL > G::TLMAX || MW * G::FR > a.TR || a.Cout % G::BN)
    return hipErrorInvalidValue;
  if (a.pool_out && TWL == 4 && MW == 1) return hipErrorInvalidValue;
  if ((a.H & (a.H - 1)) || (a.W & (a.W - 1)) || a.H > 1024 || a.W > 1024) return hipErrorInvalidValue;
  a.lw = __builtin_ctz(a.W);
  a.ltx = __builtin_ctz(a.W / G::TW);
  a.ltpl = a.ltx + __builtin_ctz(a.H / a.TR);
  const size_t tiles = (size_t)((a.Lc + a.TL - 1) / a.TL) << a.ltpl;
  if (tiles > 0x7fffffffu) return hipErrorInvalidValue;
  const size_t cb = (size_t)G::chunk_bytes(a.TL);
  size_t lds = cb;
  if (IN == TILE_FIRST) lds += sizeof(float) * (G::ROWS + 4 * a.TL) * (G::TW + 4);
  else lds *= a.cstage = (int)std::max<size_t>(1, std::min<size_t>(a.nchunk, a.lds_budget / cb));
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  static std::atomic<uint64_t> attr{0};
  if (npg_first_on_device(attr)) {
    hipError_t e = hipFuncSetAttribute((const void *)conv_tile_kernel<P, KC, MW, NW, TWL, IN, X>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((conv_tile_kernel<P, KC, MW, NW, TWL, IN, X>), dim3((unsigned)tiles, (unsigned)(a.Cout / G::BN)),
                     dim3(256), lds, s, a);
  return hipGetLastError();
}

template <class P, int KC, int MW, int NW, int TWL, TileIn IN>
hipError_t launch_tile_k(TileArgs &a, hipStream_t s) {
  if (a.act != ACT_RELU || a.res) {
    if constexpr (!P::Q8 && IN != TILE_FIRST) return a.head_w ? hipErrorInvalidValue : launch_tile_kx<P, KC, MW, NW, TWL, IN, true>(a, s);
    return hipErrorInvalidValue;
  }
  return launch_tile_kx<P, KC, MW, NW, TWL, IN, false>(a, s);
}

template <class P, int KC, TileIn IN>
hipError_t launch_tile(TileArgs &a, const TileShape &t, hipStream_t s) {
  switch (t.TWL * 100 + t.MW * 10 + t.NW) {
    case 211: return launch_tile_k<P, KC, 1, 1, 2, IN>(a, s);
    case 311: return launch_tile_k<P, KC, 1, 1, 3, IN>(a, s);
    case 321: return launch_tile_k<P, KC, 2, 1, 3, IN>(a, s);
    case 341: return launch_tile_k<P, KC, 4, 1, 3, IN>(a, s);
    case 411: return launch_tile_k<P, KC, 1, 1, 4, IN>(a, s);
    case 421: return launch_tile_k<P, KC, 2, 1, 4, IN>(a, s);
    case 441: return launch_tile_k<P, KC, 4, 1, 4, IN>(a, s);
    case 481: return launch_tile_k<P, KC, 8, 1, 4, IN>(a, s);
  }
  if constexpr (IN != TILE_FIRST) {
    switch (t.TWL * 100 + t.MW * 10 + t.NW) {
      case 212: return launch_tile_k<P, KC, 1, 2, 2, IN>(a, s);
      case 214: return launch_tile_k<P, KC, 1, 4, 2, IN>(a, s);
      case 312: return launch_tile_k<P, KC, 1, 2, 3, IN>(a, s);
      case 314: return launch_tile_k<P, KC, 1, 4, 3, IN>(a, s);
      case 322: return launch_tile_k<P, KC, 2, 2, 3, IN>(a, s);
      case 324: return launch_tile_k<P, KC, 2, 4, 3, IN>(a, s);
      case 342: return launch_tile_k<P, KC, 4, 2, 3, IN>(a, s);
      case 344: return launch_tile_k<P, KC, 4, 4, 3, IN>(a, s);
      case 412: return launch_tile_k<P, KC, 1, 2, 4, IN>(a, s);
      case 414: return launch_tile_k<P, KC, 1, 4, 4, IN>(a, s);
      case 422: return launch_tile_k<P, KC, 2, 2, 4, IN>(a, s);
      case 424: return launch_tile_k<P, KC, 2, 4, 4, IN>(a, s);
      case 442: return launch_tile_k<P, KC, 4, 2, 4, IN>(a, s);
      case 444: return launch_tile_k<P, KC, 4, 4, 4, IN>(a, s);
      case 482: return launch_tile_k<P, KC, 8, 2, 4, IN>(a, s);
    }
  }
  return hipErrorInvalidValue;
}

template <class P>
hipError_t launch_tile_any(TileArgs &a, const TileShape &t, int kc, TileIn in, hipStream_t s) {
  if (in == TILE_FIRST) return kc == 16 ? launch_tile<P, 16, TILE_FIRST>(a, t, s) : hipErrorInvalidValue;
  if (in == TILE_UPCAT) return kc == 16 ? launch_tile<P, 16, TILE_UPCAT>(a, t, s) : launch_tile<P, 32, TILE_UPCAT>(a, t, s);
  return kc == 16 ? launch_tile<P, 16, TILE_PLAIN>(a, t, s) : launch_tile<P, 32, TILE_PLAIN>(a, t, s);
}
