// General WBMM kernels for gfx950: any map, any w_h x w_w window (sides up to
// 16), coefficients from the table or from a materialised matrix, float32 and
// 16-bit.  They serve what the fixed-layout kernels of wbmm_kernels.h do not:
// maps the windows do not tile, odd image widths, rectangular windows, cached
// matrices, and float32.
//
// Shape of the work
// -----------------
// Window positions are row padded (RP = 8 or 16 columns per window row), as in
// wbmm_kernels.h.  One 8-wave workgroup runs consecutive stages of one
// channel; a stage is CW windows whose rows number 512, so that each thread
// moves exactly one window row: thread t moves row t / CW of window t % CW,
// and the lanes of a wave touch consecutive pieces of one image row.  Rows are
// read with unaligned 16-byte loads and masked (columns past the window or the
// image are zero), so there is no per-element path for odd widths or cut
// windows, except for the rows within 16 elements of the tensor's end.
//
// The coefficients (M^T fragments) are read once per workgroup into registers:
// wave T holds those of output positions 32 T .. 32 T + 31 for every K step,
// and the stages stream past them.
#pragma once

#include <type_traits>

#include "wbmm_kernels.h"

namespace wbmm {

constexpr int kGenWaves = 8;
constexpr int kGenThreads = 64 * kGenWaves;

// Where the coefficients come from: the table (forward, or read back to
// front for the input gradient), or a matrix [C, d, d] (forward, or
// transposed).
enum GenSrc { kSrcTable = 0, kSrcTableRev = 1, kSrcMat = 2, kSrcMatT = 3 };

// Division of n < 2^31 by a constant d >= 1: (n m) >> sh with
// sh = 31 + ceil(log2 d) and m = floor(2^sh / d) + 1, exact since
// m d - 2^sh is at most d <= 2^(sh - 31).
struct FastDiv {
  uint32_t m;
  int sh;
};
__host__ inline FastDiv fast_div(uint32_t d) {
  int l = 0;
  while (((uint64_t)1 << l) < d) ++l;
  return FastDiv{(uint32_t)((((uint64_t)1 << (31 + l)) / d) + 1), 31 + l};
}
__device__ __attribute__((always_inline)) inline uint32_t div_by(uint32_t n, FastDiv f) {
  return (uint32_t)(((uint64_t)n * f.m) >> f.sh);
}

// Workgroups of a launch, C tiles_per_ch of them: a grid dimension holds fewer
// than 2^32 threads, so more than 2^22 workgroups go on in the second one.
constexpr int64_t kGenGridX = (int64_t)1 << 22;
__host__ inline dim3 gen_grid(int64_t wgs) {
  if (wgs <= kGenGridX) return dim3((unsigned)wgs);
  return dim3((unsigned)kGenGridX, (unsigned)((wgs + kGenGridX - 1) / kGenGridX));
}
__device__ __attribute__((always_inline)) inline uint32_t gen_block() {
  return blockIdx.y * gridDim.x + die_major(blockIdx.x, gridDim.x);
}

struct GenArgs {
  int64_t C, H, W;
  int64_t hw, chw;   // H W, C H W
  int64_t numel;     // elements of one [B,C,H,W] tensor
  uint32_t NW, NHW;  // windows per map row, per image
  FastDiv dnw, dnhw;
  uint32_t N;        // windows per channel (below 2^31)
  int wh, ww;
  int stages;        // per channel
  int spw;           // stages per workgroup
  int tiles_per_ch;  // workgroups per channel
  int src;           // GenSrc
  int lgg;           // log2 of the windows of a row that neighbouring lanes take
};

__host__ __device__ constexpr int pow2_up(int v) { return v <= 1 ? 1 : v <= 2 ? 2 : v <= 4 ? 4 : v <= 8 ? 8 : 16; }

// S: K steps of 32 padded positions (rows_up(wh) = 32 S / RP).
template <class Tag, int RP, int S>
struct GenCfg {
  static constexpr int KP = 32 * S;                  // padded positions
  static constexpr int KR = KP / RP;                 // padded rows
  static constexpr int KRP = 32 * pow2_up(S) / RP;   // row slots per window
  static constexpr int CW = kGenThreads / KRP;       // windows per stage
  static constexpr int SUBS = CW / 16;
  static constexpr int NT = 2 * S;                   // 16-wide position tiles
  static constexpr int NPL = Tag::W16 ? 1 : 3;       // 16-bit planes of a value
  static constexpr int LDSW = KP + 8;                // pitch of a plane (elements)
  static constexpr int PLANE = CW * LDSW * 2;        // bytes
  static constexpr int XB = NPL * PLANE;             // one stage of one tensor
  static constexpr int OP = Tag::W16 ? KP + 8 : KP + 4;  // result pitch (elements)
  static constexpr int OB = CW * OP * Tag::ES;
  static constexpr int NG = kGenWaves / S;           // wave groups sharing a stage's sub-tiles
  static constexpr int SPW = cdiv(SUBS, NG);         // sub-tiles of a wave per stage
  static_assert(SUBS % NG == 0, "whole sub-tiles per wave");
  static constexpr int ND = RP * Tag::ES / 4;        // dwords of a padded row
  // Toeplitz blocks of the table: dh = -(KR - 1) .. KR - 1
  static constexpr int NBLK = 2 * KR - 1;
  static constexpr int TBB = NBLK * RP * RP * 2;     // bytes of one plane
  static constexpr int CKB = 32 * LDSW * 2;          // a chunk of 32 matrix rows
  static_assert(NPL * TBB <= XB, "blocks within one stage buffer");
};

// Window (of the stage) and row that a thread moves: neighbouring lanes take
// the same row of 2^lgg neighbouring windows, then the next rows of the same
// windows, so that a wave's rows lie together in memory: with few windows per
// map row (2^lgg is the largest power of two not above that), the rows of one
// image follow each other.
template <class G>
__device__ __attribute__((always_inline)) inline int gen_slot_window(const GenArgs &a, int t) {
  return (t / G::KRP >> a.lgg << a.lgg) | (t & ((1 << a.lgg) - 1));
}
template <class G>
__device__ __attribute__((always_inline)) inline int gen_slot_row(const GenArgs &a, int t) {
  return (t >> a.lgg) & (G::KRP - 1);
}

struct GRow {
  int64_t eoff;  // first element of the row
  int cols;      // its elements inside window and image, 0: none
};

typedef uint32_t u32x4u __attribute__((ext_vector_type(4))) __attribute__((aligned(2)));
typedef uint32_t u32x2u __attribute__((ext_vector_type(2))) __attribute__((aligned(2)));
typedef uint32_t u32u __attribute__((aligned(2)));

// Row hi of window n of channel c.
__device__ __attribute__((always_inline)) inline GRow gen_row(const GenArgs &a, int64_t c, uint32_t n, int hi) {
  GRow r;
  r.eoff = 0;
  r.cols = 0;
  if (n >= a.N || hi >= a.wh) return r;
  const uint32_t b = div_by(n, a.dnhw), rem = n - b * a.NHW;
  const uint32_t wy = div_by(rem, a.dnw), wx = rem - wy * a.NW;
  const int h = (int)wy * a.wh + hi, x0 = (int)wx * a.ww;
  const int cw = (int)a.W - x0;
  r.cols = h < (int)a.H ? (cw < a.ww ? cw : a.ww) : 0;
  r.eoff = (int64_t)b * a.chw + c * a.hw + (int64_t)h * a.W + x0;
  return r;
}

// Sixteen zero elements for the rows that do not exist.
__device__ const uint32_t gen_zero[16] = {};

// RP elements from the row's start (the ones past its end belong to the
// tensor; gen_mask clears them).  Every lane loads, with no branch around the
// loads, so that a wait for them counts exactly and leaves later loads in
// flight: rows that do not exist load zeros, rows within RP elements of the
// tensor's end its last RP elements (gen_tail moves them down).  The tensor
// holds at least RP elements.
template <class Tag, int RP>
__device__ __attribute__((always_inline)) inline void gen_load(int64_t numel, const typename Tag::S *x, const GRow &r,
                                                               uint32_t (&d)[RP * Tag::ES / 4]) {
  typedef const __attribute__((address_space(1))) u32x4u *GP;
  const int64_t last = numel - RP;
  const int64_t e = r.eoff < last ? r.eoff : last;
  const uint64_t p = r.cols > 0 ? reinterpret_cast<uint64_t>(x + e) : reinterpret_cast<uint64_t>(gen_zero);
#pragma unroll
  for (int i = 0; i < RP * Tag::ES / 4; i += 4) {
    const u32x4u u = *reinterpret_cast<GP>(p + 4 * i);
    d[i] = u.x; d[i + 1] = u.y; d[i + 2] = u.z; d[i + 3] = u.w;
  }
}

// A row within RP elements of the tensor's end: its elements moved down to
// the row's start.
template <class Tag, int RP>
__device__ __attribute__((always_inline)) inline void gen_tail(int64_t numel, const GRow &r,
                                                               uint32_t (&d)[RP * Tag::ES / 4]) {
  constexpr int ND = RP * Tag::ES / 4;
  const int64_t over = r.eoff + RP - numel;
  if (r.cols > 0 && over > 0) {
#pragma unroll 1
    for (int k = (int)over; k > 0; --k) {
#pragma unroll
      for (int i = 0; i < ND; ++i) {
        const uint32_t up = i + 1 < ND ? d[i + 1] : 0u;
        d[i] = Tag::W16 ? __builtin_amdgcn_alignbit(up, d[i], 16) : up;
      }
    }
  }
}

// Zero past the row's columns (apart from the loads, so that the wait for
// them comes where the row is used): masks for 0 .. RP columns in LDS, since
// comparing every column costs five instructions a dword.
template <class Tag, int RP>
__host__ __device__ constexpr int gen_mask_bytes() { return (RP + 1) * RP * Tag::ES; }

template <class Tag, int RP>
__device__ __attribute__((always_inline)) inline void gen_mask_table(uint32_t *tab, int tid) {
  constexpr int ND = RP * Tag::ES / 4;
  static_assert((RP + 1) * ND <= kGenThreads, "one entry per thread");
  const int cols = tid / ND, i = tid % ND;
  if (cols <= RP) {
    if constexpr (Tag::W16) tab[tid] = cols > 2 * i + 1 ? ~0u : cols > 2 * i ? 0xffffu : 0u;
    else tab[tid] = cols > i ? ~0u : 0u;
  }
}

template <class Tag, int RP>
__device__ __attribute__((always_inline)) inline void gen_mask(const uint32_t *tab, int cols,
                                                               uint32_t (&d)[RP * Tag::ES / 4]) {
  constexpr int ND = RP * Tag::ES / 4;
#pragma unroll
  for (int i = 0; i < ND; i += 4) {
    const uint4 m = *reinterpret_cast<const uint4 *>(tab + cols * ND + i);
    d[i] &= m.x; d[i + 1] &= m.y; d[i + 2] &= m.z; d[i + 3] &= m.w;
  }
}

// The first cols elements of a padded row -> y (cols <= RP; unaligned).
template <class Tag, int RP>
__device__ __attribute__((always_inline)) inline void gen_store(typename Tag::S *y, const GRow &r,
                                                                uint32_t (&d)[RP * Tag::ES / 4]) {
  constexpr int ND = RP * Tag::ES / 4;
  char *p = reinterpret_cast<char *>(y + r.eoff);
  const int nb = r.cols * Tag::ES;  // bytes
  // whole 16-byte pieces first, then the rest by the bits of its length
  const int full = nb >> 4;
  uint32_t t[4] = {0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < ND / 4; ++i) {
    if (i < full)
      *reinterpret_cast<u32x4u *>(p + 16 * i) = u32x4u{d[4 * i], d[4 * i + 1], d[4 * i + 2], d[4 * i + 3]};
    if (i == full) {
#pragma unroll
      for (int k = 0; k < 4; ++k) t[k] = d[4 * i + k];
    }
  }
  p += 16 * full;
  if (nb & 8) {
    *reinterpret_cast<u32x2u *>(p) = u32x2u{t[0], t[1]};
    p += 8;
    t[0] = t[2];
    t[1] = t[3];
  }
  if (nb & 4) {
    *reinterpret_cast<u32u *>(p) = t[0];
    p += 4;
    t[0] = t[1];
  }
  if constexpr (Tag::ES == 2) {
    if (nb & 2) *reinterpret_cast<u16 *>(p) = (u16)(t[0] & 0xffffu);
  }
}

// float32 on the bf16 matrix cores
// --------------------------------
// A float32 value is the exact sum of three bf16 values, hi + mid + lo, each
// the nearest bf16 to what is left (8 + 8 + 8 significant bits).  A product of
// two values is taken as the six partial products of weight 2^-16 and above,
//   hi hi + (hi mid + mid hi) + (mid mid + hi lo + lo hi),
// every one exact in float32, the first summed in one accumulator and the
// others in a second one: what is left out is below 2^-24 of the product.  The
// bf16 rate is sixteen times the float32 matrix rate, six products cost 3/8 of
// a float32 one.  Ranges where a part would overflow or vanish (and
// infinities and NaN) take float32 products instead: a row is "far" when one of
// its magnitudes is at least 2^60, or not zero and below 2^-96 (from 2^-103 on
// every bit of the lowest part lies above bf16's smallest normal value; a tiny
// value beside ordinary ones can decide an output alone).  What that
// costs, every row far, us (ordinary values; the float32 row kernels): forward
// w = 14 B128 C256 56x56 4390 -> 750 (280; 800), w = 7 B64 C96 56x56 174 -> 62 (38;
// 45), both gradients w = 14 B128 C192 28x28 2240 -> 325 (156; 273), w = 7 434 ->
// 136 (82; 144), a cached matrix w = 14 B64 C192 28x28 713 -> 238 (74; 406).
// Before, every product recomputed its window's address and read both values
// from global memory; now four values of a row serve every output tile of a
// wave (forward), or a stage's rows lie in LDS as float32 (gradient).
constexpr uint32_t kFarHi = (127u + 60u) << 23, kFarLo = (127u - 96u) << 23;
constexpr uint32_t kFarLoCoef = (127u - 60u) << 23;

// Magnitudes (float bits without the sign, doubled) of the values seen: the
// largest, and the smallest but zero, less one (an instruction each a value).
struct FarRange {
  uint32_t mx = 0, mn = ~0u;
  __device__ __attribute__((always_inline)) void add(uint32_t bits) {
    const uint32_t m = bits << 1, n = m - 1;
    mx = m > mx ? m : mx;
    mn = n < mn ? n : mn;
  }
  __device__ __attribute__((always_inline)) bool far() const { return mx >= 2 * kFarHi || mn < 2 * kFarLo - 1; }
};
// The same with the largest as a float, a third fewer instructions, for the
// products Y = X M: NaN may be left out, which the parts carry to the same
// outputs.
struct FarRangeFwd {
  float mx = 0.f;
  uint32_t mn = ~0u;
  __device__ __attribute__((always_inline)) void add(uint32_t a, uint32_t b) {
    asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(mx) : "v"(a), "v"(b));
    const uint32_t m = (a << 1) - 1, n = (b << 1) - 1;
    mn = m < mn ? m : mn;
    mn = n < mn ? n : mn;
  }
  __device__ __attribute__((always_inline)) bool far() const {
    return !(mx < __builtin_bit_cast(float, kFarHi)) || mn < 2 * kFarLo - 1;
  }
};

// Two values -> the dwords of their three planes.
__device__ __attribute__((always_inline)) inline void split3(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = pack2<TagBF16>(a, b);
  const float ra = a - __builtin_bit_cast(float, h << 16), rb = b - __builtin_bit_cast(float, h & 0xffff0000u);
  m = pack2<TagBF16>(ra, rb);
  const float sa = ra - __builtin_bit_cast(float, m << 16), sb = rb - __builtin_bit_cast(float, m & 0xffff0000u);
  l = pack2<TagBF16>(sa, sb);
}

// A padded row -> LDS (window-major planes); float32: returns whether the row
// is far (FWD: see FarRangeFwd).
template <class Tag, int RP, int S, bool FWD>
__device__ __attribute__((always_inline)) inline bool gen_write(unsigned char *xb, int v, int hi,
                                                                const uint32_t (&d)[RP * Tag::ES / 4]) {
  typedef GenCfg<Tag, RP, S> G;
  unsigned char *p = xb + (v * G::LDSW + hi * RP) * 2;
  bool far = false;
  if constexpr (Tag::W16) {
#pragma unroll
    for (int i = 0; i < G::ND; i += 4)
      *reinterpret_cast<uint4 *>(p + 4 * i) = make_uint4(d[i], d[i + 1], d[i + 2], d[i + 3]);
  } else {
    if constexpr (FWD) {
      FarRangeFwd mag;
#pragma unroll
      for (int i = 0; i < G::ND; i += 2) mag.add(d[i], d[i + 1]);
      far = mag.far();
    } else {
      FarRange mag;
#pragma unroll
      for (int i = 0; i < G::ND; ++i) mag.add(d[i]);
      far = mag.far();
    }
#pragma unroll
    for (int i = 0; i < RP; i += 8) {
      uint32_t h[4], m[4], l[4];
#pragma unroll
      for (int k = 0; k < 4; ++k)
        split3(__builtin_bit_cast(float, d[i + 2 * k]), __builtin_bit_cast(float, d[i + 2 * k + 1]), h[k], m[k], l[k]);
      *reinterpret_cast<uint4 *>(p + 2 * i) = make_uint4(h[0], h[1], h[2], h[3]);
      *reinterpret_cast<uint4 *>(p + G::PLANE + 2 * i) = make_uint4(m[0], m[1], m[2], m[3]);
      *reinterpret_cast<uint4 *>(p + 2 * G::PLANE + 2 * i) = make_uint4(l[0], l[1], l[2], l[3]);
    }
  }
  return far;
}

typedef u16x8 GFrag;

__device__ __attribute__((always_inline)) inline f32x4 mma_bf16(GFrag a, GFrag b, f32x4 c) { return mma<TagBF16>(a, b, c); }

// Coefficient of input position (hi, xi) and output position (ho, xo), both
// inside the window, in global memory.
template <class Tag>
__device__ __attribute__((always_inline)) inline int64_t gen_coef(const GenArgs &a, int64_t c, int hi, int xi, int ho,
                                                                  int xo) {
  const int K1 = 2 * a.ww - 1, K2 = K1 * (2 * a.wh - 1), d = a.wh * a.ww;
  if (a.src <= kSrcTableRev) {
    const int k = (hi - ho + a.wh - 1) * K1 + xi - xo + a.ww - 1;
    return c * K2 + (a.src == kSrcTableRev ? K2 - 1 - k : k);
  }
  const int i = hi * a.ww + xi, j = ho * a.ww + xo;
  return c * d * d + (a.src == kSrcMat ? i * d + j : j * d + i);
}

// ---- coefficients from the table
// Toeplitz blocks in LDS, block dh = hi - ho from -(KR - 1) to KR - 1 as
// [x_out][x_in] (zero past the window), from the table copy Ts (reversed for
// the input gradient): a fragment is then one 16-byte read at a per-lane
// base plus a constant.  float32: three planes, the lowest at tblow.
template <class Tag, int RP, int S>
__device__ __attribute__((always_inline)) inline void gen_build_tb(const GenArgs &a, const typename Tag::S *Ts,
                                                                   unsigned char *tb, unsigned char *tblow,
                                                                   int tid) {
  typedef GenCfg<Tag, RP, S> G;
  constexpr int CPR = RP / 8;  // 8-element chunks per block row
  const int K1 = 2 * a.ww - 1;
  for (int ch = tid; ch < G::NBLK * RP * CPR; ch += kGenThreads) {
    const int row = ch / CPR, xi0 = (ch % CPR) * 8;
    const int dh = row / RP - (G::KR - 1), xo = row % RP;
    const bool ok = dh > -a.wh && dh < a.wh && xo < a.ww;
    const int base = ok ? (dh + a.wh - 1) * K1 + xi0 - xo + a.ww - 1 : 0;
    const int nv = ok ? a.ww - xi0 : 0;  // columns inside the window
    const int off = (row * RP + xi0) * 2;
    unsigned char *p = tb + off;
    if constexpr (Tag::W16) {
      const uint32_t *q = reinterpret_cast<const uint32_t *>(Ts) + (base >> 1);
      const uint32_t sh = (uint32_t)(base & 1) * 16u;
      uint32_t d[5], u[4];
#pragma unroll
      for (int i = 0; i < 5; ++i) d[i] = q[i];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t w = __builtin_amdgcn_alignbit(d[i + 1], d[i], sh);
        u[i] = nv > 2 * i + 1 ? w : nv > 2 * i ? (w & 0xffffu) : 0u;
      }
      *reinterpret_cast<uint4 *>(p) = make_uint4(u[0], u[1], u[2], u[3]);
    } else {
      uint32_t h[4], m[4], l[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float f0 = nv > 2 * k ? Ts[base + 2 * k] : 0.f, f1 = nv > 2 * k + 1 ? Ts[base + 2 * k + 1] : 0.f;
        split3(f0, f1, h[k], m[k], l[k]);
      }
      *reinterpret_cast<uint4 *>(p) = make_uint4(h[0], h[1], h[2], h[3]);
      *reinterpret_cast<uint4 *>(p + G::TBB) = make_uint4(m[0], m[1], m[2], m[3]);
      *reinterpret_cast<uint4 *>(tblow + off) = make_uint4(l[0], l[1], l[2], l[3]);
    }
  }
}

// Byte offset in the blocks of lane's part of the fragment of tile pair T at
// tile 0, K step 0, and the step from there to tile h, K step s.
template <class Tag, int RP, int S>
__device__ __attribute__((always_inline)) inline int gen_tb_lane(int T, int lane) {
  const int g = lane >> 4, ln = lane & 15;
  const int hl = 8 * g / RP, xi0 = 8 * g % RP;  // row within the K step, first column
  const int ol = ln / RP, xo = ln % RP;         // row within the output tile, column
  return (((hl - ol - T * (32 / RP) + GenCfg<Tag, RP, S>::KR - 1) * RP + xo) * RP + xi0) * 2;
}
template <int RP>
__host__ __device__ constexpr int gen_tb_step(int h, int s) { return (s * (32 / RP) - h * (16 / RP)) * RP * RP * 2; }

// This wave's fragments from the blocks: out positions 32 T + 16 h .. + 15
// (h = 0, 1), K step s.  Rows past the window are zero coefficients; output
// positions past it are not stored and may hold anything.
template <class Tag, int RP, int S, int NPR>
__device__ __attribute__((always_inline)) inline void gen_frags_tb(const GenArgs &a, const unsigned char *tb, int T,
                                                                   int lane, GFrag (&fr)[NPR][2][S]) {
  typedef GenCfg<Tag, RP, S> G;
  const int g = lane >> 4;
  const int hl = 8 * g / RP;  // row within the K step
  const unsigned char *base = tb + gen_tb_lane<Tag, RP, S>(T, lane);
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int p = 0; p < NPR; ++p) {
        fr[p][h][s] = *reinterpret_cast<const GFrag *>(base + p * G::TBB + gen_tb_step<RP>(h, s));
        if (s == S - 1 && (S - 1) * (32 / RP) + hl >= a.wh) fr[p][h][s] = GFrag{0, 0, 0, 0, 0, 0, 0, 0};
      }
}

// ---- coefficients from a matrix, 16-bit
// Position-major fragment (16 columns x 8 rows per lane group) of a row-major
// LDS tile: lane (g, i) receives column 16 t + i of rows 8 g .. 8 g + 7, by
// two transposing reads.
template <int LDSW>
__device__ __attribute__((always_inline)) inline GFrag gen_tr_frag(const unsigned char *tile, int t, int lane) {
  const int g = lane >> 4, r = (lane >> 2) & 3, q = lane & 3;
  const int e0 = (8 * g + r) * LDSW + 16 * t + 4 * q;
  const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(tile + 2 * e0));
  const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4 *)(tile + 2 * (e0 + 4 * LDSW)));
  return __builtin_bit_cast(GFrag, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The matrix goes through LDS in chunks of 32 padded rows (rows and columns
// padded as window positions, pads zero), a few chunks at a time, one window
// row of one matrix row per thread.  M: chunk s holds K step s of every
// output position, read with transposing reads; M^T: chunk T holds all of
// wave T's fragments, read as they lie.  (Gathering the fragments from global
// memory took most of the kernel: B128 C256 28x28, 14 x 14 windows, bf16.)
template <class Tag, int RP, int S, int ROOM, bool TRANS>
__device__ __attribute__((always_inline)) inline void gen_frags_mat16(const GenArgs &a, const u16 *coef, int64_t c,
                                                                      int T, int tid, const uint32_t *masks,
                                                                      unsigned char *lds,
                                                                      GFrag (&fr)[1][2][S]) {
  typedef GenCfg<Tag, RP, S> G;
  constexpr int CKB = G::CKB;
  constexpr int NCK = ROOM / CKB < S ? ROOM / CKB : S;  // chunks at a time
  static_assert(NCK >= 1 && 32 * G::KR <= kGenThreads, "one row per thread and chunk");
  const int lane = tid & 63, g = lane >> 4, ln = lane & 15;
  const int d = a.wh * a.ww;
  const int64_t numel = a.C * d * d;
  const int kk = tid / G::KR, ho = tid - kk * G::KR;  // padded row of the chunk, window row of its columns
  auto row = [&](int ck) __attribute__((always_inline)) -> GRow {
    const int hi = ck * (32 / RP) + kk / RP, xi = kk % RP;
    GRow r;
    r.cols = ck < S && kk < 32 && hi < a.wh && xi < a.ww && ho < a.wh ? a.ww : 0;
    r.eoff = c * d * d + (int64_t)(hi * a.ww + xi) * d + ho * a.ww;
    return r;
  };
  uint32_t v[NCK][G::ND];
#pragma unroll
  for (int q = 0; q < NCK; ++q) gen_load<Tag, RP>(numel, coef, row(q), v[q]);
#pragma unroll
  for (int c0 = 0; c0 < S; c0 += NCK) {
#pragma unroll
    for (int q = 0; q < NCK; ++q) {
      const GRow r = row(c0 + q);
      gen_tail<Tag, RP>(numel, r, v[q]);
      gen_mask<Tag, RP>(masks, r.cols, v[q]);
      if (kk < 32) {
        unsigned char *p = lds + q * CKB + (kk * G::LDSW + ho * RP) * 2;
#pragma unroll
        for (int i = 0; i < G::ND; i += 4)
          *reinterpret_cast<uint4 *>(p + 4 * i) = make_uint4(v[q][i], v[q][i + 1], v[q][i + 2], v[q][i + 3]);
      }
    }
    __syncthreads();
    if (c0 + NCK < S) {
#pragma unroll
      for (int q = 0; q < NCK; ++q) gen_load<Tag, RP>(numel, coef, row(c0 + NCK + q), v[q]);
    }
    if constexpr (TRANS) {
      const int q = T - c0;
      if (q >= 0 && q < NCK) {
        const unsigned char *t = lds + q * CKB + (ln * G::LDSW + 8 * g) * 2;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int s = 0; s < S; ++s) fr[0][h][s] = *reinterpret_cast<const GFrag *>(t + 32 * h * G::LDSW + 64 * s);
      }
    } else {
#pragma unroll
      for (int s = c0; s < (c0 + NCK < S ? c0 + NCK : S); ++s)
#pragma unroll
        for (int h = 0; h < 2; ++h) fr[0][h][s] = gen_tr_frag<G::LDSW>(lds + (s - c0) * CKB, 2 * T + h, lane);
    }
    __syncthreads();
  }
}

// ---- coefficients from a matrix, float32: gathered from global memory
template <int RP, int S>
__device__ __attribute__((always_inline)) inline void gen_frags_mat32(const GenArgs &a, const float *coef, int64_t c,
                                                                      int T, int lane, GFrag (&fr)[3][2][S],
                                                                      FarRange &mag) {
  const int g = lane >> 4, ln = lane & 15;
  const int d = a.wh * a.ww;
  const float *cm = coef + c * d * d;
  // the eight columns of a fragment, the same for every K step and tile:
  // masks of the ones inside the window, and their offsets from the first
  const int xi0 = 8 * g % RP;
  uint32_t cmask[8];
  int eoff[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const bool in = xi0 + e < a.ww;
    eoff[e] = in ? e * (a.src == kSrcMat ? d : 1) : 0;
    cmask[e] = in ? ~0u : 0u;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = 32 * T + 16 * h + ln;
    const int ho = j / RP, xo = j % RP;
    const int j0 = ho * a.ww + xo;
    const bool jok = ho < a.wh && xo < a.ww;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int hi = (32 * s + 8 * g) / RP;
      const bool ok = jok && hi < a.wh && xi0 < a.ww;
      const uint32_t okm = ok ? ~0u : 0u;
      const int i0 = hi * a.ww + xi0;
      const int base = !ok ? 0 : a.src == kSrcMat ? i0 * d + j0 : j0 * d + i0;
      float v[8];
      uint32_t hh[4], mm[4], ll[4];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint32_t u = __builtin_bit_cast(uint32_t, cm[(uint32_t)(base + eoff[e])]) & cmask[e] & okm;
        // (the finished value, not its parts, is what stays in registers)
        asm volatile("" : "+v"(u));
        v[e] = __builtin_bit_cast(float, u);
        mag.add(u);
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) split3(v[2 * k], v[2 * k + 1], hh[k], mm[k], ll[k]);
      fr[0][h][s] = __builtin_bit_cast(GFrag, make_uint4(hh[0], hh[1], hh[2], hh[3]));
      fr[1][h][s] = __builtin_bit_cast(GFrag, make_uint4(mm[0], mm[1], mm[2], mm[3]));
      fr[2][h][s] = __builtin_bit_cast(GFrag, make_uint4(ll[0], ll[1], ll[2], ll[3]));
      // a few fragments' loads in flight at a time: all of them at once
      // would not fit the registers
      if (s % 4 == 3 || s + 1 == S) __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// float32 products of one window per lane and a tile pair (far rows, far
// coefficients): four columns of one window row per lane at a time, from
// global memory, and the same four input positions' coefficients from cc, the
// channel's table or matrix (src as in GenArgs).
template <int RP, int S>
__device__ __attribute__((always_inline)) inline void gen_far_pair(const GenArgs &a, const float *x, const float *cc,
                                                                   int src, int64_t c, uint32_t n, int T, int lane,
                                                                   f32x4 (&acc)[2]) {
  asm volatile("" : "+v"(lane));  // (what follows from it stays in this branch)
  const int g = lane >> 4, ln = lane & 15;
  const int hl = 8 * g / RP, x0 = 8 * g % RP;
  const int K1 = 2 * a.ww - 1, K2 = K1 * (2 * a.wh - 1), d = a.wh * a.ww;
  // coefficient of the lane's first input position at window row 0, and the
  // steps to the next column and row
  const int col = src == kSrcTable || src == kSrcMatT ? 1 : src == kSrcTableRev ? -1 : d;
  const int rstep = src == kSrcTable ? K1 : src == kSrcTableRev ? -K1 : a.ww * col;
  int base[2];
  bool out[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int j = 32 * T + 16 * h + ln, ho = j / RP, xo = j % RP;
    out[h] = ho < a.wh && xo < a.ww;
    const int k = (a.wh - 1 - ho) * K1 + x0 - xo + a.ww - 1, p = ho * a.ww + xo;
    base[h] = src == kSrcTable ? k : src == kSrcTableRev ? K2 - 1 - k : src == kSrcMat ? x0 * d + p : p * d + x0;
  }
#pragma unroll 1
  for (int q = 0; q < 2 * S; ++q) {
    const int hi = (q >> 1) * (32 / RP) + hl, xq = 4 * (q & 1);
    GRow r = gen_row(a, c, n, hi);
    r.eoff += x0 + xq;
    r.cols = r.cols - x0 - xq < 0 ? 0 : r.cols - x0 - xq;
    uint32_t v[4];
    gen_load<TagF32, 4>(a.numel, x, r, v);
    float bv[2][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const bool in = out[h] && hi < a.wh && x0 + xq + i < a.ww;
        const float f = cc[in ? base[h] + hi * rstep + (xq + i) * col : 0];
        bv[h][i] = in ? f : 0.f;
      }
    gen_tail<TagF32, 4>(a.numel, r, v);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float av = i < r.cols ? __builtin_bit_cast(float, v[i]) : 0.f;
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[h] = mma<TagF32>(bv[h][i], av, acc[h]);
    }
  }
}

// Registers and LDS of the forward kernel (MAT: coefficients from a matrix).
template <class Tag, int RP, int S, bool MAT>
struct GenFwd {
  typedef GenCfg<Tag, RP, S> G;
  // float32 fragments: the lowest plane (one product in six) stays in LDS as
  // Toeplitz blocks where all three would not leave registers for the rows in
  // flight
  static constexpr bool LOW = !Tag::W16 && !MAT && S >= 6;
  static constexpr int NPR = LOW ? 2 : G::NPL;          // planes in registers
  static constexpr bool TIGHT = !Tag::W16 && MAT && S >= 5;  // registers short
  static constexpr int AHEAD = TIGHT ? 2 : 3;           // stages from a row's load to its use, + 1
  static constexpr int FIX = (LOW ? G::TBB : 0) + gen_mask_bytes<Tag, RP>() + 32;  // blocks, masks, flags
  static constexpr int NOB = 2 * G::XB + 2 * G::OB + FIX <= 160 * 1024 ? 2 : 1;  // result buffers
  static constexpr int MROOM = (160 * 1024 - FIX - G::XB) / G::CKB * G::CKB;
  static constexpr int MEND = Tag::W16 && MAT ? G::XB + (MROOM < S * G::CKB ? MROOM : S * G::CKB) : 0;
  // 16-bit matrices: LDS for as many chunks as there are, one workgroup per
  // compute unit
  static constexpr int LOW_OFF = 2 * G::XB + NOB * G::OB > MEND ? 2 * G::XB + NOB * G::OB : MEND;
  static constexpr int MASK_OFF = LOW_OFF + (LOW ? G::TBB : 0);
  static constexpr int FLAG_OFF = MASK_OFF + gen_mask_bytes<Tag, RP>();
  static constexpr size_t LDS = (size_t)FLAG_OFF + 32;
  static constexpr int WGS = Tag::W16 && LDS <= 80 * 1024 ? 2 : 1;  // workgroups per compute unit
};

// Y = X M per window.  Stage s is multiplied while stage s + 1 (in registers)
// goes to the other LDS buffer, stage s + 3 is loaded and the rows of stage
// s - 1 are stored: one barrier per stage.
//
// What bounds it: 16-bit, memory while it streams (about 5 TB/s of the 7 a
// copy reaches) and, at the sizes of a layer, the prologue (2.6 us of launch,
// 4 to 5 until the first stage is multiplied); float32, the matrix cores, six
// products for one, at the 1.9 GHz this load runs at.  Measured (us, before:
// the kernels these replaced): bf16 matrix B128 C256 28x28 14 x 14 468 -> 33;
// bf16 table w = 14 B8 C96 100x167 40 -> 19; float32 table w = 14 B1 C8
// 28x28 33 -> 8.9.  The two waves of a SIMD in opposite order (float32,
// B128 C256 56x56): 368 -> 305.
template <class Tag, int RP, int S, bool MAT>
__global__ __launch_bounds__(kGenThreads, (2 * GenFwd<Tag, RP, S, MAT>::WGS)) void gen_fwd_kernel(
    const typename Tag::S *__restrict__ x, const typename Tag::S *__restrict__ coef, typename Tag::S *__restrict__ y,
    GenArgs a) {
  typedef typename Tag::S E;
  typedef GenCfg<Tag, RP, S> G;
  typedef GenFwd<Tag, RP, S, MAT> F;
  constexpr bool DEEP = F::AHEAD == 3;  // two stages of rows in flight
  constexpr bool TWO = F::NOB == 2;
  extern __shared__ __align__(16) unsigned char smem[];
  unsigned char *xbuf = smem, *obuf = smem + 2 * G::XB;
  int *flag = reinterpret_cast<int *>(smem + F::FLAG_OFF);
  uint32_t *masks = reinterpret_cast<uint32_t *>(smem + F::MASK_OFF);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, ln = lane & 15;
  const uint32_t bid = gen_block();
  const int64_t c = bid / (uint32_t)a.tiles_per_ch;
  if (c >= a.C) return;
  const int s0 = (int)(bid - (uint32_t)c * (uint32_t)a.tiles_per_ch) * a.spw;
  const int nst = a.stages - s0 < a.spw ? a.stages - s0 : a.spw;
  const uint32_t n0 = (uint32_t)s0 * G::CW;
  const int v = gen_slot_window<G>(a, tid), hi = gen_slot_row<G>(a, tid);

  // this thread's row of stage s (none past the last stage)
  auto row = [&](int s) __attribute__((always_inline)) -> GRow { return s < nst ? gen_row(a, c, n0 + s * G::CW + v, hi) : GRow{0, 0}; };

  // ---- stages 0 and 1 in flight, the table -> LDS, this wave's fragments
  // (the table first, ahead of the rows: two entries per thread, K2 <= 961)
  const int K2 = (2 * a.ww - 1) * (2 * a.wh - 1);
  E tv[2] = {(E)0, (E)0};
  if constexpr (!MAT) {
    const E *tc = coef + c * K2;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = tid + i * kGenThreads < K2 ? tid + i * kGenThreads : K2 - 1;
      tv[i] = tc[a.src == kSrcTableRev ? K2 - 1 - k : k];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  uint32_t d0[G::ND], d1[G::ND];
  gen_load<Tag, RP>(a.numel, x, row(0), d0);
  if constexpr (DEEP) gen_load<Tag, RP>(a.numel, x, row(1), d1);
  __builtin_amdgcn_sched_barrier(0);
  E *Ts = reinterpret_cast<E *>(obuf);
  FarRange cmag;  // coefficients seen (float32)
  if constexpr (!MAT) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = tid + i * kGenThreads;
      if constexpr (!Tag::W16) cmag.add(__builtin_bit_cast(uint32_t, tv[i]));
      if (k < K2 + 10) Ts[k] = k < K2 ? tv[i] : (E)0;
    }
  }
  if (tid < 5) flag[tid] = -1;
  gen_mask_table<Tag, RP>(masks, tid);
  __syncthreads();
  const int T = wave % S, sg = wave / S;  // tile pair, sub-tile group
  GFrag fr[F::NPR][2][S];
  if constexpr (MAT) {
    constexpr int ROOM = F::LOW_OFF - G::XB;
    if constexpr (Tag::W16) {
      if (a.src == kSrcMat) gen_frags_mat16<Tag, RP, S, ROOM, false>(a, coef, c, T, tid, masks, xbuf + G::XB, fr);
      else gen_frags_mat16<Tag, RP, S, ROOM, true>(a, coef, c, T, tid, masks, xbuf + G::XB, fr);
    } else
      gen_frags_mat32<RP, S>(a, coef, c, T, lane, fr, cmag);
  } else {
    gen_build_tb<Tag, RP, S>(a, Ts, xbuf + G::XB, F::LOW ? smem + F::LOW_OFF : xbuf + G::XB + 2 * G::TBB, tid);
  }
  if constexpr (!Tag::W16) {
    // far coefficients: a huge or a tiny one, or none of normal size though
    // not all are zero
    if (__any(cmag.far()) && lane == 0) flag[2] = 1;
    if (__any(cmag.mx != 0) && lane == 0) flag[3] = 1;
    if (__any(cmag.mx >= 2 * kFarLoCoef) && lane == 0) flag[4] = 1;
  }
  __syncthreads();
  if constexpr (!MAT) gen_frags_tb<Tag, RP, S>(a, xbuf + G::XB, T, lane, fr);
  bool cfar = false;
  if constexpr (!Tag::W16) cfar = flag[2] > 0 || (flag[3] > 0 && flag[4] < 0);
  auto write = [&](int s, uint32_t (&d)[G::ND]) __attribute__((always_inline)) {
    const GRow r = row(s);
    gen_tail<Tag, RP>(a.numel, r, d);
    gen_mask<Tag, RP>(masks, r.cols, d);
#pragma unroll
    for (int i = 0; i < G::ND; ++i) asm volatile("" : "+v"(d[i]));  // (the rows arrive here, on every path)
    if (hi < G::KR) {
      if (gen_write<Tag, RP, S, true>(xbuf + (s & 1) * G::XB, v, hi, d)) flag[s & 1] = s;
    }
  };
  write(0, d0);
  if constexpr (DEEP) {
    gen_load<Tag, RP>(a.numel, x, row(2), d0);
  } else {
    gen_load<Tag, RP>(a.numel, x, row(1), d1);
  }
  __builtin_amdgcn_sched_barrier(0);
  __syncthreads();

  auto store = [&](int s) __attribute__((always_inline)) {
    const GRow r = row(s);
    if (r.cols > 0) {
      const unsigned char *ob = obuf + (TWO ? (s & 1) * G::OB : 0) + (v * G::OP + hi * RP) * Tag::ES;
      uint32_t o[G::ND];
#pragma unroll
      for (int i = 0; i < G::ND; i += 4) {
        const uint4 u = *reinterpret_cast<const uint4 *>(ob + 4 * i);
        o[i] = u.x; o[i + 1] = u.y; o[i + 2] = u.z; o[i + 3] = u.w;
      }
      gen_store<Tag, RP>(y, r, o);
    }
  };
  // products of stage s: this wave's tile pair of its sub-tiles sg + i NG
  const unsigned char *lowp = smem + F::LOW_OFF + gen_tb_lane<Tag, RP, S>(T, lane);
  auto compute = [&](int s) __attribute__((always_inline)) {
    const unsigned char *xs = xbuf + (s & 1) * G::XB;
    unsigned char *os = obuf + (TWO ? (s & 1) * G::OB : 0);
    if (sg >= G::NG) return;
    bool far = false;
    if constexpr (!Tag::W16) far = cfar || __builtin_amdgcn_readfirstlane(flag[s & 1]) == s;
    constexpr int NJ = Tag::W16 ? G::SPW : 1;  // sub-tiles at a time
#pragma unroll 1
    for (int i0 = 0; i0 < G::SPW; i0 += NJ) {
      const int u0 = sg + i0 * G::NG;
      const unsigned char *xp = xs + ((16 * u0 + ln) * G::LDSW + 8 * g) * 2;
      constexpr int US = 16 * G::NG * G::LDSW * 2;  // bytes from one of its sub-tiles to the next
      f32x4 acc[NJ][2];
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[j][0] = acc[j][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (Tag::W16) {
#pragma unroll
        for (int k = 0; k < S; ++k) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) {
            const GFrag xf = *reinterpret_cast<const GFrag *>(xp + j * US + 64 * k);
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[j][h] = mma<Tag>(fr[0][h][k], xf, acc[j][h]);
          }
        }
      } else {
        if (far) {
          const uint32_t n = n0 + s * G::CW + 16 * u0 + ln;
          gen_far_pair<RP, S>(a, x, coef + c * (MAT ? a.wh * a.ww * a.wh * a.ww : K2), a.src, c, n, T, lane, acc[0]);
        } else {
          // three sums per tile: hi hi, then the partial products of weight
          // 2^-8 (mb) and 2^-16 (lb); the operands of step k + 1 are read
          // while step k is multiplied
          f32x4 mb[2], lb[2];
          mb[0] = mb[1] = lb[0] = lb[1] = f32x4{0.f, 0.f, 0.f, 0.f};
          struct Ops {
            GFrag xh, xm, xl, fl[2];
          } op[2];
          auto fetch = [&](int k, Ops &o) __attribute__((always_inline)) {
            o.xh = *reinterpret_cast<const GFrag *>(xp + 64 * k);
            o.xm = *reinterpret_cast<const GFrag *>(xp + G::PLANE + 64 * k);
            o.xl = *reinterpret_cast<const GFrag *>(xp + 2 * G::PLANE + 64 * k);
            if constexpr (F::LOW) {
#pragma unroll
              for (int h = 0; h < 2; ++h) o.fl[h] = *reinterpret_cast<const GFrag *>(lowp + gen_tb_step<RP>(h, k));
            }
          };
          fetch(0, op[0]);
#pragma unroll
          for (int k = 0; k < S; ++k) {
            const Ops &o = op[k & 1];
            if (k + 1 < S) fetch(k + 1, op[(k + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
            GFrag fl[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              if constexpr (F::LOW) {
                fl[h] = o.fl[h];
                if (k == S - 1 && (S - 1) * (32 / RP) + 8 * g / RP >= a.wh) fl[h] = GFrag{0, 0, 0, 0, 0, 0, 0, 0};
              } else {
                fl[h] = fr[2][h][k];
              }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[0][h] = mma_bf16(fr[0][h][k], o.xh, acc[0][h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) mb[h] = mma_bf16(fr[1][h][k], o.xh, mb[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) lb[h] = mma_bf16(fl[h], o.xh, lb[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) mb[h] = mma_bf16(fr[0][h][k], o.xm, mb[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) lb[h] = mma_bf16(fr[1][h][k], o.xm, lb[h]);
#pragma unroll
            for (int h = 0; h < 2; ++h) lb[h] = mma_bf16(fr[0][h][k], o.xl, lb[h]);
            __builtin_amdgcn_sched_barrier(0);
          }
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0][h][e] += mb[h][e] + lb[h][e];
        }
      }
      // window ln of the sub-tile, positions 32 T + 16 h + 4 g .. + 3
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        E *o = reinterpret_cast<E *>(os) + (16 * (u0 + j * G::NG) + ln) * G::OP + 32 * T + 4 * g;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f32x4 v4 = acc[j][h];
          if constexpr (Tag::W16)
            *reinterpret_cast<uint2 *>(o + 16 * h) = uint2{pack2<Tag>(v4[0], v4[1]), pack2<Tag>(v4[2], v4[3])};
          else
            *reinterpret_cast<float4 *>(o + 16 * h) = float4{v4[0], v4[1], v4[2], v4[3]};
        }
      }
    }
  };
  // stage s + 1 from d to LDS, stage s + AHEAD into d, the previous stage's
  // rows out
  auto move = [&](int s, uint32_t (&d)[G::ND]) __attribute__((always_inline)) {
    // (also past the last stage, with zeros: no branch, see gen_load)
    write(s + 1, d);
    // (the stores before the loads: the next wait for rows, which counts the
    // loads behind them only, then leaves those in flight)
    if constexpr (TWO) {
      if (s > 0) store(s - 1);
    }
    gen_load<Tag, RP>(a.numel, x, row(s + F::AHEAD), d);
  };
  // float32 (one workgroup per compute unit): the second wave of each SIMD
  // takes a stage's copies before its products, the first one after, so that
  // the copies' vector instructions run beside the other wave's products
  // (two loops, not a branch inside one: the waits for rows stay exact)
  auto stage = [&](auto early, int s, uint32_t (&da)[G::ND], uint32_t (&db)[G::ND]) __attribute__((always_inline)) {
    compute(s);
    if constexpr (!early.value) move(s, da);
    __syncthreads();
    if constexpr (!TWO) {
      store(s);
      __syncthreads();
    }
    if constexpr (early.value) move(s + 1, db);
  };
  auto run = [&](auto early) __attribute__((always_inline)) {
    if constexpr (early.value) move(0, d1);
    if constexpr (DEEP) {
      for (int s = 0; s < nst; s += 2) {
        stage(early, s, d1, d0);
        if (s + 1 >= nst) break;
        stage(early, s + 1, d0, d1);
      }
    } else {
      for (int s = 0; s < nst; ++s) stage(early, s, d1, d1);
    }
  };
  if (!Tag::W16 && wave >= kGenWaves / 2) {
    run(std::true_type{});
    // (the last move stored the last stage's rows)
    return;
  }
  run(std::false_type{});
  if constexpr (TWO) store(nst - 1);
}

// ---------------------------------------------- float32, many windows
// Y = X M from the table for maps that fill the chip with 16-window units,
// one per wave: no stages, no barriers.  A wave reads its windows' fragments
// straight from global memory (eight consecutive columns of one window row
// per lane and K step), splits them in registers, multiplies them by the
// table's fragments in LDS, tile pair by tile pair, and stores four consecutive
// columns per lane; the next unit's rows are in flight meanwhile.  Two waves
// per SIMD, at different points of their units, keep the matrix cores busy
// through each other's splitting, loads and stores.
//
// What bounds it: the matrix cores at the rate the card sustains.  B128 C256
// 56x56, w = 14: 275 us for 316 GFLOP of partial products, 1150 TFLOP/s (a large
// bf16 matrix product reaches 1190 to 1360 on this card, which lowers its clock under
// it); 257 without loads and stores, 227 with the products alone.  The staged
// kernel above: 295.
template <int RP, int S>
struct GenDirect {
  typedef GenCfg<TagF32, RP, S> G;
  // a fragment depends on 2 k - t (K step, output tile) alone: NF of them,
  // each stored in lane order (a fragment read covers 1 KB without bank
  // conflicts; from Toeplitz blocks half of the LDS cycles were conflicts)
  static constexpr int NF = 4 * S - 2;
  static constexpr int PL = NF * 1024;  // bytes of one plane
  static constexpr int TS_OFF = 3 * PL;             // table copy, then the masks of 0 .. 8 columns, flags
  static constexpr int MASK_OFF = TS_OFF + 4 * 976;
  static constexpr int FLAG_OFF = MASK_OFF + 9 * 32;
  static constexpr size_t LDS = (size_t)FLAG_OFF + 16;
};

template <int RP, int S>
__global__ __launch_bounds__(kGenThreads, 2) void gen_direct_kernel(const float *__restrict__ x,
                                                                    const float *__restrict__ tab,
                                                                    float *__restrict__ y, GenArgs a) {
  typedef GenDirect<RP, S> D;
  constexpr int KROWS = 32 / RP;  // window rows per K step
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, ln = lane & 15;
  const uint32_t bid = gen_block();
  const int64_t c = bid / (uint32_t)a.tiles_per_ch;
  if (c >= a.C) return;
  // units of this workgroup (spw rounds of eight), this wave's every eighth
  const int u0 = (int)(bid - (uint32_t)c * (uint32_t)a.tiles_per_ch) * a.spw * kGenWaves;
  const int nu = (int)((a.N + 15) / 16);
  const int u1 = nu - u0 < a.spw * kGenWaves ? nu : u0 + a.spw * kGenWaves;

  // ---- the table -> LDS -> blocks
  const int K2 = (2 * a.ww - 1) * (2 * a.wh - 1);
  float *Ts = reinterpret_cast<float *>(smem + D::TS_OFF);
  uint32_t *masks = reinterpret_cast<uint32_t *>(smem + D::MASK_OFF);
  int *flag = reinterpret_cast<int *>(smem + D::FLAG_OFF);
  const float *tc = tab + c * K2;
  FarRange cmag;
  for (int k = tid; k < K2 + 10; k += kGenThreads) {
    const float f = k < K2 ? tc[a.src == kSrcTableRev ? K2 - 1 - k : k] : 0.f;
    cmag.add(__builtin_bit_cast(uint32_t, f));
    Ts[k] = f;
  }
  if (tid < 72) masks[tid] = tid / 8 > tid % 8 ? ~0u : 0u;
  if (tid < 3) flag[tid] = 0;
  __syncthreads();
  for (int ch = tid; ch < D::NF * 64; ch += kGenThreads) {
    const int l = ch & 63, lg = l >> 4, lo = l & 15;
    const int dh = (ch / 64 - (2 * S - 1)) * (16 / RP) + 8 * lg / RP - lo / RP, xo = lo % RP, xi = 8 * lg % RP;
    const bool ok = dh > -a.wh && dh < a.wh && xo < a.ww;
    const int nv = ok ? a.ww - xi : 0;  // columns inside the window
    const float *t = Ts + (ok ? (dh + a.wh - 1) * (2 * a.ww - 1) + xi - xo + a.ww - 1 : 0);
    uint32_t hh[4], mm[4], ll[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float f0 = nv > 2 * k ? t[2 * k] : 0.f, f1 = nv > 2 * k + 1 ? t[2 * k + 1] : 0.f;
      split3(f0, f1, hh[k], mm[k], ll[k]);
    }
    unsigned char *p = smem + ch * 16;
    *reinterpret_cast<uint4 *>(p) = make_uint4(hh[0], hh[1], hh[2], hh[3]);
    *reinterpret_cast<uint4 *>(p + D::PL) = make_uint4(mm[0], mm[1], mm[2], mm[3]);
    *reinterpret_cast<uint4 *>(p + 2 * D::PL) = make_uint4(ll[0], ll[1], ll[2], ll[3]);
  }
  if (__any(cmag.far()) && lane == 0) flag[0] = 1;
  if (__any(cmag.mx != 0) && lane == 0) flag[1] = 1;
  if (__any(cmag.mx >= 2 * kFarLoCoef) && lane == 0) flag[2] = 1;
  __syncthreads();
  const bool cfar = flag[0] || (flag[1] && !flag[2]);

  // this lane's window of a unit: its first element, rows and columns inside
  // the image (0 rows: no window)
  struct Win {
    int64_t eoff;
    int rows, cols;
  };
  auto window = [&](int u) __attribute__((always_inline)) -> Win {
    Win w = {0, 0, 0};
    const uint32_t n = 16u * (uint32_t)u + ln;
    const uint32_t b = div_by(n, a.dnhw), rem = n - b * a.NHW;
    const uint32_t wy = div_by(rem, a.dnw), wx = rem - wy * a.NW;
    const int h0 = (int)wy * a.wh, x0 = (int)wx * a.ww;
    const bool ok = u < u1 && n < a.N;
    w.rows = !ok ? 0 : (int)a.H - h0 < a.wh ? (int)a.H - h0 : a.wh;
    w.cols = (int)a.W - x0 < a.ww ? (int)a.W - x0 : a.ww;
    w.eoff = (int64_t)b * a.chw + c * a.hw + (int64_t)h0 * a.W + x0;
    return w;
  };
  const int hl = 8 * g / RP, x0 = 8 * g % RP;  // row within a K step, first column
  const int64_t last = a.numel - 8;
  typedef const __attribute__((address_space(1))) u32x4u *GP;
  // (every lane loads, as in gen_load)
  auto load = [&](const Win &w, uint32_t (&raw)[S][8]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int r = KROWS * s + hl;
      int64_t e = w.eoff + (int64_t)r * a.W + x0;
      e = e < last ? e : last;
      const uint64_t p = r < w.rows && x0 < w.cols ? reinterpret_cast<uint64_t>(x + e) : reinterpret_cast<uint64_t>(gen_zero);
#pragma unroll
      for (int i = 0; i < 8; i += 4) {
        const u32x4u u = *reinterpret_cast<GP>(p + 4 * i);
        raw[s][i] = u.x; raw[s][i + 1] = u.y; raw[s][i + 2] = u.z; raw[s][i + 3] = u.w;
      }
    }
  };

  uint32_t raw[S][8];
  Win cur = window(u0 + wave);
  load(cur, raw);
  const unsigned char *tb0 = smem + (2 * S - 1) * 1024 + lane * 16;
  for (int u = u0 + wave; u < u1; u += kGenWaves) {
    // ---- the rows of this unit -> planes; the next unit's in flight
    GFrag xp[3][S];
    bool far = false;
    {
      const int nv = cur.cols - x0 < 0 ? 0 : cur.cols - x0 > 8 ? 8 : cur.cols - x0;
      const uint4 ma = *reinterpret_cast<const uint4 *>(masks + 8 * nv), mb = *reinterpret_cast<const uint4 *>(masks + 8 * nv + 4);
      const uint32_t m[8] = {ma.x, ma.y, ma.z, ma.w, mb.x, mb.y, mb.z, mb.w};
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const int r = KROWS * s + hl;
        const int64_t over = cur.eoff + (int64_t)r * a.W + x0 - last;
        if (r < cur.rows && x0 < cur.cols && over > 0) {
          // within eight elements of the tensor's end: see gen_tail
#pragma unroll 1
          for (int k = (int)over; k > 0; --k)
#pragma unroll
            for (int i = 0; i < 8; ++i) raw[s][i] = i < 7 ? raw[s][i + 1] : 0u;
        }
        FarRangeFwd mag;
        uint32_t hh[4], mm[4], ll[4];
#pragma unroll
        for (int i = 0; i < 8; ++i) raw[s][i] &= m[i];
#pragma unroll
        for (int i = 0; i < 8; i += 2) mag.add(raw[s][i], raw[s][i + 1]);
        far |= mag.far();
#pragma unroll
        for (int i = 0; i < 4; ++i)
          split3(__builtin_bit_cast(float, raw[s][2 * i]), __builtin_bit_cast(float, raw[s][2 * i + 1]), hh[i], mm[i], ll[i]);
        xp[0][s] = __builtin_bit_cast(GFrag, make_uint4(hh[0], hh[1], hh[2], hh[3]));
        xp[1][s] = __builtin_bit_cast(GFrag, make_uint4(mm[0], mm[1], mm[2], mm[3]));
        xp[2][s] = __builtin_bit_cast(GFrag, make_uint4(ll[0], ll[1], ll[2], ll[3]));
      }
    }
    const Win w = cur;
    // window ln, positions 16 t + 4 g .. + 3
    auto store = [&](int t, int g, const float (&v)[4]) __attribute__((always_inline)) {
      const int pos = 16 * t + 4 * g, r = pos / RP, xc = pos % RP;
      const int nc = r < w.rows ? w.cols - xc : 0;
      float *q = y + w.eoff + (int64_t)r * a.W + xc;
      if (nc >= 4) {
        *reinterpret_cast<u32x4a *>(q) = u32x4a{__builtin_bit_cast(uint32_t, v[0]), __builtin_bit_cast(uint32_t, v[1]),
                                                __builtin_bit_cast(uint32_t, v[2]), __builtin_bit_cast(uint32_t, v[3])};
      } else if (nc > 0) {
        q[0] = v[0];
        if (nc > 1) q[1] = v[1];
        if (nc > 2) q[2] = v[2];
      }
    };
    far = cfar || __any(far);
    cur = window(u + kGenWaves);
    load(cur, raw);
    __builtin_amdgcn_sched_barrier(0);
    // ---- output tiles 2 T, 2 T + 1
    const unsigned char *tb = tb0;
#pragma unroll 1
    for (int T = far ? S : 0; T < S; ++T, tb -= 2048) {
      f32x4 acc[2], mb[2], lb[2];
      acc[0] = acc[1] = mb[0] = mb[1] = lb[0] = lb[1] = f32x4{0.f, 0.f, 0.f, 0.f};
      {
        // (step, tile) by (step, tile); the blocks of the next one are read
        // while this one is multiplied (both tiles' at once would not fit
        // the registers)
        GFrag op[2][3];
        auto fetch = [&](int k, int h, GFrag (&o)[3]) __attribute__((always_inline)) {
#pragma unroll
          for (int p = 0; p < 3; ++p)
            o[p] = *reinterpret_cast<const GFrag *>(tb + p * D::PL + (2 * k - h) * 1024);
        };
        fetch(0, 0, op[0]);
#pragma unroll
        for (int q = 0; q < 2 * S; ++q) {
          const int k = q / 2, h = q % 2;
          const GFrag(&o)[3] = op[q & 1];
          if (q + 1 < 2 * S) fetch((q + 1) / 2, (q + 1) % 2, op[(q + 1) & 1]);
          __builtin_amdgcn_sched_barrier(0);
          lb[h] = mma_bf16(o[2], xp[0][k], lb[h]);
          mb[h] = mma_bf16(o[1], xp[0][k], mb[h]);
          acc[h] = mma_bf16(o[0], xp[0][k], acc[h]);
          lb[h] = mma_bf16(o[1], xp[1][k], lb[h]);
          mb[h] = mma_bf16(o[0], xp[1][k], mb[h]);
          lb[h] = mma_bf16(o[0], xp[2][k], lb[h]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = acc[h][e] + (mb[h][e] + lb[h][e]);
        store(2 * T + h, g, v);
      }
    }
    if (far) {
      // float32 products: four columns of one window row per lane at a time
      // (from memory again: kept, they would cost the usual path registers),
      // against the table's entries for them and every output tile.  Input
      // positions past the window have zero coefficients; outputs past it are
      // not stored, and what their lanes read (still LDS) does not matter.
      f32x4 acc[2 * S];
#pragma unroll
      for (int t = 0; t < 2 * S; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      int l = lane;
      asm volatile("" : "+v"(l));  // (what follows from it stays in this branch)
      const int K1 = 2 * a.ww - 1, hf = 8 * (l >> 4) / RP, xf = 8 * (l >> 4) % RP, lo = l & 15;
      const float *tl = Ts + (hf - lo / RP + a.wh - 1) * K1 + xf - lo % RP + a.ww - 1;
#pragma unroll 1
      for (int q = 0; q < 2 * S; ++q) {
        const int r = KROWS * (q >> 1) + hf, xq = xf + 4 * (q & 1);
        GRow f;
        f.eoff = w.eoff + (int64_t)r * a.W + xq;
        f.cols = r < w.rows ? w.cols - xq : 0;
        uint32_t v[4];
        gen_load<TagF32, 4>(a.numel, x, f, v);
        gen_tail<TagF32, 4>(a.numel, f, v);
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = i < f.cols ? v[i] : 0u;
        const float *tq = tl + KROWS * (q >> 1) * K1 + 4 * (q & 1);
#pragma unroll
        for (int t = 0; t < 2 * S; ++t) {
          float bv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            bv[i] = tq[i - t * (16 / RP) * K1];
            bv[i] = r < a.wh && xq + i < a.ww ? bv[i] : 0.f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i) acc[t] = mma<TagF32>(bv[i], __builtin_bit_cast(float, v[i]), acc[t]);
        }
      }
#pragma unroll
      for (int t = 0; t < 2 * S; ++t) {
        const float v[4] = {acc[t][0], acc[t][1], acc[t][2], acc[t][3]};
        store(t, l >> 4, v);
      }
    }

  }
}

// ---------------------------------------------- 16-bit, many windows
// The same for 16-bit values: one part per value, and every output tile of a
// unit accumulated together, so that a fragment of the table (which depends
// on 2 k - t alone) is read once per unit and serves every (K step, tile) pair
// that uses it.  The sums run over the K steps in order, as in the staged
// kernel: the same bits.
//
// What bounds it: the rows' way through the vector memory unit, 28 or 14 of
// every 32 or 16 bytes a lane asks for.  Staged kernel and this one, us: bf16
// w = 14 B8 C96 100x167 19.5 -> 18.6, w = 13 B16 C200 60x61 22.6 -> 20.8, w = 10
// B8 C96 100x167 21.1 -> 19.0, w = 7 17.3 -> 15.7; float16 7 x 14 windows B32 C96
// 56x56 13.7 -> 12.4, 16 x 3 windows B64 C40 48x48 15.6 -> 12.0.  Up to five K
// steps two workgroups share a compute unit (128 registers); with six and more
// that spilled (w = 14: 24.1), and one of twice the registers is the better.
// Five steps hold half of the tiles at a time.
template <int RP, int S>
struct GenDirect16 {
  static constexpr int NF = 4 * S - 2;
  static constexpr int TP = S == 5 ? S : 2 * S;     // output tiles accumulated together
  static constexpr int WGS = S <= 5 ? 2 : 1;        // workgroups per compute unit
  static constexpr int TS_OFF = NF * 1024;          // table copy, then the masks of 0 .. 8 columns
  static constexpr int MASK_OFF = TS_OFF + 2 * 976;
  static constexpr size_t LDS = (size_t)MASK_OFF + 9 * 16;
};

// PADK: the window's rows do not fill the last K step
template <class Tag, int RP, int S, bool PADK>
__global__ __launch_bounds__(kGenThreads, (GenDirect16<RP, S>::WGS * 2)) void gen_direct16_kernel(const typename Tag::S *__restrict__ x,
                                                                      const typename Tag::S *__restrict__ tab,
                                                                      typename Tag::S *__restrict__ y, GenArgs a) {
  typedef typename Tag::S E;
  typedef GenDirect16<RP, S> D;
  constexpr int KROWS = 32 / RP;  // window rows per K step
  extern __shared__ __align__(16) unsigned char smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, ln = lane & 15;
  const uint32_t bid = gen_block();
  const int64_t c = bid / (uint32_t)a.tiles_per_ch;
  if (c >= a.C) return;
  // units of this workgroup (spw rounds of eight), this wave's every eighth
  const int u0 = (int)(bid - (uint32_t)c * (uint32_t)a.tiles_per_ch) * a.spw * kGenWaves;
  const int nu = (int)((a.N + 15) / 16);
  const int u1 = nu - u0 < a.spw * kGenWaves ? nu : u0 + a.spw * kGenWaves;

  // ---- the table, ahead of the first rows
  const int K2 = (2 * a.ww - 1) * (2 * a.wh - 1);
  E *Ts = reinterpret_cast<E *>(smem + D::TS_OFF);
  uint32_t *masks = reinterpret_cast<uint32_t *>(smem + D::MASK_OFF);
  const E *tc = tab + c * K2;
  E tv[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = tid + i * kGenThreads < K2 ? tid + i * kGenThreads : K2 - 1;
    tv[i] = tc[a.src == kSrcTableRev ? K2 - 1 - k : k];
  }
  __builtin_amdgcn_sched_barrier(0);

  // this lane's window of a unit: its first element, rows and columns inside
  // the image (0 rows: no window)
  struct Win {
    int64_t eoff;
    int rows, cols;
  };
  auto window = [&](int u) __attribute__((always_inline)) -> Win {
    Win w = {0, 0, 0};
    const uint32_t n = 16u * (uint32_t)u + ln;
    const uint32_t b = div_by(n, a.dnhw), rem = n - b * a.NHW;
    const uint32_t wy = div_by(rem, a.dnw), wx = rem - wy * a.NW;
    const int h0 = (int)wy * a.wh, x0 = (int)wx * a.ww;
    const bool ok = u < u1 && n < a.N;
    w.rows = !ok ? 0 : (int)a.H - h0 < a.wh ? (int)a.H - h0 : a.wh;
    w.cols = (int)a.W - x0 < a.ww ? (int)a.W - x0 : a.ww;
    w.eoff = (int64_t)b * a.chw + c * a.hw + (int64_t)h0 * a.W + x0;
    return w;
  };
  const int hl = 8 * g / RP, x0 = 8 * g % RP;  // row within a K step, first column
  const int64_t last = a.numel - 8;
  typedef const __attribute__((address_space(1))) u32x4u *GP;
  // (every lane loads, as in gen_load)
  auto load = [&](const Win &w, u32x4u (&raw)[S]) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int r = KROWS * s + hl;
      int64_t e = w.eoff + (int64_t)r * a.W + x0;
      e = e < last ? e : last;
      const uint64_t p = r < w.rows && x0 < w.cols ? reinterpret_cast<uint64_t>(x + e) : reinterpret_cast<uint64_t>(gen_zero);
      raw[s] = *reinterpret_cast<GP>(p);
    }
  };
  u32x4u raw[S];
  Win cur = window(u0 + wave);
  load(cur, raw);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int k = tid + i * kGenThreads;
    if (k < K2 + 10) Ts[k] = k < K2 ? tv[i] : (E)0;
  }
  if (tid < 36) {
    const int cols = tid >> 2, i = tid & 3;
    masks[tid] = cols > 2 * i + 1 ? ~0u : cols > 2 * i ? 0xffffu : 0u;
  }
  __syncthreads();
  // ---- its fragments, in lane order
  for (int ch = tid; ch < D::NF * 64; ch += kGenThreads) {
    const int l = ch & 63, lg = l >> 4, lo = l & 15;
    const int dh = (ch / 64 - (2 * S - 1)) * (16 / RP) + 8 * lg / RP - lo / RP, xo = lo % RP, xi = 8 * lg % RP;
    const bool ok = dh > -a.wh && dh < a.wh && xo < a.ww;
    const int nv = ok ? a.ww - xi : 0;  // columns inside the window
    const int base = ok ? (dh + a.wh - 1) * (2 * a.ww - 1) + xi - xo + a.ww - 1 : 0;
    const uint32_t *q = reinterpret_cast<const uint32_t *>(Ts) + (base >> 1);
    const uint32_t sh = (uint32_t)(base & 1) * 16u;
    uint32_t d[5], u[4];
#pragma unroll
    for (int i = 0; i < 5; ++i) d[i] = q[i];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = __builtin_amdgcn_alignbit(d[i + 1], d[i], sh);
      u[i] = nv > 2 * i + 1 ? w : nv > 2 * i ? (w & 0xffffu) : 0u;
    }
    *reinterpret_cast<uint4 *>(smem + ch * 16) = make_uint4(u[0], u[1], u[2], u[3]);
  }
  __syncthreads();

  const unsigned char *tb = smem + lane * 16;
  const bool pad = PADK && KROWS * (S - 1) + hl >= a.wh;  // rows past the window: zero coefficients there
  for (int u = u0 + wave; u < u1; u += kGenWaves) {
    GFrag xf[S];
    {
      const int nv = cur.cols - x0 < 0 ? 0 : cur.cols - x0 > 8 ? 8 : cur.cols - x0;
      const uint4 m = *reinterpret_cast<const uint4 *>(masks + 4 * nv);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        uint32_t d[4] = {raw[s].x, raw[s].y, raw[s].z, raw[s].w};
        const int r = KROWS * s + hl;
        const int64_t over = cur.eoff + (int64_t)r * a.W + x0 - last;
        if (r < cur.rows && x0 < cur.cols && over > 0) {
          // within eight elements of the tensor's end: see gen_tail
#pragma unroll 1
          for (int k = (int)over; k > 0; --k)
#pragma unroll
            for (int i = 0; i < 4; ++i) d[i] = __builtin_amdgcn_alignbit(i < 3 ? d[i + 1] : 0u, d[i], 16);
        }
        xf[s] = __builtin_bit_cast(GFrag, make_uint4(d[0] & m.x, d[1] & m.y, d[2] & m.z, d[3] & m.w));
        asm volatile("" : "+v"(xf[s]));
      }
    }
    const Win w = cur;
    cur = window(u + kGenWaves);
    load(cur, raw);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t0 = 0; t0 < 2 * S; t0 += D::TP) {
      f32x4 acc[D::TP];
#pragma unroll
      for (int t = 0; t < D::TP; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int f = 0; f < D::NF; ++f) {
        const int q = f - (2 * S - 1);  // 2 k - t
        if (q > 2 * (S - 1) - t0 || q < 1 - t0 - D::TP) continue;
        const GFrag fr = *reinterpret_cast<const GFrag *>(tb + f * 1024);
#pragma unroll
        for (int k = 0; k < S; ++k) {
          const int t = 2 * k - q - t0;
          if (t < 0 || t >= D::TP) continue;
          if (PADK && k == S - 1) acc[t] = mma<Tag>(pad ? GFrag{0, 0, 0, 0, 0, 0, 0, 0} : fr, xf[k], acc[t]);
          else acc[t] = mma<Tag>(fr, xf[k], acc[t]);
        }
      }
      // window ln, positions 16 (t0 + t) + 4 g .. + 3
#pragma unroll
      for (int t = 0; t < D::TP; ++t) {
        const int r = 16 / RP * (t0 + t) + 4 * g / RP, xc = 4 * g % RP;
        const int nc = r < w.rows ? w.cols - xc : 0;
        const uint32_t a0 = pack2<Tag>(acc[t][0], acc[t][1]), a1 = pack2<Tag>(acc[t][2], acc[t][3]);
        E *q = y + w.eoff + (int64_t)r * a.W + xc;
        if (nc >= 4) {
          *reinterpret_cast<u32x2u *>(q) = u32x2u{a0, a1};
        } else if (nc > 0) {
          if (nc >= 2) *reinterpret_cast<u32u *>(q) = a0;
          if (nc & 1) q[nc - 1] = (E)((nc == 1 ? a0 : a1) & 0xffffu);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// ---------------------------------------------------- table gradient
// dT = the sums of X^T dY over windows along equal offsets.  K = windows: the
// position-major fragments of x and dy come from transposing reads of their
// window-major stages.  Wave (ph, pg) multiplies input tiles ph S .. + S - 1
// with a quarter of the output tiles; products of tile pairs with equal
// difference share an accumulator (S + NPO - 1 of them; 16-bit rows of eight
// have one per pair, at most three more).  At the end every wave sums the
// diagonals of its accumulators, and the waves' sums are added in order.
//
// Pads.  A pad position holds zero, and its product with an infinity or NaN
// is NaN, which must reach no entry of dT.  Pad columns have places of their
// own in every accumulator and are left out of the diagonals.  Pad rows,
// 16-bit: with rows of sixteen a tile is one row, and the one past a window of
// odd height (ODD) is not multiplied (by a constant of the kernel: tested in
// the loops it cost up to 12 %); with rows of eight half a tile can be a pad
// row, and a shared accumulator would add it to a row of the window, so each
// pair has its own and the pad half is left out as the pad columns are.
// float32: infinities and NaN are far rows, and only their products leave pad
// rows out.
//
// DX (16-bit): the fused backward.  The same stages feed the input gradient
// dY M^T as in the forward kernel (wave T holds the reversed table's
// fragments of output positions 32 T .. + 31), so dY is read once and x, dy and
// dx move in one launch; the rows of dX are stored a stage later.  Stages,
// accumulators and sums are the same with and without DX, and the products of
// dX those of the forward kernel: the same bits either way.
//
// What bounds it: 16-bit, memory and the copies' vector instructions (one
// 8-wave workgroup per compute unit, two stages of rows in flight, row
// addresses kept from load to store, columns masked from a table in LDS:
// B8 C96 100x167 w = 14 fused 38 -> 35 us, B64 C96 56x56 w = 7 33 -> 29; as
// separate launches 40 and 36, the four-wave kernels 69 and 46); float32, the
// matrix cores and the splitting of the rows, which one LDS buffer per stage
// leaves beside no products (B128 C192 28x28 w = 14: 85 us, float32 products
// 122).
template <class Tag, int RP, int S, bool DX, bool ODD>
struct GenDt {
  typedef GenCfg<Tag, RP, S> G;
  static_assert(!DX || Tag::W16, "fused backward: 16-bit");
  static_assert(!ODD || (Tag::W16 && RP == 16), "the last tile is a pad: 16-bit rows of sixteen");
  static constexpr int NTW = G::NT - ODD;          // tiles with rows of the window
  static constexpr int NPO = cdiv(NTW, 4);         // output tiles of a wave (at most)
  static constexpr int R = 16 / RP;                // window rows per tile
  // tile differences i - q + NPO - 1 of a wave's input and output tiles, its
  // accumulators, and the one of a pair
  static constexpr int NB = S + NPO - 1;
  static constexpr bool SHARE = R == 1 || !Tag::W16;
  static constexpr int NR = SHARE ? NB : S * NPO;
  __host__ __device__ static constexpr int at(int i, int q) { return SHARE ? i - q + NPO - 1 : i * NPO + q; }
  static constexpr int KST = G::CW / 32;           // K steps per stage
  static constexpr int NBUF = Tag::W16 ? 2 : 1;    // stages in LDS
  // float32: the smaller partial products in sums of their own where the
  // registers allow; elsewhere the five of a tile pair and 32 windows are summed
  // from zero, smallest first, and added once.  All six in one accumulator
  // rounded six times as often at the sum's full size, and always downwards:
  // the matrix cores cut the addends that are small beside the largest.  That
  // is also why the high parts' product is not among the five.  w = 14, error of
  // dT against 64 bits, one accumulator -> five apart (all six from zero; float32
  // products): B28 C36 98x98 6.0e-7 -> 1.9e-7 (4.0e-7; 4.0e-7), B1 C1 1500x1500
  // 8.4e-7 -> 2.7e-7 (1.1e-6; 6.3e-7).
  static constexpr bool LOWACC = !Tag::W16 && S <= 6;
  static constexpr int STAGE = 2 * G::XB;          // x and dy
  static constexpr int NBIN = R * R * 2 * RP;      // diagonals of a tile's R x R blocks, padded
  static constexpr int BT = 4;                     // tiles binned at a time
  static constexpr int SCR = kGenWaves * BT * kBinTile * 4;
  static constexpr int BINS = kGenWaves * NB * NBIN * 4;
  static constexpr int O_OFF = NBUF * STAGE;       // two result buffers
  static constexpr int END = O_OFF + (DX ? 2 * G::OB : 0);
  static constexpr int MASK_OFF = END > SCR + BINS ? END : SCR + BINS;
  static constexpr int FLAG_OFF = MASK_OFF + gen_mask_bytes<Tag, RP>();
  static constexpr size_t LDS = (size_t)FLAG_OFF + 16;
};

// First output tile of wave (ph, pg): quarters rounded down for one half of
// the input tiles and up for the other, so that the two waves of a SIMD (pg
// equal) have the same work together.
template <int NT>
__device__ __attribute__((always_inline)) inline int gen_dt_cut(int ph, int pg) {
  return (NT * pg + (ph ? 3 : 0)) >> 2;
}

template <class Tag, int RP, int S, bool DX, bool ODD>
__global__ __launch_bounds__(kGenThreads, 2) void gen_dt_kernel(
    const typename Tag::S *__restrict__ x, const typename Tag::S *__restrict__ dy,
    const typename Tag::S *__restrict__ tab, typename Tag::S *__restrict__ dxo, float *__restrict__ out, GenArgs a) {
  typedef GenCfg<Tag, RP, S> G;
  typedef GenDt<Tag, RP, S, DX, ODD> D;
  constexpr int NPO = D::NPO, NR = D::NR, NB = D::NB, R = D::R;
  extern __shared__ __align__(16) unsigned char smem[];
  int *flag = reinterpret_cast<int *>(smem + D::FLAG_OFF);
  uint32_t *masks = reinterpret_cast<uint32_t *>(smem + D::MASK_OFF);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 4, ln = lane & 15;
  const uint32_t bid = gen_block();
  const int64_t c = bid / (uint32_t)a.tiles_per_ch;
  if (c >= a.C) return;
  const int slab = (int)(bid - (uint32_t)c * (uint32_t)a.tiles_per_ch);
  const int s0 = slab * a.spw;
  const int nst = a.stages - s0 < a.spw ? a.stages - s0 : a.spw;
  const uint32_t n0 = (uint32_t)s0 * G::CW;
  const int v = gen_slot_window<G>(a, tid), hi = gen_slot_row<G>(a, tid);
  const int ph = wave >> 2, pg = wave & 3;
  const int po0 = gen_dt_cut<D::NTW>(ph, pg), po1 = gen_dt_cut<D::NTW>(ph, pg + 1);
  const int npo = po1 - po0;
  const bool xpad = ODD && ph == 1;  // this wave's last input tile is past the window

  auto row = [&](int s) __attribute__((always_inline)) -> GRow {
    return s < nst ? gen_row(a, c, n0 + s * G::CW + v, hi) : GRow{0, 0};
  };
  f32x4 acc[NR], lowacc[D::LOWACC ? NR : 1];
  auto &low = [&]() -> auto & {
    if constexpr (D::LOWACC) return lowacc;
    else return acc;
  }();
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = low[r] = f32x4{0.f, 0.f, 0.f, 0.f};
  // this thread's row of one stage, of x and dy
  struct Rows {
    GRow r;
    uint32_t x[G::ND], g[G::ND];
  };
  auto load = [&](int s, Rows &d) __attribute__((always_inline)) {
    d.r = row(s);
    gen_load<Tag, RP>(a.numel, x, d.r, d.x);
    gen_load<Tag, RP>(a.numel, dy, d.r, d.g);
  };
  auto write = [&](int s, unsigned char *st, Rows &d) __attribute__((always_inline)) {
    gen_tail<Tag, RP>(a.numel, d.r, d.x);
    gen_tail<Tag, RP>(a.numel, d.r, d.g);
    gen_mask<Tag, RP>(masks, d.r.cols, d.x);
    gen_mask<Tag, RP>(masks, d.r.cols, d.g);
#pragma unroll
    for (int i = 0; i < G::ND; ++i) asm volatile("" : "+v"(d.x[i]), "+v"(d.g[i]));  // (the rows arrive here, on every path)
    if (hi < G::KR) {
      const bool fx = gen_write<Tag, RP, S, false>(st, v, hi, d.x), fg = gen_write<Tag, RP, S, false>(st + G::XB, v, hi, d.g);
      if (fx || fg) flag[s & 1] = s;
    }
  };
  auto products = [&](const unsigned char *st) __attribute__((always_inline)) {
    if constexpr (Tag::W16) {
#pragma unroll
      for (int ks = 0; ks < D::KST; ++ks) {
        const unsigned char *xt = st + ks * 32 * G::LDSW * 2, *gt = xt + G::XB;
        GFrag bf[NPO];
#pragma unroll
        for (int q = 0; q < NPO; ++q) bf[q] = dt_frag16<G::LDSW>(gt, q < npo ? po0 + q : po0, lane);
#pragma unroll
        for (int i = 0; i < S; ++i) {
          if (i == S - 1 && xpad) continue;
          const GFrag af = dt_frag16<G::LDSW>(xt, ph * S + i, lane);
#pragma unroll
          for (int q = 0; q < NPO; ++q)
            if (q < npo) acc[D::at(i, q)] = mma<Tag>(af, bf[q], acc[D::at(i, q)]);
        }
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < D::KST; ++ks) {
        const unsigned char *xt = st + ks * 32 * G::LDSW * 2, *gt = xt + G::XB;
        GFrag bf[3][NPO], af[2][3];
#pragma unroll
        for (int q = 0; q < NPO; ++q)
#pragma unroll
          for (int p = 0; p < 3; ++p)
            bf[p][q] = dt_frag16<G::LDSW>(gt + p * G::PLANE, q < npo ? po0 + q : po0, lane);
#pragma unroll
        for (int p = 0; p < 3; ++p) af[0][p] = dt_frag16<G::LDSW>(xt + p * G::PLANE, ph * S, lane);
#pragma unroll
        for (int i = 0; i < S; ++i) {
          // (the next tile's fragments are read while this one is multiplied)
          if (i + 1 < S) {
#pragma unroll
            for (int p = 0; p < 3; ++p) af[(i + 1) & 1][p] = dt_frag16<G::LDSW>(xt + p * G::PLANE, ph * S + i + 1, lane);
          }
          __builtin_amdgcn_sched_barrier(0);
          const GFrag(&f)[3] = af[i & 1];
#define WBMM_DT_PART(PA, PB, ACC) \
  _Pragma("unroll") for (int q = 0; q < NPO; ++q) if (q < npo) ACC = mma_bf16(f[PA], bf[PB][q], ACC);
          if constexpr (D::LOWACC) {
            WBMM_DT_PART(2, 0, low[D::at(i, q)])
            WBMM_DT_PART(0, 2, low[D::at(i, q)])
            WBMM_DT_PART(1, 1, low[D::at(i, q)])
            WBMM_DT_PART(1, 0, low[D::at(i, q)])
            WBMM_DT_PART(0, 1, low[D::at(i, q)])
            WBMM_DT_PART(0, 0, acc[D::at(i, q)])
          } else {
#pragma unroll
            for (int q = 0; q < NPO; ++q) {
              if (q >= npo) continue;
              f32x4 t = mma_bf16(f[2], bf[0][q], f32x4{0.f, 0.f, 0.f, 0.f});
              t = mma_bf16(f[0], bf[2][q], t);
              t = mma_bf16(f[1], bf[1][q], t);
              t = mma_bf16(f[1], bf[0][q], t);
              t = mma_bf16(f[0], bf[1][q], t);
              f32x4 &r = acc[D::at(i, q)];
              r = mma_bf16(f[0], bf[0][q], r);
#pragma unroll
              for (int e = 0; e < 4; ++e) r[e] += t[e];
            }
          }
#undef WBMM_DT_PART
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };

  // float32 products of a stage with far rows: its rows as they are in the
  // place of the planes, window-major
  constexpr int FP = G::KP + 8;  // pitch
  static_assert(Tag::W16 || 2 * G::CW * FP * 4 <= D::STAGE, "float32 rows within the planes");
  // (loaded again: kept from the planes' writes on, they cost the usual path
  // registers)
  auto far_write = [&](int s) __attribute__((always_inline)) {
    int vf = v, hf = hi;
    asm volatile("" : "+v"(vf), "+v"(hf));  // (what follows from them stays in this branch)
    const GRow r = gen_row(a, c, n0 + s * G::CW + vf, hf);
#pragma unroll 1
    for (int k = 0; k < 2; ++k) {
      uint32_t d[G::ND];
      gen_load<Tag, RP>(a.numel, k ? dy : x, r, d);
      gen_tail<Tag, RP>(a.numel, r, d);
      gen_mask<Tag, RP>(masks, r.cols, d);
      float *p = reinterpret_cast<float *>(smem) + (k * G::CW + vf) * FP + hf * RP;
      if (hf < G::KR) {
#pragma unroll
        for (int i = 0; i < G::ND; i += 4)
          *reinterpret_cast<uint4 *>(p + i) = make_uint4(d[i], d[i + 1], d[i + 2], d[i + 3]);
      }
    }
  };
  auto far_products = [&]() __attribute__((always_inline)) {
    const float *px = reinterpret_cast<const float *>(smem) + g * FP + ln, *pg = px + G::CW * FP;
    // rows of sixteen: no products of a tile past the window
    const bool xcut = R == 1 && ph * S + S - 1 >= a.wh;
    const int ocut = (R == 1 && po1 > a.wh ? a.wh : po1) - po0;
    // rows of eight: the pairs apart, without their pad rows
    f32x4 t[R == 1 ? 1 : S * NPO];
    if constexpr (R == 2) {
#pragma unroll
      for (int k = 0; k < S * NPO; ++k) t[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll 1
    for (int w = 0; w < G::CW; w += 4, px += 4 * FP, pg += 4 * FP) {
      float av[S], bv[NPO];
#pragma unroll
      for (int q = 0; q < NPO; ++q) bv[q] = pg[16 * (q < npo ? po0 + q : 0)];
#pragma unroll
      for (int i = 0; i < S; ++i) av[i] = px[16 * (ph * S + i)];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < S; ++i) {
        if (i == S - 1 && xcut) continue;
#pragma unroll
        for (int q = 0; q < NPO; ++q) {
          if (q >= ocut) continue;
          f32x4 &r = R == 1 ? acc[D::at(i, q)] : t[R == 1 ? 0 : i * NPO + q];
          r = mma<TagF32>(av[i], bv[q], r);
        }
      }
    }
    if constexpr (R == 2) {
#pragma unroll
      for (int i = 0; i < S; ++i)
#pragma unroll
        for (int q = 0; q < NPO; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const bool ok = 2 * (ph * S + i) + (4 * g + e) / RP < a.wh && 2 * (po0 + q) + ln / RP < a.wh;
            acc[D::at(i, q)][e] += ok ? t[i * NPO + q][e] : 0.f;
          }
    }
  };

  // ---- input gradient: the reversed table's fragments of tile pair T, the
  // products of stage s and the rows of a finished stage out
  const int T = wave % S, sg = wave / S;
  GFrag fr[1][2][DX ? S : 1];
  unsigned char *obuf = smem + D::O_OFF;
  auto dx_products = [&](int s, const unsigned char *st) __attribute__((always_inline)) {
    if constexpr (DX) {
      if (sg >= G::NG) return;
      const unsigned char *gp = st + G::XB + ((16 * sg + ln) * G::LDSW + 8 * g) * 2;
      typename Tag::S *o = reinterpret_cast<typename Tag::S *>(obuf + (s & 1) * G::OB) + (16 * sg + ln) * G::OP + 32 * T + 4 * g;
#pragma unroll
      for (int j = 0; j < G::SPW; ++j) {
        f32x4 r[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int k = 0; k < S; ++k) {
          const GFrag gf = *reinterpret_cast<const GFrag *>(gp + 16 * j * G::NG * G::LDSW * 2 + 64 * k);
#pragma unroll
          for (int h = 0; h < 2; ++h) r[h] = mma<Tag>(fr[0][h][k], gf, r[h]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h)
          *reinterpret_cast<uint2 *>(o + 16 * j * G::NG * G::OP + 16 * h) =
              uint2{pack2<Tag>(r[h][0], r[h][1]), pack2<Tag>(r[h][2], r[h][3])};
      }
    }
  };
  auto dx_store = [&](int s, const GRow &r) __attribute__((always_inline)) {
    if constexpr (DX) {
      if (r.cols > 0) {
        const unsigned char *ob = obuf + (s & 1) * G::OB + (v * G::OP + hi * RP) * Tag::ES;
        uint32_t o[G::ND];
#pragma unroll
        for (int i = 0; i < G::ND; i += 4) {
          const uint4 u = *reinterpret_cast<const uint4 *>(ob + 4 * i);
          o[i] = u.x; o[i + 1] = u.y; o[i + 2] = u.z; o[i + 3] = u.w;
        }
        gen_store<Tag, RP>(dxo, r, o);
      }
    }
  };

  const int K1 = 2 * a.ww - 1, K2 = K1 * (2 * a.wh - 1);
  typename Tag::S tv[2] = {};
  if constexpr (DX) {
    // (the table first, ahead of the rows; K2 <= 961)
    const typename Tag::S *tc = tab + c * K2;
#pragma unroll
    for (int i = 0; i < 2; ++i) tv[i] = tc[K2 - 1 - (tid + i * kGenThreads < K2 ? tid + i * kGenThreads : K2 - 1)];
    __builtin_amdgcn_sched_barrier(0);
  }
  Rows d0, d1;
  load(0, d0);
  if constexpr (D::NBUF == 2) load(1, d1);
  __builtin_amdgcn_sched_barrier(0);
  if (tid < 2) flag[tid] = -1;
  gen_mask_table<Tag, RP>(masks, tid);
  if constexpr (DX) {
    typename Tag::S *Ts = reinterpret_cast<typename Tag::S *>(obuf);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int k = tid + i * kGenThreads;
      if (k < K2 + 10) Ts[k] = k < K2 ? tv[i] : (typename Tag::S)0;
    }
    __syncthreads();
    gen_build_tb<Tag, RP, S>(a, Ts, smem + D::STAGE, nullptr, tid);
  }
  __syncthreads();
  if constexpr (D::NBUF == 2) {
    if constexpr (DX) gen_frags_tb<Tag, RP, S>(a, smem + D::STAGE, T, lane, fr);
    GRow rprev = {0, 0}, rcur = d0.r;
    write(0, smem, d0);
    load(2, d0);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // stage s + 1 (in d) to LDS, the rows of stage s - 1 out, stage s + 3 into d
    auto stage = [&](int s, Rows &d) __attribute__((always_inline)) {
      const unsigned char *st = smem + (s & 1) * D::STAGE;
      products(st);
      dx_products(s, st);
      const GRow rnext = d.r;
      write(s + 1, smem + ((s + 1) & 1) * D::STAGE, d);
      dx_store(s - 1, rprev);
      load(s + 3, d);
      rprev = rcur;
      rcur = rnext;
      __syncthreads();
    };
    for (int s = 0; s < nst; s += 2) {
      stage(s, d1);
      if (s + 1 >= nst) break;
      stage(s + 1, d0);
    }
    dx_store(nst - 1, rprev);
    if constexpr (DX) __syncthreads();  // (the scratch below reaches the result buffers)
  } else {
    for (int s = 0; s < nst; ++s) {
      write(s, smem, d0);
      __syncthreads();
      const int far = flag[s & 1];
      load(s + 1, d0);
      if (__builtin_expect(!Tag::W16 && __builtin_amdgcn_readfirstlane(far) == s, 0)) {
        far_write(s);
        __syncthreads();
        far_products();
      } else {
        products(smem);
      }
      __syncthreads();
    }
  }

  // ---- diagonals of the wave's tiles, each R x R blocks of RP x RP: a block
  // is written skewed, element (xi, xo) at column (xo - xi) mod RP of row xi,
  // so that column s holds diagonal dw = -s above row RP - s and RP - s below;
  // one lane sums one column of one block.  Pad columns, and with rows of
  // eight pad rows, are written as zero, whatever their products were.
  float *scr = reinterpret_cast<float *>(smem) + wave * D::BT * kBinTile;
  float *bins = reinterpret_cast<float *>(smem + D::SCR);
  float *mine = bins + wave * NB * D::NBIN;
#pragma unroll
  for (int r0 = 0; r0 < NB; r0 += D::BT) {
    wave_lds_sync();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int rr = 4 * g + e;
      const bool cols = (rr & (RP - 1)) < a.ww && (ln & (RP - 1)) < a.ww;
      float *p = scr + rr * 17 + (ln & ~(RP - 1)) + ((ln - rr) & (RP - 1));
#pragma unroll
      for (int j = 0; j < D::BT; ++j) {
        if (r0 + j >= NB) continue;
        float t = 0.f;
        if constexpr (D::SHARE) {
          t = acc[r0 + j][e];
          if constexpr (D::LOWACC) t += low[r0 + j][e];
        } else {
#pragma unroll
          for (int q = 0; q < NPO; ++q) {
            const int i = r0 + j - (NPO - 1) + q;
            if (i < 0 || i >= S) continue;
            if (2 * (ph * S + i) + rr / RP < a.wh && 2 * (po0 + q) + ln / RP < a.wh) t += acc[D::at(i, q)][e];
          }
        }
        p[j * kBinTile] = cols ? t : 0.f;
      }
    }
    wave_lds_sync();
    constexpr int TPT = R * R * RP;  // columns of a tile
#pragma unroll
    for (int k = 0; k < D::BT * TPT / 64; ++k) {
      const int t = lane + 64 * k;
      const int j = t / TPT, b = t % TPT / RP, sft = t % RP;  // tile, block (ra R + rb), column
      if (r0 + j < NB) {
        const float *p = scr + j * kBinTile + b / R * RP * 17 + b % R * RP + sft;
        float lo = 0.f, up = 0.f;
#pragma unroll
        for (int xi = 0; xi < RP; ++xi) {
          const float f = p[xi * 17];
          const bool below = xi + sft >= RP;
          lo += below ? 0.f : f;
          up += below ? f : 0.f;
        }
        float *o = mine + (r0 + j) * D::NBIN + b * 2 * RP + RP - 1;
        o[-sft] = lo;
        if (sft > 0) o[RP - sft] = up;
      }
    }
  }
  __syncthreads();
  // ---- entry (dh, dw): the waves' diagonals of the tiles P = pi - po and
  // blocks with dh = P R + ra - rb, in wave order
  float *o = out + ((int64_t)slab * a.C + c) * K2;
  for (int k = tid; k < K2; k += kGenThreads) {
    const int dh = k / K1 - (a.wh - 1), dw = k - k / K1 * K1 - (a.ww - 1);
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < kGenWaves; ++w) {
      const int base = gen_dt_cut<D::NTW>(w >> 2, w & 3) - (w >> 2) * S + NPO - 1;
#pragma unroll
      for (int b = 0; b < R * R; ++b) {
        const int pr = dh - (b / R - b % R);  // P R
        if (R == 2 && (pr & 1)) continue;
        const int r = pr / R + base;
        if (r >= 0 && r < NB) sum += bins[(w * NB + r) * D::NBIN + b * 2 * RP + RP - 1 + dw];
      }
    }
    o[k] = sum;
  }
}

}  // namespace wbmm
