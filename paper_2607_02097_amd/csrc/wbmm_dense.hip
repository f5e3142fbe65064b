// Cached-matrix (dense) form of WBMM for any window w_h x w_w with
// d = w_h w_w <= 256 (Alg. 1 with the matrix built once, eq. index_select):
//   build:    M_c[i, j] = T[c, I(i, j)]                    (matrix per channel)
//   gradient: dM_c = sum over windows of X_window^T dY_window   (float32)
//   bin:      dT[c, k] = sum of dM_c[i, j] over I(i, j) = k (fixed order)
// Positions are row-major inside a window, p = h * w_w + x.  M is an
// arbitrary dense matrix here (the table form's Toeplitz structure is not
// used), so rectangular windows, fused matrices and any cached M share one
// path.  The kernels are generic over the window (runtime sizes) and
// instantiated once per dtype.  The products X_window M_c and X_window M_c^T
// are the general kernels' (wbmm_gen.h).
#include "wbmm_kernels.h"

namespace wbmm {

struct DenseArgs {
  int64_t B, C, H, W;
  int wh, ww, d;
  int NH, NW;
  int64_t N;  // windows per channel
};

// Element offset of window position p of window n (channel c), or -1 when
// the position lies in the zero padding.
__device__ __attribute__((always_inline)) inline int64_t dense_offset(const DenseArgs &a, int64_t c, int64_t n, int p) {
  const int64_t nhw = (int64_t)a.NH * a.NW;
  const int64_t b = n / nhw;
  const int64_t r = n - b * nhw;
  const int64_t wy = r / a.NW, wx = r - wy * a.NW;
  const int h = p / a.ww, x = p - (p / a.ww) * a.ww;
  const int64_t gh = wy * a.wh + h, gw = wx * a.ww + x;
  if (gh >= a.H || gw >= a.W) return -1;
  return ((b * a.C + c) * a.H + gh) * a.W + gw;
}

// M_c[i, j] = T[c, I(i, j)], i the input and j the output position.
template <class Tag>
__global__ __launch_bounds__(256) void dense_build_kernel(const typename Tag::S *__restrict__ t,
                                                          typename Tag::S *__restrict__ m, int64_t C, int wh,
                                                          int ww) {
  const int d = wh * ww;
  const int64_t k1 = 2 * ww - 1, k2 = (int64_t)(2 * wh - 1) * k1;
  const int64_t total = C * d * d;
  for (int64_t e = blockIdx.x * 256LL + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t c = e / ((int64_t)d * d);
    const int r = (int)(e - c * d * d);
    const int i = r / d, j = r - (r / d) * d;
    const int hi = i / ww, xi = i - hi * ww, ho = j / ww, xo = j - ho * ww;
    m[e] = t[c * k2 + (hi - ho + wh - 1) * k1 + (xi - xo + ww - 1)];
  }
}

// dM_c = sum over windows of X^T dY (float32).  One workgroup = (channel,
// 64 x 64 block of dM); K = the channel's windows, in stages of 32 (16-bit)
// or 16 (float32) windows staged window-major; each wave owns one 16-row
// strip of the block (four 16 x 16 accumulators).
template <class Tag>
struct DenseDmCfg {
  static constexpr int CW = Tag::W16 ? 32 : 16;
  static constexpr int BP = 64;                                        // block side
  static constexpr int LDSP = Tag::W16 ? BP + 8 : BP + 16;             // pitch (elements)
  static constexpr size_t LDS = (size_t)2 * CW * LDSP * Tag::ES;
};

template <class Tag>
__global__ __launch_bounds__(256) void dense_dm_kernel(const typename Tag::S *__restrict__ x,
                                                       const typename Tag::S *__restrict__ dy,
                                                       float *__restrict__ dm, DenseArgs a, int nblk) {
  typedef typename Tag::S S;
  typedef typename Tag::Frag Frag;
  typedef DenseDmCfg<Tag> G;
  extern __shared__ __align__(16) unsigned char smem[];
  S *Xs = reinterpret_cast<S *>(smem);
  S *Gs = Xs + G::CW * G::LDSP;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, ln = lane & 15;
  const int64_t c = blockIdx.x / (nblk * nblk);
  const int blk = (int)(blockIdx.x - c * nblk * nblk);
  const int i0 = (blk / nblk) * G::BP, j0 = (blk - (blk / nblk) * nblk) * G::BP;
  const int d = a.d;

  f32x4 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int64_t n0 = 0; n0 < a.N; n0 += G::CW) {
    __syncthreads();  // previous stage consumed
    for (int e = tid; e < 2 * G::CW * G::BP; e += 256) {
      const int tens = e / (G::CW * G::BP);
      const int r = e - tens * (G::CW * G::BP);
      const int v = r / G::BP, pp = r - (r / G::BP) * G::BP;
      const int p = (tens ? j0 : i0) + pp;
      S val = (S)0;
      if (p < d && n0 + v < a.N) {
        const int64_t o = dense_offset(a, c, n0 + v, p);
        if (o >= 0) val = (tens ? dy : x)[o];
      }
      (tens ? Gs : Xs)[v * G::LDSP + pp] = val;
    }
    __syncthreads();
    if constexpr (Tag::W16) {
      const Frag af = dt_frag16<G::LDSP>(reinterpret_cast<const unsigned char *>(Xs), wave, lane);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        acc[q] = mma<Tag>(af, dt_frag16<G::LDSP>(reinterpret_cast<const unsigned char *>(Gs), q, lane), acc[q]);
    } else {
#pragma unroll
      for (int ks = 0; ks < G::CW / 4; ++ks) {
        const float af = Xs[(4 * ks + g) * G::LDSP + 16 * wave + ln];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = mma<Tag>(af, Gs[(4 * ks + g) * G::LDSP + 16 * q + ln], acc[q]);
      }
    }
  }
  float *mc = dm + c * (int64_t)d * d;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int j = j0 + 16 * q + ln;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * wave + 4 * g + r;
      if (i < d && j < d) mc[(int64_t)i * d + j] = acc[q][r];
    }
  }
}

// dT[c, k] = sum over the pairs (i, j) with I(i, j) = k of dM_c[i, j], in a
// fixed order (output rows, then columns).
__global__ __launch_bounds__(256) void dense_bin_kernel(const float *__restrict__ dm, float *__restrict__ dt,
                                                        int64_t C, int wh, int ww) {
  const int d = wh * ww;
  const int k1 = 2 * ww - 1, k2 = (2 * wh - 1) * k1;
  const int64_t e = blockIdx.x * 256LL + threadIdx.x;
  if (e >= C * k2) return;
  const int64_t c = e / k2;
  const int k = (int)(e - c * k2);
  const int dh = k / k1 - (wh - 1), dw = k - (k / k1) * k1 - (ww - 1);
  const float *mc = dm + c * (int64_t)d * d;
  float s = 0.f;
  for (int ho = dh < 0 ? -dh : 0; ho < (dh > 0 ? wh - dh : wh); ++ho)
    for (int xo = dw < 0 ? -dw : 0; xo < (dw > 0 ? ww - dw : ww); ++xo)
      s += mc[(int64_t)((ho + dh) * ww + xo + dw) * d + ho * ww + xo];
  dt[e] = s;
}

// ------------------------------------------------------------ launchers

static DenseArgs dense_args(const Geom &g, int wh, int ww) {
  DenseArgs a;
  a.B = g.B; a.C = g.C; a.H = g.H; a.W = g.W;
  a.wh = wh; a.ww = ww; a.d = wh * ww;
  a.NH = (int)((g.H + wh - 1) / wh);
  a.NW = (int)((g.W + ww - 1) / ww);
  a.N = g.B * (int64_t)a.NH * a.NW;
  return a;
}

template <class Tag>
static hipError_t run_dense_build(const void *t, void *m, int64_t C, int wh, int ww, hipStream_t st) {
  const int64_t total = C * (int64_t)(wh * ww) * (wh * ww);
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  dense_build_kernel<Tag><<<dim3((unsigned)blocks), dim3(256), 0, st>>>((const typename Tag::S *)t,
                                                                         (typename Tag::S *)m, C, wh, ww);
  return hipGetLastError();
}

template <class Tag>
static hipError_t run_dense_dm(const void *x, const void *dy, float *dm, const Geom &g, int wh, int ww,
                               hipStream_t st) {
  typedef DenseDmCfg<Tag> G;
  DenseArgs a = dense_args(g, wh, ww);
  const int nblk = (a.d + G::BP - 1) / G::BP;
  typedef typename Tag::S S;
  dense_dm_kernel<Tag><<<dim3((unsigned)(g.C * nblk * nblk)), dim3(256), G::LDS, st>>>(
      (const S *)x, (const S *)dy, dm, a, nblk);
  return hipGetLastError();
}

hipError_t launch_dense_build(Dt dt, const void *t, void *m, int64_t C, int wh, int ww, hipStream_t st) {
  switch (dt) {
    case Dt::F32: return run_dense_build<TagF32>(t, m, C, wh, ww, st);
    case Dt::BF16: return run_dense_build<TagBF16>(t, m, C, wh, ww, st);
    case Dt::F16: return run_dense_build<TagF16>(t, m, C, wh, ww, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dense_backward_matrix(Dt dt, const void *x, const void *dy, float *dm, const Geom &g, int wh,
                                        int ww, hipStream_t st) {
  switch (dt) {
    case Dt::F32: return run_dense_dm<TagF32>(x, dy, dm, g, wh, ww, st);
    case Dt::BF16: return run_dense_dm<TagBF16>(x, dy, dm, g, wh, ww, st);
    case Dt::F16: return run_dense_dm<TagF16>(x, dy, dm, g, wh, ww, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_dense_bin(const float *dm, float *dt, int64_t C, int wh, int ww, hipStream_t st) {
  const int64_t total = C * (int64_t)(2 * wh - 1) * (2 * ww - 1);
  dense_bin_kernel<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st>>>(dm, dt, C, wh, ww);
  return hipGetLastError();
}

}  // namespace wbmm
