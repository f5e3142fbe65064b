// One instantiation unit of the general kernels (wbmm_gen.h): one dtype,
// every row pitch and K-step count.
// Compiled with -DWBMM_INST_TAG=<TagF32|TagBF16|TagF16>.
#include "wbmm_gen.h"
#include "wbmm_plan.h"

namespace wbmm {

static GenArgs gen_args(const Geom &g, int wh, int ww) {
  GenArgs a;
  a.C = g.C; a.H = g.H; a.W = g.W;
  a.hw = g.H * g.W;
  a.chw = g.C * a.hw;
  a.numel = g.B * a.chw;
  const int64_t nh = cdiv64(g.H, wh), nw = cdiv64(g.W, ww);
  a.NW = (uint32_t)nw;
  a.NHW = (uint32_t)(nh * nw);
  a.dnw = fast_div(a.NW);
  a.dnhw = fast_div(a.NHW);
  a.N = (uint32_t)(g.B * nh * nw);
  a.wh = wh; a.ww = ww;
  a.stages = 0; a.spw = 0; a.tiles_per_ch = 0; a.src = 0; a.lgg = 0;
  return a;
}

// Neighbouring windows whose rows neighbouring lanes move: see gen_slot_window.
template <class G>
static void gen_lanes(GenArgs &a) {
  a.lgg = 0;
  while ((2 << a.lgg) <= (int64_t)a.NW && (2 << a.lgg) <= G::CW) ++a.lgg;
}

template <class Tag, int RP, int S>
static hipError_t gen_fwd(const void *x, const void *coef, void *y, const Geom &g, int wh, int ww, int src,
                          hipStream_t st) {
  typedef typename Tag::S E;
  typedef GenCfg<Tag, RP, S> G;
  GenArgs a = gen_args(g, wh, ww);
  a.src = src;
  const int ncu = compute_units();
  if constexpr (!Tag::W16) {
    // float32 from the table: one unit of 16 windows per wave where they fill
    // half of the chip's 2048 waves (w = 14, us: B16 C96 56x56, 1536 units, 24.8
    // -> 22.3; B128 C256 56x56 295 -> 275; w = 9 B128 C256 36x36 187 -> 138; but
    // B1 C64 75x100, 192 units, 10.2 against 13.7); rows of eight always (w = 7
    // B1 C64 75x100 6.5 -> 5.7, B64 C96 56x56 48.8 -> 35.0)
    if (src < kSrcMat && (RP == 8 || g.C * cdiv64(a.N, 16) >= 1024)) {
      typedef GenDirect<RP, S> D;
      a.stages = (int)cdiv64(a.N, 16 * kGenWaves);
      gen_plan(g.C, a.stages, ncu > 0 ? ncu : 256, 1.0, 1 << 20, &a.spw, &a.tiles_per_ch);
      gen_direct_kernel<RP, S><<<gen_grid(g.C * a.tiles_per_ch), dim3(kGenThreads), D::LDS, st>>>(
          (const float *)x, (const float *)coef, (float *)y, a);
      return hipGetLastError();
    }
  }
  if constexpr (Tag::W16) {
    // 16-bit from the table: the same line of half of the chip's waves (bf16,
    // w = 14, us: B4 C96 75x124, 1344 units, 9.5 -> 8.7; B1 C64 75x100, 192 units,
    // 5.0 against 6.5; 5 x 9 windows B4 C64 45x63, 1024 units, 4.8 -> 4.7)
    if (src < kSrcMat && g.C * cdiv64(a.N, 16) >= 1024) {
      typedef GenDirect16<RP, S> D;
      a.stages = (int)cdiv64(a.N, 16 * kGenWaves);
      gen_plan(g.C, a.stages, (ncu > 0 ? ncu : 256) * D::WGS, 1.0, 1 << 20, &a.spw, &a.tiles_per_ch);
      const dim3 dgrid = gen_grid(g.C * a.tiles_per_ch);
      if (wh % (32 / RP))
        gen_direct16_kernel<Tag, RP, S, true><<<dgrid, dim3(kGenThreads), D::LDS, st>>>((const E *)x, (const E *)coef, (E *)y, a);
      else
        gen_direct16_kernel<Tag, RP, S, false><<<dgrid, dim3(kGenThreads), D::LDS, st>>>((const E *)x, (const E *)coef, (E *)y, a);
      return hipGetLastError();
    }
  }
  a.stages = (int)cdiv64(a.N, G::CW);
  gen_lanes<G>(a);
  const int wgs = src >= kSrcMat ? GenFwd<Tag, RP, S, true>::WGS : GenFwd<Tag, RP, S, false>::WGS;
  gen_plan(g.C, a.stages, (int64_t)(ncu > 0 ? ncu : 256) * wgs, 1.5, 1 << 20, &a.spw, &a.tiles_per_ch);
  const dim3 grid = gen_grid(g.C * a.tiles_per_ch), block(kGenThreads);
  constexpr size_t ltab = GenFwd<Tag, RP, S, false>::LDS, lmat = GenFwd<Tag, RP, S, true>::LDS;
  static_assert(ltab <= 160 * 1024 && lmat <= 160 * 1024, "workgroup LDS above the 160 KB of a compute unit");
  if (src >= kSrcMat)
    gen_fwd_kernel<Tag, RP, S, true><<<grid, block, lmat, st>>>((const E *)x, (const E *)coef, (E *)y, a);
  else if constexpr (Tag::W16 || RP == 16)
    gen_fwd_kernel<Tag, RP, S, false><<<grid, block, ltab, st>>>((const E *)x, (const E *)coef, (E *)y, a);
  return hipGetLastError();
}

// Tensors or matrices of fewer than 16 elements, shorter than the row loads
// of the general kernels: one thread per output.
template <class Tag>
__global__ __launch_bounds__(256) void gen_small_kernel(const typename Tag::S *__restrict__ x,
                                                        const typename Tag::S *__restrict__ coef,
                                                        typename Tag::S *__restrict__ y, GenArgs a) {
  for (int64_t e = blockIdx.x * 256LL + threadIdx.x; e < a.numel; e += (int64_t)gridDim.x * 256) {
    const int64_t gx = e % a.W, gy = e / a.W % a.H, c = e / a.hw % a.C;
    const int64_t wy = gy / a.wh, wx = gx / a.ww;
    const typename Tag::S *plane = x + e / a.hw * a.hw;
    float s = 0.f;
    for (int hi = 0; hi < a.wh && wy * a.wh + hi < a.H; ++hi)
      for (int xi = 0; xi < a.ww && wx * a.ww + xi < a.W; ++xi) {
        const typename Tag::S m = coef[gen_coef<Tag>(a, c, hi, xi, (int)(gy - wy * a.wh), (int)(gx - wx * a.ww))];
        const typename Tag::S v = plane[(wy * a.wh + hi) * a.W + wx * a.ww + xi];
        if constexpr (Tag::W16) s += to_f32<Tag>(v) * to_f32<Tag>(m);
        else s += v * m;
      }
    if constexpr (Tag::W16) y[e] = (u16)(pack2<Tag>(s, 0.f) & 0xffffu);
    else y[e] = s;
  }
}

template <class Tag>
static hipError_t run_gen_fwd(const void *x, const void *coef, void *y, const Geom &g, int wh, int ww, int src,
                              hipStream_t st) {
  const int64_t d = (int64_t)wh * ww;
  GenArgs a = gen_args(g, wh, ww);
  if (a.numel < 16 || (src >= kSrcMat && g.C * d * d < 16)) {
    typedef typename Tag::S E;
    a.src = src;
    const int64_t blocks = cdiv64(a.numel, 256);
    gen_small_kernel<Tag><<<dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, st>>>(
        (const E *)x, (const E *)coef, (E *)y, a);
    return hipGetLastError();
  }
  if (ww <= 8) {
    switch ((wh + 3) / 4) {
      case 1: return gen_fwd<Tag, 8, 1>(x, coef, y, g, wh, ww, src, st);
      case 2: return gen_fwd<Tag, 8, 2>(x, coef, y, g, wh, ww, src, st);
      case 3: return gen_fwd<Tag, 8, 3>(x, coef, y, g, wh, ww, src, st);
      case 4: return gen_fwd<Tag, 8, 4>(x, coef, y, g, wh, ww, src, st);
    }
  } else {
    switch ((wh + 1) / 2) {
      case 1: return gen_fwd<Tag, 16, 1>(x, coef, y, g, wh, ww, src, st);
      case 2: return gen_fwd<Tag, 16, 2>(x, coef, y, g, wh, ww, src, st);
      case 3: return gen_fwd<Tag, 16, 3>(x, coef, y, g, wh, ww, src, st);
      case 4: return gen_fwd<Tag, 16, 4>(x, coef, y, g, wh, ww, src, st);
      case 5: return gen_fwd<Tag, 16, 5>(x, coef, y, g, wh, ww, src, st);
      case 6: return gen_fwd<Tag, 16, 6>(x, coef, y, g, wh, ww, src, st);
      case 7: return gen_fwd<Tag, 16, 7>(x, coef, y, g, wh, ww, src, st);
      case 8: return gen_fwd<Tag, 16, 8>(x, coef, y, g, wh, ww, src, st);
    }
  }
  return hipErrorInvalidValue;
}

// Table gradient, with dx (16-bit) the fused backward: at most max_slabs
// partial tables per channel, which the caller's workspace holds (one: dt is
// written directly); the partials are summed by the sum kernel behind it.
// One workgroup per compute unit is planned for, with or without dx, so that
// both have the same slabs.
template <class Tag, int RP, int S>
static hipError_t gen_dt(const void *x, const void *dy, const void *t, void *dx, float *dt, float *ws, const Geom &g,
                         int wh, int ww, int64_t max_slabs, hipStream_t st) {
  typedef typename Tag::S E;
  typedef GenCfg<Tag, RP, S> G;
  GenArgs a = gen_args(g, wh, ww);
  a.stages = (int)cdiv64(a.N, G::CW);
  gen_lanes<G>(a);
  const int ncu = compute_units();
  gen_plan(g.C, a.stages, ncu > 0 ? ncu : 256, 3.0, max_slabs, &a.spw, &a.tiles_per_ch);
  float *out = a.tiles_per_ch > 1 ? ws : dt;
  const dim3 grid = gen_grid(g.C * a.tiles_per_ch), block(kGenThreads);
  auto launch = [&](auto odd) {
    constexpr bool ODD = decltype(odd)::value;
    constexpr size_t lds = GenDt<Tag, RP, S, false, ODD>::LDS, flds = GenDt<Tag, RP, S, Tag::W16, ODD>::LDS;
    static_assert(lds <= 160 * 1024 && flds <= 160 * 1024, "workgroup LDS above the 160 KB of a compute unit");
    if (dx)
      gen_dt_kernel<Tag, RP, S, Tag::W16, ODD><<<grid, block, flds, st>>>((const E *)x, (const E *)dy, (const E *)t,
                                                                          (E *)dx, out, a);
    else
      gen_dt_kernel<Tag, RP, S, false, ODD><<<grid, block, lds, st>>>((const E *)x, (const E *)dy, nullptr, nullptr,
                                                                      out, a);
  };
  if constexpr (Tag::W16 && RP == 16) {
    if (wh & 1) launch(std::true_type{});
    else launch(std::false_type{});
  } else {
    launch(std::false_type{});
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.tiles_per_ch <= 1) return e;
  return launch_dt_sum(ws, dt, g.C * (int64_t)(2 * wh - 1) * (2 * ww - 1), nullptr, nullptr, 0, a.tiles_per_ch, st);
}

// Table gradient of a tensor of fewer than 16 elements: one thread per entry.
template <class Tag>
__global__ __launch_bounds__(256) void gen_small_dt_kernel(const typename Tag::S *__restrict__ x,
                                                           const typename Tag::S *__restrict__ dy,
                                                           float *__restrict__ dt, GenArgs a) {
  const int64_t K1 = 2 * a.ww - 1, K2 = K1 * (2 * a.wh - 1);
  for (int64_t e = blockIdx.x * 256LL + threadIdx.x; e < a.C * K2; e += (int64_t)gridDim.x * 256) {
    const int64_t c = e / K2, k = e - c * K2;
    const int64_t dh = k / K1 - (a.wh - 1), dw = k % K1 - (a.ww - 1);
    float s = 0.f;
    for (int64_t o = 0; o < a.numel; ++o) {  // output position o, input at offset (dh, dw) in the same window
      const int64_t gx = o % a.W, gy = o / a.W % a.H;
      if (o / a.hw % a.C != c) continue;
      const int64_t hx = gx + dw, hy = gy + dh;
      if (hx < gx / a.ww * a.ww || hx >= (gx / a.ww + 1) * a.ww || hx >= a.W) continue;
      if (hy < gy / a.wh * a.wh || hy >= (gy / a.wh + 1) * a.wh || hy >= a.H) continue;
      const int64_t i = o + dh * a.W + dw;
      if constexpr (Tag::W16) s += to_f32<Tag>(x[i]) * to_f32<Tag>(dy[o]);
      else s += x[i] * dy[o];
    }
    dt[e] = s;
  }
}

template <class Tag>
static hipError_t run_gen_dt(const void *x, const void *dy, const void *t, void *dx, float *dt, float *ws,
                             const Geom &g, int wh, int ww, int64_t max_slabs, hipStream_t st) {
  GenArgs a = gen_args(g, wh, ww);
  if (a.numel < 16) {
    typedef typename Tag::S E;
    if (dx) return hipErrorInvalidValue;
    const int64_t blocks = cdiv64(g.C * (int64_t)(2 * wh - 1) * (2 * ww - 1), 256);
    gen_small_dt_kernel<Tag><<<dim3((unsigned)blocks), dim3(256), 0, st>>>((const E *)x, (const E *)dy, dt, a);
    return hipGetLastError();
  }
  if (ww <= 8) {
    switch ((wh + 3) / 4) {
      case 1: return gen_dt<Tag, 8, 1>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 2: return gen_dt<Tag, 8, 2>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 3: return gen_dt<Tag, 8, 3>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 4: return gen_dt<Tag, 8, 4>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
    }
  } else {
    switch ((wh + 1) / 2) {
      case 1: return gen_dt<Tag, 16, 1>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 2: return gen_dt<Tag, 16, 2>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 3: return gen_dt<Tag, 16, 3>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 4: return gen_dt<Tag, 16, 4>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 5: return gen_dt<Tag, 16, 5>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 6: return gen_dt<Tag, 16, 6>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 7: return gen_dt<Tag, 16, 7>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
      case 8: return gen_dt<Tag, 16, 8>(x, dy, t, dx, dt, ws, g, wh, ww, max_slabs, st);
    }
  }
  return hipErrorInvalidValue;
}

template <>
hipError_t GenEntry<WBMM_INST_TAG>::backward(const void *x, const void *dy, const void *t, void *dx, float *dt,
                                             void *ws, const Geom &g, int wh, int ww, int64_t max_slabs,
                                             hipStream_t st) {
  return run_gen_dt<WBMM_INST_TAG>(x, dy, t, dx, dt, (float *)ws, g, wh, ww, max_slabs, st);
}

template <>
hipError_t GenEntry<WBMM_INST_TAG>::forward(const void *x, const void *coef, void *y, const Geom &g, int wh, int ww,
                                            int src, hipStream_t st) {
  return run_gen_fwd<WBMM_INST_TAG>(x, coef, y, g, wh, ww, src, st);
}

}  // namespace wbmm
