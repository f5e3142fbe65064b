// Dispatch of (dtype, window size) to the kernel instantiations compiled in
// the wbmm_inst.hip translation units.
#include <hip/hip_runtime.h>

#include "wbmm_internal.h"

namespace wbmm {

#define WBMM_TABLES(tag)                                                                  \
  extern Entry entries_##tag##_1[kInstWindows], entries_##tag##_5[kInstWindows],          \
      entries_##tag##_9[kInstWindows], entries_##tag##_13[kInstWindows];                 \
  static Entry *const tables_##tag[4] = {entries_##tag##_1, entries_##tag##_5, entries_##tag##_9, \
                                         entries_##tag##_13};
WBMM_TABLES(TagF32)
WBMM_TABLES(TagBF16)
WBMM_TABLES(TagF16)
#undef WBMM_TABLES

namespace {

const Entry *find(Dt dt, int w) {
  if (w < kMinWindow || w > kMaxWindow) return nullptr;
  const int u = (w - 1) / kInstWindows;
  const int k = (w - 1) % kInstWindows;
  switch (dt) {
    case Dt::F32: return &tables_TagF32[u][k];
    case Dt::BF16: return &tables_TagBF16[u][k];
    case Dt::F16: return &tables_TagF16[u][k];
  }
  return nullptr;
}

}  // namespace

hipError_t launch_forward(Dt dt, const void *x, const void *table, void *y, const Geom &g,
                          bool reverse_table, hipStream_t stream) {
  const Entry *e = find(dt, g.w);
  if (!e) return hipErrorInvalidValue;
  return e->fwd(x, table, y, g, reverse_table, stream);
}

hipError_t launch_dtable(Dt dt, const void *x, const void *dy, float *dtable, void *workspace,
                         const Geom &g, hipStream_t stream) {
  const Entry *e = find(dt, g.w);
  if (!e) return hipErrorInvalidValue;
  return e->dtable(x, dy, dtable, workspace, g, stream);
}

hipError_t launch_backward(Dt dt, const void *x, const void *dy, const void *table, void *dx, float *dtable,
                           void *workspace, const Geom &g, hipStream_t stream) {
  const Entry *e = find(dt, g.w);
  if (!e) return hipErrorInvalidValue;
  return e->bwd(x, dy, table, dx, dtable, workspace, g, stream);
}

hipError_t launch_hier_forward(Dt dt, const void *x, const void *table_g, const void *table_l, void *y,
                               const Geom &g, bool reverse_tables, hipStream_t stream) {
  const Entry *e = find(dt, g.w);
  if (!e) return hipErrorInvalidValue;
  return e->hier_fwd(x, table_g, table_l, y, g, reverse_tables, stream);
}

hipError_t launch_hier_stream(Dt dt, const void *x, const void *dy, const void *table_g, const void *table_l,
                              void *dx, float *dtable_g, float *dtable_l, void *workspace, size_t workspace_bytes,
                              const Geom &g, hipStream_t stream, bool *done) {
  *done = false;
  const Entry *e = find(dt, g.w);
  if (!e) return hipErrorInvalidValue;
  return e->hier_stream(x, dy, table_g, table_l, dx, dtable_g, dtable_l, workspace, workspace_bytes, g, stream,
                        done);
}

DtPlan plan_dtable(Dt dt, const Geom &g) {
  const Entry *e = find(dt, g.w);
  if (!e) return DtPlan{0, 0};
  return e->plan(g);
}

size_t dtable_workspace_bytes(Dt dt, const Geom &g) {
  const DtPlan p = plan_dtable(dt, g);
  if (p.slabs <= 1) return 0;
  const int64_t k1 = 2 * g.w - 1;
  return (size_t)p.slabs * (size_t)g.C * (size_t)(k1 * k1) * sizeof(float);
}

hipError_t launch_dense_forward(Dt dt, const void *x, const void *m, void *y, const Geom &g, int wh, int ww,
                                bool trans, hipStream_t stream) {
  const int src = trans ? 3 : 2;
  switch (dt) {
    case Dt::F32: return GenEntry<TagF32>::forward(x, m, y, g, wh, ww, src, stream);
    case Dt::BF16: return GenEntry<TagBF16>::forward(x, m, y, g, wh, ww, src, stream);
    case Dt::F16: return GenEntry<TagF16>::forward(x, m, y, g, wh, ww, src, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_rect_forward(Dt dt, const void *x, const void *table, void *y, const Geom &g, int wh, int ww,
                               bool reverse_table, hipStream_t stream) {
  const int src = reverse_table ? 1 : 0;
  switch (dt) {
    case Dt::F32: return GenEntry<TagF32>::forward(x, table, y, g, wh, ww, src, stream);
    case Dt::BF16: return GenEntry<TagBF16>::forward(x, table, y, g, wh, ww, src, stream);
    case Dt::F16: return GenEntry<TagF16>::forward(x, table, y, g, wh, ww, src, stream);
  }
  return hipErrorInvalidValue;
}

// As many partial tables as fill the chip a few times over, each of at least
// one stage of 32 windows.
int64_t rect_max_slabs(const Geom &g) {
  const int64_t stages = (g.N + 31) / 32, fill = (1024 + g.C - 1) / g.C;
  return fill < stages ? fill : stages;
}

hipError_t launch_rect_dtable(Dt dt, const void *x, const void *dy, float *dtable, void *workspace, const Geom &g,
                              int wh, int ww, hipStream_t stream) {
  const int64_t slabs = rect_max_slabs(g);
  switch (dt) {
    case Dt::F32: return GenEntry<TagF32>::backward(x, dy, nullptr, nullptr, dtable, workspace, g, wh, ww, slabs, stream);
    case Dt::BF16: return GenEntry<TagBF16>::backward(x, dy, nullptr, nullptr, dtable, workspace, g, wh, ww, slabs, stream);
    case Dt::F16: return GenEntry<TagF16>::backward(x, dy, nullptr, nullptr, dtable, workspace, g, wh, ww, slabs, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace wbmm
