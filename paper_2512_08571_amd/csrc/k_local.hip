// Matrix-free local operator: dispatch by precision (kernels in k_local_impl.h,
// instantiated in k_local_f64.hip, k_local_f32.hip, k_local_bf16.hip).
#include <algorithm>
#include <vector>

#include "fe_internal.h"

namespace fehx {

constexpr int PLANE_WAVES = 2048;

fe_status launch_local_f64(const LocalBatch &B, hipStream_t s);
fe_status launch_local_f32(const LocalBatch &B, hipStream_t s);
fe_status launch_local_bf16(const LocalBatch &B, hipStream_t s);

// A wave of the plane kernels walks its cells one after another, so a launch
// with few columns and tiles leaves most of the device idle for the length of
// a column.  Its columns are then cut into segments: enough for two waves per
// SIMD of 256 CUs, at most one per cell, and at most PLANE_SIDE_BYTES for the
// planes that two segments share (each segment's first plane goes to a side
// block of planes laid out as Y's, added to Y after the last colour phase).
int plane_segment_count(const Mesh *m, int nlanes, int64_t ldy, int vt, int elem_bytes) {
  const int64_t waves = (int64_t)(m->phase_off[1] - m->phase_off[0]) * ((nlanes + vt - 1) / vt);
  const int64_t plane = (int64_t)m->Mn[0] * m->Mn[1] * ldy * elem_bytes;
  int64_t n = (PLANE_WAVES + waves - 1) / waves;
  n = std::min<int64_t>(n, m->N[2]);
  n = std::min<int64_t>(n, PLANE_SIDE_BYTES / plane);
  return (int)std::max<int64_t>(n, 1);
}

int plane_vt(int nq, int lpt) { return ((64 / nq) & ~1) * lpt; }

bool plane_mesh(const Mesh *m) { return !m->offd && m->nq == m->np; }

// bytes of the side block of an application to a block of nlanes lanes with
// leading dimension ldy (lanes), for either width of a thread
int64_t plane_side_need(const Mesh *m, int nlanes, int64_t ldy, int prec) {
  if (!plane_mesh(m) || prec != FE_F64) return 0;
  const int es = 8;
  int64_t need = 0;
  for (int lpt = 1; lpt <= 1; ++lpt) {
    const int n = plane_segment_count(m, nlanes, ldy, plane_vt(m->nq, lpt), es);
    if (n > 1) need = std::max(need, (int64_t)n * m->Mn[0] * m->Mn[1] * ldy * es);
  }
  return need;
}

// The mesh's side block is shared by every application of the mesh, which may
// come on any stream: applications on one stream are in order by themselves;
// the first one on another stream waits for the device, and from then on each
// records an event that one on another stream waits for.
fe_status plane_side_enter(Mesh *m, hipStream_t s) {
  if (m->side_used && m->side_stream != s) {
    if (!m->side_ev) {
      FE_HIP_TRY(hipEventCreateWithFlags(&m->side_ev, hipEventDisableTiming));
      FE_HIP_TRY(hipDeviceSynchronize());
    } else {
      FE_HIP_TRY(hipStreamWaitEvent(s, m->side_ev, 0));
    }
  }
  m->side_used = true;
  m->side_stream = s;
  return FE_OK;
}
fe_status plane_side_leave(Mesh *m, hipStream_t s) {
  if (m->side_ev) FE_HIP_TRY(hipEventRecord(m->side_ev, s));
  return FE_OK;
}

// The count for a launch and its side block: the launch's own, or the mesh's
// (then *shared: enter and leave around the use).  A block that cannot be had
// now (the stream is capturing, a captured graph holds the mesh's smaller one,
// no memory) means one segment.
int plane_segments(Mesh *m, const LocalLaunch &L, int vt, int elem_bytes, hipStream_t s, void **side, bool *shared) {
  const int n = plane_segment_count(m, L.nlanes, L.ldy, vt, elem_bytes);
  *side = L.side;
  *shared = false;
  if (n == 1 || L.side) return n;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return 1;
  const int64_t need = (int64_t)n * m->Mn[0] * m->Mn[1] * L.ldy * elem_bytes;
  if (m->ws_bytes[11] < need && (m->graphs > 0 || ensure_workspace(m, 11, need))) return 1;
  *side = m->ws[11];
  *shared = true;
  return n;
}

fe_status launch_local_batch(const LocalBatch &B, hipStream_t s) {
  if (B.n < 1) return FE_OK;
  Mesh *m0 = B.ms[0];
  for (int i = 0; i < B.n; ++i) {
    Mesh *m = B.ms[i];
    if (m->nq != m->np && m->nq != m->np + 2 && m->nq != m->np + 3)
      return set_error(FE_EUNSUPPORTED, "this build has kernels for n_q = n_p, n_p + 2 and n_p + 3 only");
    if (m->np != m0->np || m->nq != m0->nq || m->cplx != m0->cplx || m->device != m0->device)
      return set_error(FE_EINVAL, "a batched launch needs one degree, quadrature, field type and device");
    if (B.Ls[i].prec != B.Ls[0].prec || B.Ls[i].vt != B.Ls[0].vt || B.Ls[i].store32 != B.Ls[0].store32)
      return set_error(FE_EINVAL, "a batched launch needs one precision, block type and vector tile");
  }
  // general-metric systems and the rest run different kernels: one launch set each
  auto general = [&](int i) { return B.ms[i]->offd && !B.Ls[i].mass; };
  int ngen = 0;
  for (int i = 0; i < B.n; ++i) ngen += general(i) ? 1 : 0;
  if (ngen > 0 && ngen < B.n) {
    for (int kind = 0; kind < 2; ++kind) {
      std::vector<Mesh *> ms;
      std::vector<LocalLaunch> Ls;
      for (int i = 0; i < B.n; ++i)
        if (general(i) == (kind == 1)) { ms.push_back(B.ms[i]); Ls.push_back(B.Ls[i]); }
      LocalBatch P = B;
      P.ms = ms.data(); P.Ls = Ls.data(); P.n = (int)ms.size();
      const fe_status st = launch_local_batch(P, s);
      if (st) return st;
    }
    return FE_OK;
  }
  if (B.Ls[0].prec == FE_F64) return launch_local_f64(B, s);
  if (B.Ls[0].prec == FE_F32) return launch_local_f32(B, s);
  if (B.Ls[0].prec == FE_BF16) return launch_local_bf16(B, s);
  return set_error(FE_EINVAL, "unknown precision");
}

fe_status launch_local(Mesh *m, const LocalLaunch &L, hipStream_t s) {
  Mesh *ms[1] = {m};
  LocalBatch B;
  B.ms = ms;
  B.Ls = &L;
  B.n = 1;
  return launch_local_batch(B, s);
}

}  // namespace fehx
