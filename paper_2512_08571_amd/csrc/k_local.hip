// Matrix-free local operator: dispatch by precision (kernels in k_local_impl.h,
// instantiated in k_local_f64.hip, k_local_f32.hip, k_local_bf16.hip).
#include <algorithm>
#include <mutex>
#include <vector>

#include "fe_internal.h"

namespace fehx {

fe_status launch_local_f64(const LocalBatch &B, hipStream_t s);
fe_status launch_local_f32(const LocalBatch &B, hipStream_t s);
fe_status launch_local_bf16(const LocalBatch &B, hipStream_t s);
fe_status launch_local_mass(const LocalBatch &B, hipStream_t s);

// A wave (or block) walks its cells one after another, so a launch with few
// columns and tiles leaves most of the device idle for the length of a column.
// Its columns are then cut into segments (the planes at the cuts go to a side
// block and are formed after the last colour phase, in the order of uncut
// columns: the count does not show in the result).  The count is the one of
// least cost, summed over the colour phases (odd cell counts have five small
// ones): rounds of the device's units, per_unit items each, times cells per
// item.  An item's first gather and last plane cost about half a cell; a cell
// takes about 1 + 2 k with k waves on a SIMD (FP64, 7 points: 20 us alone, 34 us
// by twos).  Measured per
// colour phase, 7 points: FP64 12^3 cells x 256 lanes, 1152 waves in two segments
// (1.1 rounds) 362 us, in three 285; FP32 16^3 x 256, 1024 waves whole 500 us, in
// two segments 395; the whole mass operator on 11 x 13 x 12 cells x 101 lanes
// (nine phases) in five segments 463 us, in the model's twelve 380.
// (SEG_MAX: past it every unit of the device has a segment of the four or more
// columns to itself; k_planes_join takes segments x cells below 2^32)
constexpr int64_t SEG_MAX = 2048;
int segment_count(const int *phase_off, int nphase, int64_t cells, int64_t tiles, int units, int per_unit, int64_t cap,
                  double *cost) {
  per_unit = std::max(per_unit, 1);              // (an occupancy query may answer none)
  auto round = [](int64_t k) { return k ? 1.0 + 2.0 * k : 0.0; };
  int best = 1;
  double least = 0;
  for (int64_t n = 1; n <= std::max<int64_t>(1, std::min<int64_t>({cells, cap, SEG_MAX, (1LL << 31) / cells})); ++n) {
    double c = 0;
    for (int ph = 0; ph < nphase; ++ph) {
      const int64_t k = ((int64_t)(phase_off[ph + 1] - phase_off[ph]) * tiles * n + units - 1) / units;
      c += (double)(k / per_unit) * round(per_unit) + round(k % per_unit);
    }
    c *= (cells + n - 1) / n + 0.5;
    if (n == 1 || c < least) { best = (int)n; least = c; }
  }
  if (cost) *cost = least;
  return best;
}

// Bytes of the side block per segment: two halves of [cut][column][x][y][lane] in
// the compute type, cut s the first plane of segment s, half 0 what that segment
// adds to it and half 1 what the one below does (cut 0: the periodic wrap).
int64_t side_seg_bytes(const Mesh *m, int64_t side_lanes, int elem_bytes) {
  return 2LL * m->N[0] * m->N[1] * m->np * m->np * side_lanes * elem_bytes;
}

// (k_planes_join's grid has the nodes along a_1 as its y)
static int64_t side_room(const Mesh *m, int64_t side_bytes, int64_t seg_bytes) {
  return m->Mn[1] > 65535 ? 0 : side_bytes / seg_bytes;
}

int plane_segment_count(const Mesh *m, int nq, int nlanes, bool f64, int lpt, int64_t side_bytes, double *cost) {
  const int vt = plane_vt(nq, lpt), tiles = (nlanes + vt - 1) / vt;
  return segment_count(m->phase_off.data(), m->nphase, m->N[2], tiles, 4 * m->cus, plane_waves(nq, f64, lpt),
                       side_room(m, side_bytes, side_seg_bytes(m, (int64_t)tiles * vt, f64 ? 8 : 4)), cost);
}

// the same for the staged kernels: blocks on CUs (distorted 8 x 10 x 8 cells
// degree 4 x 64 FP64 vectors, whole columns 240 us, segments 117; 9 points
// 12^3 cells degree 6 x 128 2157 and 1770)
int block_segment_count(const Mesh *m, int tiles, int per_cu, int64_t seg_bytes, int64_t side_bytes) {
  return segment_count(m->phase_off.data(), m->nphase, m->N[2], tiles, m->cus, per_cu, side_room(m, side_bytes, seg_bytes),
                       nullptr);
}

bool plane_mesh(const Mesh *m) { return !m->offd && m->nq == m->np; }

// The choice depends on the system and its blocks alone, never on those it
// shares a launch with.  The plane kernels take affine cells with a diagonal
// metric (the mass operator: affine cells) and, in FP32 and BF16, complex
// vectors as pairs of lanes; a z plane past their span goes to the staged kernel.
LocalKind local_kind(const Mesh *m, const LocalLaunch &L) {
  const size_t es = L.prec == FE_F64 ? 8 : L.prec == FE_F32 || L.store32 ? 4 : 2;
  const bool reach = (int64_t)m->Mn[0] * m->Mn[1] * L.ldy * (int64_t)es < PLANE_SPAN;
  const bool pairs = L.prec != FE_F64 && !((L.ldx | L.ldy | L.nlanes) & 1) &&
                     ((uintptr_t)L.X | (uintptr_t)L.Y) % (2 * es) == 0;
  if (L.mass) return m->distorted || !reach ? LOCAL_STAGED : pairs ? LOCAL_MASS_PAIRS : LOCAL_MASS;
  if (m->offd) return LOCAL_GENERAL;
  if (m->nq != m->np || !reach || (m->cplx && L.prec != FE_F64 && !pairs)) return LOCAL_STAGED;
  return pairs ? LOCAL_PLANES_PAIRS : LOCAL_PLANES;
}

// Whether threads of two lanes (a third faster per lane on a full device) beat
// threads of one (0.55 of the time per cell, twice the waves) for real blocks;
// both form the same sums.
// FP32, 7 points, a colour phase: 14^3 cells x 8 vectors pairs 38 us, ones 23;
// 16^3 x 256 pairs 313, ones (255 vectors) 349.
bool plane_pairs_pay(const LocalBatch &B, int nq) {
  double one = 0, two = 0;
  for (int i = 0; i < B.n; ++i) {
    const LocalLaunch &L = B.Ls[i];
    const int64_t side = side_limit(L);
    double c1, c2;
    plane_segment_count(B.ms[i], nq, L.nlanes, false, 1, side, &c1);
    plane_segment_count(B.ms[i], nq, L.nlanes, false, 2, side, &c2);
    one += 0.55 * c1;
    two += c2;
  }
  return two <= one;
}

// bytes of the side block of an application to a block of nlanes lanes: for the
// plane kernels with either width of a thread; one segment per cell elsewhere
// (the widest tile there holds 32 lanes)
int64_t plane_side_need(const Mesh *m, int nlanes, int prec) {
  const bool f64 = prec == FE_F64;
  int64_t need = 0;
  for (int lpt = 1; lpt <= (f64 ? 1 : 2); ++lpt) {
    const int vt = plane_mesh(m) ? plane_vt(m->nq, lpt) : 32;
    const int64_t seg = side_seg_bytes(m, (int64_t)(nlanes + vt - 1) / vt * vt, f64 ? 8 : 4);
    const int64_t n = plane_mesh(m) ? plane_segment_count(m, m->nq, nlanes, f64, lpt, SIDE_BYTES, nullptr)
                                    : std::min<int64_t>(m->N[2], SIDE_BYTES / seg);
    if (n > 1) need = std::max(need, n * seg);
  }
  return need;
}

// ---- side blocks ------------------------------------------------------------
// They belong to the device: as many as it has meshes, up to SIDE_BLOCKS,
// allocated when a mesh is made, so that an application allocates nothing,
// whichever mesh it is on.  The last mesh frees all but the first block, which
// the next mesh of the process finds (a program that makes and destroys one
// mesh at a time paid 0.2 ms for making and 0.6 for destroying each).
// An application that cuts its columns holds one while it enqueues and leaves
// an event behind; the next on that stream follows in stream order, one on
// another stream takes a block whose event has passed.  Without a block (all in
// use by other streams, no memory for one, or a stream that is capturing, whose
// graph may be replayed beside anything) columns stay whole, with the same
// result.  The event orders work on the device only: without the fence to the
// host it costs 0.7 us of an application, with it 2.5.
// 192 MiB hold the segments that the device's fill asks for: 12^3 cells of 9
// points x 256 FP64 lanes, three of 48 MiB, 3026 us an application, whole
// columns 3490.
constexpr int SIDE_BLOCKS = 4, SIDE_DEVICES = 64;
struct SideBlock {
  void *p = nullptr, *q = nullptr;
  hipEvent_t done = nullptr;
  hipStream_t s = nullptr;   // of the last use
  bool used = false, held = false;
};
namespace {
struct SidePool {
  std::mutex mu;
  int meshes = 0;
  SideBlock blocks[SIDE_BLOCKS];
};
SidePool g_side[SIDE_DEVICES];

// the event has passed; asked without upsetting a capture on another stream
bool event_passed(hipEvent_t e) {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  const hipError_t r = hipEventQuery(e);
  (void)hipThreadExchangeStreamCaptureMode(&mode);
  if (r != hipSuccess) (void)hipGetLastError();
  return r == hipSuccess;
}
}  // namespace

void side_pool_enter(int device) {
  if (device < 0 || device >= SIDE_DEVICES) return;
  SidePool &P = g_side[device];
  std::lock_guard<std::mutex> g(P.mu);
  const int i = P.meshes++;
  if (i >= SIDE_BLOCKS || P.blocks[i].p) return;
  SideBlock b;
  if (hipEventCreateWithFlags(&b.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess) {
    if (hipMalloc(&b.p, (size_t)SIDE_BYTES / 2) == hipSuccess) {
      if (hipMalloc(&b.q, (size_t)SIDE_BYTES / 2) == hipSuccess) {
        P.blocks[i] = b;
        return;
      }
      hipFree(b.p);
    }
    hipEventDestroy(b.done);
  }
  (void)hipGetLastError();                       // columns stay whole
}

// (the device has been synchronised)
void side_pool_leave(int device) {
  if (device < 0 || device >= SIDE_DEVICES) return;
  SidePool &P = g_side[device];
  std::lock_guard<std::mutex> g(P.mu);
  if (--P.meshes > 0) return;
  for (int i = 1; i < SIDE_BLOCKS; ++i) {
    SideBlock &b = P.blocks[i];
    if (b.p) {
      hipFree(b.p);
      hipFree(b.q);
      hipEventDestroy(b.done);
    }
    b = SideBlock();
  }
}

void *SideUse::take(int device, hipStream_t s, int64_t *half) {
  if (device < 0 || device >= SIDE_DEVICES) return nullptr;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(s, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  if (cs != hipStreamCaptureStatusNone) return nullptr;
  SidePool &P = g_side[device];
  std::lock_guard<std::mutex> g(P.mu);
  SideBlock *found = nullptr;
  for (SideBlock &b : P.blocks)
    if (b.p && !b.held && b.used && b.s == s) { found = &b; break; }
  // (a handle may be a new stream's: for one and the same stream the wait is nothing)
  if (found && hipStreamWaitEvent(s, found->done, 0) != hipSuccess) {
    (void)hipGetLastError();
    found = nullptr;
  }
  if (!found)
    for (SideBlock &b : P.blocks)
      if (b.p && !b.held && (!b.used || event_passed(b.done))) { found = &b; break; }
  if (!found) return nullptr;
  found->held = true;
  block_ = found;
  device_ = device;
  s_ = s;
  *half = (char *)found->q - (char *)found->p;
  return found->p;
}

SideUse::~SideUse() {
  if (!block_) return;
  std::lock_guard<std::mutex> g(g_side[device_].mu);
  block_->used = true;
  block_->s = s_;
  // without an event behind the work the block is not given out again
  block_->held = hipEventRecord(block_->done, s_) != hipSuccess;
}

static fe_status launch_local_kind(const LocalBatch &B, hipStream_t s) {
  for (int i = 1; i < B.n && B.kind <= LOCAL_GENERAL; ++i)
    if (B.Ls[i].vt != B.Ls[0].vt) return set_error(FE_EINVAL, "a batched launch of the staged kernel needs one vector tile");
  if (B.kind >= LOCAL_MASS) return launch_local_mass(B, s);
  if (B.Ls[0].prec == FE_F64) return launch_local_f64(B, s);
  if (B.Ls[0].prec == FE_F32) return launch_local_f32(B, s);
  if (B.Ls[0].prec == FE_BF16) return launch_local_bf16(B, s);
  return set_error(FE_EINVAL, "unknown precision");
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
    if (B.Ls[i].prec != B.Ls[0].prec || B.Ls[i].store32 != B.Ls[0].store32)
      return set_error(FE_EINVAL, "a batched launch needs one precision and block type");
  }
  // systems that run different kernels: one launch set each
  LocalBatch P = B;
  P.kind = local_kind(B.ms[0], B.Ls[0]);
  int same = 1;
  while (same < B.n && local_kind(B.ms[same], B.Ls[same]) == P.kind) ++same;
  if (same == B.n) return launch_local_kind(P, s);
  std::vector<Mesh *> ms;
  std::vector<LocalLaunch> Ls;
  for (int kind = LOCAL_STAGED; kind <= LOCAL_MASS_PAIRS; ++kind) {
    ms.clear();
    Ls.clear();
    for (int i = 0; i < B.n; ++i)
      if (local_kind(B.ms[i], B.Ls[i]) == kind) { ms.push_back(B.ms[i]); Ls.push_back(B.Ls[i]); }
    P.ms = ms.data(); P.Ls = Ls.data(); P.n = (int)ms.size();
    P.kind = (LocalKind)kind;
    const fe_status st = P.n ? launch_local_kind(P, s) : (fe_status)FE_OK;
    if (st) return st;
  }
  return FE_OK;
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
