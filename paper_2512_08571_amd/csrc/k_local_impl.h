// Matrix-free local operator H_loc X on gfx950 (Sec. 3.2, eqns ggaReal /
// ggaCmplx, Alg. 2), one subdomain on one GPU.
//
// Work decomposition (the GPU analogue of the paper's multilevel batches,
// Sec. 4.1): a workgroup owns one column of cells along a_2 and one tile of
// VT real vector lanes (for complex meshes the real and imaginary parts of a
// vector sit in adjacent lanes, the paper's level-2 re/im batches).  It walks
// the column cell by cell: the 1D contraction sweeps of Alg. 2 with the
// even-odd decomposition (each thread applies one 1D matrix to one line of
// points for one lane, table rows read as wave-uniform scalars) and the
// quadrature-point stage of eqn refact, on LDS blocks [point][lane] (lanes
// fastest); the block is staged in LDS and every sweep is its own pass.  These
// kernels serve n_q > n_p and the general metric (sheared and distorted
// cells); k_local_planes.h serves n_q = n_p with a diagonal metric.
//
// Scatter Y += Q^(e)T Y^(e) without atomics and deterministically:
//  * along a_2 the shared node plane of consecutive cells is summed in LDS
//    (and the periodic first/last plane of the column at the end); where a
//    column is cut into segments, the two halves of a cut's plane go to a side
//    block in the compute type and k_planes_join adds them up in the order of
//    the uncut column, so that the cuts do not show in the result;
//  * across columns the columns are coloured 2 (or 3 for an odd count) per
//    axis and launched colour by colour; a node shared by several columns is
//    stored by the column of the lowest colour phase and read-modify-written
//    by the later ones, so no two concurrently running workgroups touch the
//    same node and the summation order is fixed.
#pragma once
#include <algorithm>
#include <type_traits>
#include <vector>

#include "fe_internal.h"

namespace fehx {

// ---- storage conversions -----------------------------------------------------
struct bf16s { uint16_t b; };

__device__ __forceinline__ float bf16_to_f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);   // round to nearest even
  return (uint16_t)(u >> 16);
}

template <typename TS, typename TC> struct Cvt;
template <> struct Cvt<double, double> {
  static __device__ __forceinline__ double ld(const double *p, int64_t i) { return p[i]; }
  static __device__ __forceinline__ void st(double *p, int64_t i, double v) { p[i] = v; }
};
template <> struct Cvt<float, float> {
  static __device__ __forceinline__ float ld(const float *p, int64_t i) { return p[i]; }
  static __device__ __forceinline__ void st(float *p, int64_t i, float v) { p[i] = v; }
};
template <> struct Cvt<bf16s, float> {
  static __device__ __forceinline__ float ld(const bf16s *p, int64_t i) { return bf16_to_f(p[i].b); }
  static __device__ __forceinline__ void st(bf16s *p, int64_t i, float v) { p[i].b = f_to_bf16(v); }
};

// L consecutive lanes of one node row: global (storage type, 16-byte vector
// access for the wide forms) and LDS (compute type)
template <typename TS, typename TC, int L> struct VecIO;
template <typename TS, typename TC> struct VecIO<TS, TC, 1> {
  static __device__ __forceinline__ void ld(const TS *p, TC (&v)[1]) { v[0] = Cvt<TS, TC>::ld(p, 0); }
  static __device__ __forceinline__ void st(TS *p, const TC (&v)[1]) { Cvt<TS, TC>::st(p, 0, v[0]); }
};
template <> struct VecIO<double, double, 2> {
  static __device__ __forceinline__ void ld(const double *p, double (&v)[2]) {
    const double2 a = *(const double2 *)p; v[0] = a.x; v[1] = a.y;
  }
  static __device__ __forceinline__ void st(double *p, const double (&v)[2]) { *(double2 *)p = make_double2(v[0], v[1]); }
};
template <> struct VecIO<float, float, 4> {
  static __device__ __forceinline__ void ld(const float *p, float (&v)[4]) {
    const float4 a = *(const float4 *)p; v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  }
  static __device__ __forceinline__ void st(float *p, const float (&v)[4]) { *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]); }
};
template <> struct VecIO<bf16s, float, 8> {
  static __device__ __forceinline__ void ld(const bf16s *p, float (&v)[8]) {
    const uint4 a = *(const uint4 *)p;
    const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void st(bf16s *p, const float (&v)[8]) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = (uint32_t)f_to_bf16(v[2 * i]) | ((uint32_t)f_to_bf16(v[2 * i + 1]) << 16);
    *(uint4 *)p = make_uint4(w[0], w[1], w[2], w[3]);
  }
};
template <typename TC, int L> struct LdsVec {
  static __device__ __forceinline__ void st(TC *p, const TC (&v)[L]) {
#pragma unroll
    for (int j = 0; j < L; ++j) p[j] = v[j];
  }
  static __device__ __forceinline__ void ld(const TC *p, TC (&v)[L]) {
#pragma unroll
    for (int j = 0; j < L; ++j) v[j] = p[j];
  }
};
template <> struct LdsVec<double, 2> {
  static __device__ __forceinline__ void st(double *p, const double (&v)[2]) { *(double2 *)p = make_double2(v[0], v[1]); }
  static __device__ __forceinline__ void ld(const double *p, double (&v)[2]) {
    const double2 a = *(const double2 *)p; v[0] = a.x; v[1] = a.y;
  }
};
template <> struct LdsVec<float, 4> {
  static __device__ __forceinline__ void st(float *p, const float (&v)[4]) { *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]); }
  static __device__ __forceinline__ void ld(const float *p, float (&v)[4]) {
    const float4 a = *(const float4 *)p; v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  }
};
template <> struct LdsVec<float, 8> {
  static __device__ __forceinline__ void st(float *p, const float (&v)[8]) {
    *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
    *(float4 *)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
  static __device__ __forceinline__ void ld(const float *p, float (&v)[8]) {
    const float4 a = *(const float4 *)p, b = *(const float4 *)(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};
// lanes per element of the wide form: 16 bytes of storage
template <typename TS> struct WideLanes { static constexpr int value = 16 / sizeof(TS); };

// ---- kernel arguments ----------------------------------------------------------
template <typename TC> struct KArgs {
  const void *X;
  void *Y;
  int64_t ldx, ldy;
  int nlanes;
  int N0, N1, N2, M0, M1, M2, p;
  int dmask;           // bit d: axis d has Dirichlet faces (interior nodes g - 1)
  int offd;            // off-diagonal metric terms (sheared box): gradients staged in LDS
  const int *cols;
  int ncols, ntiles;
  const TC *tab;
  const TC *wq;
  const TC *coef;
  int64_t coef_cell;   // coefficient elements per cell (0: one block for all cells)
  int gga;
  const double *dinv;
  int ncoef;           // coefficient blocks per cell (4, or NCOEF_GEN with the per-point metric)
  const TC *ptab;      // plane kernels: tables (PlaneTab), the gather's N table, coefficients, Bloch factors
  const TC *pgather;
  const TC *pcoef;
  TC pkap[3];
  int nseg;            // segments a column is cut into, and the planes at their cuts (side_seg_bytes)
  TC *side;            // (the first half)
  int64_t side_half;   // elements from its first half to the second
};

// ---- even-odd application of a packed centro-(anti)symmetric 1D matrix ----------
// tab rows q < ceil(NOUT/2): E[q][0..ceil(NIN/2)) then O[q][0..floor(NIN/2)).
template <typename TC> using cptr = const __attribute__((address_space(4))) TC *;

// A wave-uniform table pointer whose value the compiler cannot see through:
// the table is re-read with scalar loads at each use instead of being hoisted
// out of the loops into (spilled) registers.
template <typename TC> __device__ __forceinline__ cptr<TC> scalar_table(const TC *p) {
  uint64_t a = reinterpret_cast<uint64_t>(p);
  asm volatile("" : "+s"(a));
  return reinterpret_cast<cptr<TC>>(a);
}

template <int NIN, int NOUT, int SYM, typename TC>
__device__ __forceinline__ void eo_apply(cptr<TC> __restrict__ t, const TC (&x)[NIN], TC (&y)[NOUT]) {
  constexpr int CI = (NIN + 1) / 2, HI = NIN / 2, CO = (NOUT + 1) / 2, HO = NOUT / 2;
  TC xp[CI], xm[HI > 0 ? HI : 1];
#pragma unroll
  for (int i = 0; i < HI; ++i) {
    xp[i] = x[i] + x[NIN - 1 - i];
    xm[i] = x[i] - x[NIN - 1 - i];
  }
  if constexpr (NIN & 1) xp[HI] = x[HI];
#pragma unroll
  for (int q = 0; q < CO; ++q) {
    cptr<TC> E = t + q * NIN;
    cptr<TC> O = E + CI;
    TC e = 0, o = 0;
#pragma unroll
    for (int i = 0; i < CI; ++i) e = fma(E[i], xp[i], e);
#pragma unroll
    for (int i = 0; i < HI; ++i) o = fma(O[i], xm[i], o);
    if ((NOUT & 1) && q == HO) {
      y[q] = (SYM > 0) ? e : o;
    } else {
      y[q] = e + o;
      y[NOUT - 1 - q] = (SYM > 0) ? (e - o) : (o - e);
    }
  }
}

// One 1D contraction over every line of a block: each work item is one
// (line, lane); 'dec' maps a line to (source base, stride, destination base,
// stride) in points.
template <int NIN, int NOUT, int SYM, int VT, int NT, typename TC, typename Dec>
__device__ __forceinline__ void line_pass(const TC *__restrict__ src, TC *__restrict__ dst,
                                          const TC *__restrict__ tab, int nlines, Dec dec) {
  const int total = nlines * VT;
  for (int t = threadIdx.x; t < total; t += NT) {
    const int v = t % VT, l = t / VT;
    int sb, ss, db, ds;
    dec(l, sb, ss, db, ds);
    TC x[NIN], y[NOUT];
#pragma unroll
    for (int i = 0; i < NIN; ++i) x[i] = src[(sb + i * ss) * VT + v];
    eo_apply<NIN, NOUT, SYM>(scalar_table(tab), x, y);
#pragma unroll
    for (int i = 0; i < NOUT; ++i) dst[(db + i * ds) * VT + v] = y[i];
  }
}

// Quadrature-point stage for reference direction D (eqn refact / Alg. 2):
// for each line along D of the interpolated field Y0 (src):
//   T   = Dtilde u                                  (gradient along D)
//   F   = G_DD w T + Vtilde^G_D u                   (flux for Dtilde^T)
//   z   = Vtilde^G_D T  [+ (V + |k|^2/2) w u  for D = 0]  [- i kappa_D w T]
//   out = Dtilde^T F + z,   accumulated into dst (initialised by D = 0).
// C holds the cell's weighted coefficients [4][NQ3] staged in LDS (threads of
// one line read the same addresses).  The weight w_Q det J of a point on a
// line along D through (a, b) is W2[line] (w_a w_b, from LDS once per line)
// times the wave-uniform factor w_i det J, pre-multiplied in the table by
// g_DD (kinetic flux) and kappa_D (Bloch term).
// Value of the partner lane (lane ^ 1: the real / imaginary part of the same
// vector) by a DPP quad permutation [1, 0, 3, 2]; both lanes of a pair are
// always active together (tiles hold whole vectors, VT even).
__device__ __forceinline__ double swap_pair(double x) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0xB1, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0xB1, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ float swap_pair(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
}

// The quadrature-point work of one line along reference direction D: given
// the interpolated field u on the line's points, o = Dtilde^T F + z with
//   T = Dtilde u,  F = G_DD w T + Vtilde^G_D u,
//   z = Vtilde^G_D T  [+ (V + |k|^2/2) w u for D = 0]  [- i kappa_D w T],
// line l through (a, b) = (l % NQ, l / NQ) of the other two directions.
template <int D, int NQ, int VT, bool CPLX, typename TC, bool OFFD = false>
__device__ __forceinline__ void dir_line(const TC (&u)[NQ], TC (&out)[NQ], int l, int base, int stride,
                                         const TC *__restrict__ tD, const TC *__restrict__ tDT,
                                         const TC *__restrict__ tgw, const TC *__restrict__ tkw, const KArgs<TC> &a,
                                         const TC *__restrict__ C, const TC *__restrict__ W2, int lane,
                                         const TC *__restrict__ T3 = nullptr,
                                         int v = 0) {
  constexpr int NQ3 = NQ * NQ * NQ;
  const TC *cL = C;
  const TC *cG = C + (1 + D) * NQ3;
  TC T[NQ], F[NQ], z[NQ], o[NQ];
  eo_apply<NQ, NQ, -1>(scalar_table(tD), u, T);
  const TC w2 = W2[l];
  cptr<TC> gw = scalar_table(tgw + D * NQ);
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int Q = base + i * stride;
    if constexpr (OFFD) {
      // general metric (sheared or distorted cells): the weighted metric row
      // of direction D at this point from the coefficient blocks 4-9, the
      // other two reference gradients from LDS
      constexpr int OD[3][3] = {{4, 7, 8}, {7, 5, 9}, {8, 9, 6}};
      F[i] = C[OD[D][D] * NQ3 + Q] * T[i];
#pragma unroll
      for (int t = 0; t < 3; ++t)
        if (t != D) F[i] = fma(C[OD[D][t] * NQ3 + Q], T3[(t * NQ3 + Q) * VT + v], F[i]);
    } else {
      F[i] = (w2 * gw[i]) * T[i];
    }
    z[i] = 0;
    if (a.gga) {
      const TC vg = cG[Q];
      F[i] = fma(vg, u[i], F[i]);
      z[i] = vg * T[i];
    }
    if (D == 0) z[i] = fma(cL[Q], u[i], z[i]);
    if constexpr (CPLX) {
      // -i kappa w T: real lane gets +kappa w T_im, imaginary lane -kappa w T_re
      const TC tp = swap_pair(T[i]);
      const TC kw = OFFD ? C[(10 + D) * NQ3 + Q] : w2 * scalar_table(tkw + D * NQ)[i];
      z[i] = fma((lane & 1) ? -kw : kw, tp, z[i]);
    }
  }
  eo_apply<NQ, NQ, -1>(scalar_table(tDT), F, o);
#pragma unroll
  for (int i = 0; i < NQ; ++i) out[i] = o[i] + z[i];
}

// Lines along D of the interpolated field src (pass-per-sweep path): the
// D = 0 contribution initialises dst, the others are added.  OFFD: the
// off-diagonal metric terms read the other gradients from T3.
template <int D, int NQ, int VT, bool CPLX, typename TC, bool OFFD, int NT>
__device__ __forceinline__ void dir_pass(const TC *__restrict__ src, TC *__restrict__ dst, const TC *tD,
                                         const TC *tDT, const TC *tgw, const TC *tkw, const KArgs<TC> &a,
                                         const TC *__restrict__ C, const TC *__restrict__ W2, int lane0,
                                         const TC *__restrict__ T3) {
  constexpr int NQ2 = NQ * NQ;
  for (int t = threadIdx.x; t < NQ2 * VT; t += NT) {
    const int v = t % VT, l = t / VT;
    int base, stride;
    if (D == 0) { base = l * NQ; stride = 1; }
    else if (D == 1) { base = (l / NQ) * NQ2 + (l % NQ); stride = NQ; }
    else { base = l; stride = NQ2; }
    TC u[NQ], o[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) u[i] = src[(base + i * stride) * VT + v];
    dir_line<D, NQ, VT, CPLX, TC, OFFD>(u, o, l, base, stride, tD, tDT, tgw, tkw, a, C, W2, lane0 + v, T3, v);
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const int idx = (base + i * stride) * VT + v;
      if (D == 0) dst[idx] = o[i];
      else dst[idx] += o[i];
    }
  }
}

// The three reference gradients of src (D-tilde along x, y, z lines) into
// T3[D][point][lane], one pass over the lines of all three directions.
template <int NQ, int VT, int NT, typename TC>
__device__ __forceinline__ void grad_pass(const TC *__restrict__ src, TC *__restrict__ T3, const TC *tD) {
  constexpr int NQ2 = NQ * NQ, NQ3 = NQ2 * NQ;
  for (int t = threadIdx.x; t < 3 * NQ2 * VT; t += NT) {
    const int D = t / (NQ2 * VT), rem = t % (NQ2 * VT);
    const int v = rem % VT, l = rem / VT;
    int base, stride;
    if (D == 0) { base = l * NQ; stride = 1; }
    else if (D == 1) { base = (l / NQ) * NQ2 + (l % NQ); stride = NQ; }
    else { base = l; stride = NQ2; }
    TC u[NQ], g[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) u[i] = src[(base + i * stride) * VT + v];
    eo_apply<NQ, NQ, -1>(scalar_table(tD), u, g);
#pragma unroll
    for (int i = 0; i < NQ; ++i) T3[(D * NQ3 + base + i * stride) * VT + v] = g[i];
  }
}

// first cell of segment s of a column of n cells cut into nseg
__device__ __host__ __forceinline__ int seg_start(int s, int n, int nseg) { return (int)((int64_t)s * n / nseg); }

__device__ __forceinline__ int colour_of(int c, int n) { return ((n & 1) && c == n - 1) ? 2 : (c & 1); }

// FP64 blocks are capped at 512 threads so each lane may use 256 VGPRs.
template <typename TC> struct MaxThreads { static constexpr int value = sizeof(TC) == 8 ? 512 : 1024; };

// Threads per block: one work item per (line, lane) of the widest pass.
template <int NQ, int VT, typename TC> struct BlockSize {
  static constexpr int raw = ((NQ * NQ * VT + 63) / 64) * 64;
  static constexpr int value = raw > MaxThreads<TC>::value ? MaxThreads<TC>::value : (raw < 128 ? 128 : raw);
};

// One work item: segment seg of the column (cx, cy) = a.cols[col] of cells
// along a_2 for vector lanes [tile VT, tile VT + VT).  Ends with a barrier, so the block may
// start another item right away.
//
// Block elements: LPE consecutive lanes of one node (LPE = 1, or the 16-byte
// wide form when every block, leading dimension and lane count is aligned to
// it), so a node's VT lanes are VT / LPE elements and one element is one
// global and one LDS vector access.
template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, int LPE, bool SH>
__device__ __forceinline__ void local_column(const KArgs<TC> &a, const int col, const int seg, const int tile) {
  constexpr int NP2 = NP * NP, NP3 = NP2 * NP, NQ2 = NQ * NQ, NQ3 = NQ2 * NQ;
  constexpr int NT = BlockSize<NQ, VT, TC>::value;
  static_assert(VT <= 255 && NP <= 15, "packed element metadata holds lane offsets < 256 and planes < 16");
  static_assert(VT % LPE == 0, "the vector tile must hold whole elements");
  static_assert(NQ >= NP, "n_q >= n_p");
  constexpr int NV = VT / LPE;                     // elements per node
  constexpr int XPT = (NP3 * NV + NT - 1) / NT;   // block elements per thread
  constexpr int NCF = SH ? NCOEF_GEN : 4;          // coefficient blocks staged per cell
  constexpr int CPT = (NCF * NQ3 + NT - 1) / NT;  // coefficients per thread
  constexpr int OFF_N = 0;
  constexpr int OFF_NT = OFF_N + ((NQ + 1) / 2) * NP;
  constexpr int OFF_D = OFF_NT + ((NP + 1) / 2) * NQ;
  constexpr int OFF_DT = OFF_D + ((NQ + 1) / 2) * NQ;
  constexpr int OFF_GW = OFF_DT + ((NQ + 1) / 2) * NQ;
  constexpr int OFF_KW = OFF_GW + 3 * NQ;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  TC *A = reinterpret_cast<TC *>(smem_raw);
  TC *B = A + NQ3 * VT;
  TC *Ycar = B + NQ3 * VT;
  TC *Yfst = Ycar + NP2 * VT;
  TC *Cf = Yfst + NP2 * VT;          // cell coefficients [NCF][NQ3]
  TC *W2 = Cf + NCF * NQ3;           // w_a w_b per line [NQ2]
  TC *T3 = W2 + NQ2;                 // [3][NQ3][VT] gradients (sheared boxes only)

  const int cx = a.cols[2 * col], cy = a.cols[2 * col + 1];
  const int c0 = seg_start(seg, a.N2, a.nseg), c1 = seg_start(seg + 1, a.N2, a.nseg);
  const int lane0 = tile * VT;
  const int tid = threadIdx.x;
  const TS *__restrict__ X = (const TS *)a.X;
  TS *__restrict__ Y = (TS *)a.Y;
  const TC *tN = a.tab + OFF_N, *tNT = a.tab + OFF_NT, *tD = a.tab + OFF_D, *tDT = a.tab + OFF_DT;
  const TC *tGW = a.tab + OFF_GW, *tKW = a.tab + OFF_KW;
  const int p = a.p;
  const int ax = colour_of(cx, a.N0), by = colour_of(cy, a.N1);
  const int axl = colour_of(cx == 0 ? a.N0 - 1 : cx - 1, a.N0);
  const int axr = colour_of(cx == a.N0 - 1 ? 0 : cx + 1, a.N0);
  const int byl = colour_of(cy == 0 ? a.N1 - 1 : cy - 1, a.N1);
  const int byr = colour_of(cy == a.N1 - 1 ? 0 : cy + 1, a.N1);

  // this thread's block elements e = tid + r NT: the x/y part of the node
  // index, and packed {plane k, lane offset v, in range, read-modify-write,
  // place (i, j) in a side block's plane}
  int exy[XPT], emeta[XPT];
#pragma unroll
  for (int r = 0; r < XPT; ++r) {
    const int e = tid + r * NT;
    const int v = (e % NV) * LPE, n = e / NV;
    const int i = n % NP, j = (n / NP) % NP;
    // periodic axes wrap; a Dirichlet axis numbers its interior nodes g - 1
    // and has no DoF on its faces (such nodes are gathered as zero and not
    // stored)
    int gx = cx * p + i, gy = cy * p + j;
    bool inb = true;
    if (a.dmask & 1) { gx -= 1; inb = inb && gx >= 0 && gx < a.M0; } else if (gx >= a.M0) gx -= a.M0;
    if (a.dmask & 2) { gy -= 1; inb = inb && gy >= 0 && gy < a.M1; } else if (gy >= a.M1) gy -= a.M1;
    exy[r] = gx + a.M0 * gy;
    const bool xs = (i == 0) || (i == NP - 1), ys = (j == 0) || (j == NP - 1);
    const int axo = (i == 0) ? axl : axr, byo = (j == 0) ? byl : byr;
    const bool rmw = !((!xs || ax < axo) && (!ys || by < byo));
    const bool ok = e < NP3 * NV && lane0 + v < a.nlanes && inb;
    emeta[r] = (n / NP2) | (v << 4) | (ok ? 1 << 12 : 0) | (rmw ? 1 << 13 : 0) | ((i * NP + j) << 14);
  }
  auto ek = [&](int r) { return emeta[r] & 15; };
  auto elane = [&](int r) { return lane0 + ((emeta[r] >> 4) & 255); };
  auto eok = [&](int r) { return (emeta[r] >> 12) & 1; };
  auto ermw = [&](int r) { return (emeta[r] >> 13) & 1; };
  const int64_t MM = (int64_t)a.M0 * a.M1;
  const int zoff = (a.dmask & 4) ? 1 : 0;
  auto node_of = [&](int r, int cz) -> int64_t {
    int gz = cz * p + ek(r) - zoff;
    if (!zoff && gz >= a.M2) gz -= a.M2;
    return (int64_t)exy[r] + MM * gz;
  };
  // this column's plane of half 0 (a segment's first plane) or 1 (the last plane
  // of the one below) of cut sg (layout at side_seg_bytes)
  const int side_lanes = a.ntiles * VT;
  auto side_at = [&](int sg, int half) {
    return a.side + half * a.side_half + ((int64_t)sg * (a.N0 * a.N1) + cx + a.N0 * cy) * NP2 * side_lanes;
  };
  // plane k of cell cz holds DoFs (always on a periodic a_2)
  auto zin = [&](int k, int cz) { const int gz = cz * p + k - zoff; return !zoff || (gz >= 0 && gz < a.M2); };

  for (int t = tid; t < NQ2; t += NT) W2[t] = a.wq[t];
  // dpre: the node's D^-1 entry (filter steps), applied when the block is
  // staged so that its load stays in flight with the others
  TC xpre[XPT][LPE], dpre[XPT], cpre[CPT], ypre[XPT][LPE];
  auto prefetch = [&](int cz) {
#pragma unroll
    for (int r = 0; r < XPT; ++r) {
#pragma unroll
      for (int jj = 0; jj < LPE; ++jj) xpre[r][jj] = 0;
      dpre[r] = 0;
      if (eok(r) && zin(ek(r), cz)) {
        const int64_t g = node_of(r, cz);
        VecIO<TS, TC, LPE>::ld(X + g * a.ldx + elane(r), xpre[r]);
        if (a.dinv) dpre[r] = (TC)a.dinv[g];
      }
    }
    const TC *src = a.coef + (cx + (int64_t)a.N0 * (cy + (int64_t)a.N1 * cz)) * a.coef_cell;
    const int nst = (a.ncoef < NCF ? a.ncoef : NCF) * NQ3;   // the blocks this instance reads
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
      const int e = tid + r * NT;
      cpre[r] = e < nst ? src[e] : (TC)0;
    }
  };
  const bool one = a.nseg == 1;
  TC *const side0 = side_at(seg, 0), *const side1 = side_at(seg + 1 < a.nseg ? seg + 1 : 0, 1);
  prefetch(c0);

  for (int cz = c0; cz < c1; ++cz) {
    // stage X^(e) = Q^(e) X -> A[k][j][i][lane] and the coefficients -> Cf
#pragma unroll
    for (int r = 0; r < XPT; ++r) {
      const int e = tid + r * NT;
      if (a.dinv) {
#pragma unroll
        for (int jj = 0; jj < LPE; ++jj) xpre[r][jj] *= dpre[r];
      }
      if (e < NP3 * NV) LdsVec<TC, LPE>::st(A + e * LPE, xpre[r]);
    }
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
      const int e = tid + r * NT;
      if (e < NCF * NQ3) Cf[e] = cpre[r];
    }
    const int kskip0 = (one && cz == 0) ? 0 : -1;      // plane held back for the wrap
    const int kskip1 = (cz < c1 - 1) ? NP - 1 : -1;    // plane carried to the next cell
    // planes of this cell at a cut, which go to the side block
    auto at_cut = [&](int k) { return !one && ((k == 0 && cz == c0) || (k == NP - 1 && cz == c1 - 1)); };
    __syncthreads();
    // Y0 = (N x N x N) X^(e): along x and y
    line_pass<NP, NQ, 1, VT, NT>(A, B, tN, NP2, [](int l, int &sb, int &ss, int &db, int &ds) {
      sb = l * NP; ss = 1; db = l * NQ; ds = 1; });
    __syncthreads();
    line_pass<NP, NQ, 1, VT, NT>(B, A, tN, NP * NQ, [](int l, int &sb, int &ss, int &db, int &ds) {
      const int k = l / NQ, q1 = l % NQ;
      sb = k * NP * NQ + q1; ss = NQ; db = k * NQ2 + q1; ds = NQ; });
    __syncthreads();
    // next cell's block and coefficients, and the values this cell will
    // read-modify-write (stored by earlier phases), in flight from here on
    auto prefetch_next = [&]() {
      if (cz + 1 < c1) prefetch(cz + 1);
#pragma unroll
      for (int r = 0; r < XPT; ++r) {
#pragma unroll
        for (int jj = 0; jj < LPE; ++jj) ypre[r][jj] = 0;
        if (eok(r) && ermw(r) && ek(r) != kskip0 && ek(r) != kskip1 && zin(ek(r), cz) && !at_cut(ek(r)))
          VecIO<TS, TC, LPE>::ld(Y + node_of(r, cz) * a.ldy + elane(r), ypre[r]);
      }
    };
    // every sweep its own pass; the off-diagonal metric needs all three
    // gradients at a point, staged in T3 first
    auto separate_passes = [&](auto offd_tag) {
      constexpr bool OFFD = decltype(offd_tag)::value;
      line_pass<NP, NQ, 1, VT, NT>(A, B, tN, NQ2, [](int l, int &sb, int &ss, int &db, int &ds) {
        sb = l; ss = NQ2; db = l; ds = NQ2; });
      __syncthreads();
      if constexpr (OFFD) {
        grad_pass<NQ, VT, NT>(B, T3, tD);
        __syncthreads();
      }
      dir_pass<0, NQ, VT, CPLX, TC, OFFD, NT>(B, A, tD, tDT, tGW, tKW, a, Cf, W2, lane0, T3);
      __syncthreads();
      dir_pass<1, NQ, VT, CPLX, TC, OFFD, NT>(B, A, tD, tDT, tGW, tKW, a, Cf, W2, lane0, T3);
      __syncthreads();
      dir_pass<2, NQ, VT, CPLX, TC, OFFD, NT>(B, A, tD, tDT, tGW, tKW, a, Cf, W2, lane0, T3);
      prefetch_next();
      __syncthreads();
      // Y^(e) = (N x N x N)^T Z: along z (A -> B), y (B -> A), x (A -> B)
      line_pass<NQ, NP, 1, VT, NT>(A, B, tNT, NQ2, [](int l, int &sb, int &ss, int &db, int &ds) {
        sb = l; ss = NQ2; db = l; ds = NQ2; });
      __syncthreads();
      line_pass<NQ, NP, 1, VT, NT>(B, A, tNT, NP * NQ, [](int l, int &sb, int &ss, int &db, int &ds) {
        const int k = l / NQ, q1 = l % NQ;
        sb = k * NQ2 + q1; ss = NQ; db = k * NP * NQ + q1; ds = NQ; });
      __syncthreads();
      line_pass<NQ, NP, 1, VT, NT>(A, B, tNT, NP2, [](int l, int &sb, int &ss, int &db, int &ds) {
        sb = l * NQ; ss = 1; db = l * NP; ds = 1; });
      __syncthreads();
    };
    if constexpr (SH) {
      if (a.offd) separate_passes(std::true_type{});
      else separate_passes(std::false_type{});
    } else {
      separate_passes(std::false_type{});
    }
    // node planes shared along a_2: plane 0 takes the carry, plane NP-1 is
    // carried (or, in the last cell, takes the column's first plane)
    for (int t = tid; t < NP2 * VT; t += NT) {
      TC *top = B + (NP - 1) * NP2 * VT;
      if (cz != c0) B[t] += Ycar[t];
      else if (one) Yfst[t] = B[t];
      if (one && cz == a.N2 - 1) top[t] += (cz == 0) ? B[t] : Yfst[t];
    }
    __syncthreads();
    if (cz < c1 - 1)
      for (int t = tid; t < NP2 * VT; t += NT) Ycar[t] = B[(NP - 1) * NP2 * VT + t];
    // write the completed planes: store (first phase) or read-modify-write
#pragma unroll
    for (int r = 0; r < XPT; ++r) {
      if (!eok(r) || ek(r) == kskip0 || ek(r) == kskip1 || !zin(ek(r), cz)) continue;
      const int e = tid + r * NT;
      TC val[LPE], out[LPE];
      LdsVec<TC, LPE>::ld(B + e * LPE, val);
      if (at_cut(ek(r))) {
        TC *q = (ek(r) == 0 ? side0 : side1) + (emeta[r] >> 14) * side_lanes + elane(r);
        if constexpr (LPE * sizeof(TC) == 16) {
          VecIO<TC, TC, LPE>::st(q, val);
        } else {
#pragma unroll
          for (int jj = 0; jj < LPE; ++jj) q[jj] = val[jj];
        }
        continue;
      }
#pragma unroll
      for (int jj = 0; jj < LPE; ++jj) out[jj] = ermw(r) ? ypre[r][jj] + val[jj] : val[jj];
      VecIO<TS, TC, LPE>::st(Y + node_of(r, cz) * a.ldy + elane(r), out);
    }
    __syncthreads();
  }
}

// XCD-aware placement: block b runs on XCD b % 8; each XCD gets a contiguous
// range of work items so the tiles of one column share an L2.  'grid' must be
// a multiple of 8.
__device__ __forceinline__ int xcd_item(int b, int grid) { return (b & 7) * (grid >> 3) + (b >> 3); }

// Register budget: at most 128 VGPRs (4 waves per SIMD), so that two FP64
// blocks of 7 waves, or one FP32/BF16 block of up to 16 waves, are resident
// per CU.  FP64 kernels of degree 7 and up (or with 8 and more quadrature
// points per direction) hold more live values in the line passes than 128
// registers: they get 256 (2 waves per SIMD) rather than spilling to scratch
// (measured per H X: complex p = 7, 24^3 cells, 512 vectors 90 -> 61 ms;
// real p = 8, 12^3 cells, 256 vectors 7.5 -> 3.7 ms).
template <int NP, int NQ, typename TC> struct LocalWaves {
  static constexpr int value = std::is_same<TC, double>::value && (NP >= 7 || NQ >= 8) ? 2 : 4;
};
#define FEHX_LOCAL_BOUNDS __launch_bounds__((BlockSize<NQ, VT, TC>::value)) __attribute__((amdgpu_waves_per_eu(LocalWaves<NP, NQ, TC>::value)))

template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, int LPE, bool SH>
__device__ __forceinline__ void local_item(const KArgs<TC> &a, int w) {
  const int cs = w / a.ntiles, tile = w - cs * a.ntiles;
  const int col = cs / a.nseg;
  local_column<NP, NQ, VT, CPLX, TS, TC, LPE, SH>(a, col, cs - col * a.nseg, tile);
}

// The planes of Y at the cuts: per node the one to four columns that hold it
// in the order of their colour phases, each with the sum of its two halves and
// each sum so far rounded to the block's type, which is what uncut columns do.
// The plane kernels begin at zero and, where the block has the arithmetic's
// type, meet the halves of the column's own wrap (cut 0) one after the other.
// A node of a cut's plane is 2^tl threads of two lanes, as few as hold its
// lanes up to a wave; its loads are in flight together.  Bound by reading the
// two halves, much of it from the caches: eleven cuts of 11 x 13 columns of 7
// points x 101 FP64 lanes, 175 MB, 19 us; eight systems of 7^3 cells x 48 lanes
// 28 us (a wave per node took 24.5 and 68).
constexpr int JOIN_MAXB = 16, JOIN_THREADS = 256;
template <typename TS, typename TC> struct JoinArgs {
  struct {
    TS *Y;
    const TC *side;
    int64_t side_half, ldy;
    int M0, M1, N0, N1, N2, p, dmask, nseg, side_lanes, nlanes;
  } sys[JOIN_MAXB];
  int tl;
  int planes;
  int segs;                                      // along the grid's z, per system
  unsigned rsegs, rp;                            // 2^32 / segs, 2^32 / p, rounded up: quotients by __umulhi
};
template <typename TS, typename TC> __global__ void __launch_bounds__(JOIN_THREADS) k_planes_join(JoinArgs<TS, TC> J) {
  typedef TC Two __attribute__((ext_vector_type(2)));
  const int zs = __umulhi(blockIdx.z, J.rsegs), sg = blockIdx.z - zs * J.segs;
  const auto &a = J.sys[zs];
  const int gx = (blockIdx.x * JOIN_THREADS + threadIdx.x) >> J.tl, gy = blockIdx.y;
  if (gx >= a.M0 || gy >= a.M1 || sg >= a.nseg) return;
  const int64_t gz = (int64_t)((unsigned)(sg * a.N2) / (unsigned)a.nseg) * a.p - (a.dmask & 4 ? 1 : 0);
  if (gz < 0) return;                            // a Dirichlet face: no DoFs
  // the cells of a node along an axis, the lower colour first, and its index in each
  auto cells = [&](int g, int n, int (&c)[2], int (&i)[2]) {
    c[0] = c[1] = __umulhi((unsigned)g, J.rp);
    i[0] = i[1] = g - c[0] * a.p;
    if (i[0]) return 1;
    const int left = c[0] == 0 ? n - 1 : c[0] - 1;
    const bool swap = colour_of(left, n) < colour_of(c[0], n);
    c[0] = swap ? left : c[1];
    i[0] = swap ? a.p : 0;
    c[1] = swap ? c[1] : left;
    i[1] = swap ? 0 : a.p;
    return 2;
  };
  int cx[2], ix[2], cy[2], iy[2];
  const int nx = cells(gx + (a.dmask & 1), a.N0, cx, ix);
  const int ny = cells(gy + ((a.dmask >> 1) & 1), a.N1, cy, iy);
  const int NP = a.p + 1, n = nx * ny;
  const int64_t cut = (int64_t)a.N0 * a.N1 * NP * NP * a.side_lanes;
  auto at = [&](int x, int y) {
    return a.side + sg * cut + ((int64_t)((cx[x] + a.N0 * cy[y]) * NP + ix[x]) * NP + iy[y]) * a.side_lanes;
  };
  // in phase order: x within y
  const TC *const s[4] = {at(0, 0), nx == 2 ? at(1, 0) : at(0, ny - 1), at(0, ny - 1), at(nx - 1, ny - 1)};
  const bool apart = J.planes && sizeof(TS) == sizeof(TC) && sg == 0;
  TS *q = a.Y + (gz * ((int64_t)a.M0 * a.M1) + gx + (int64_t)a.M0 * gy) * a.ldy;
  const int step = 2 << J.tl;
  for (int l = 2 * (threadIdx.x & ((1 << J.tl) - 1)); l < a.nlanes; l += step) {
    Two up[4], lo[4];
    auto load = [&](int k) {
      up[k] = *(const Two *)(s[k] + l);
      lo[k] = *(const Two *)(s[k] + a.side_half + l);
    };
    load(0);
    if (n > 1) load(1);
    if (n > 2) {
      load(2);
      load(3);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      TS sum;
      auto add = [&](int k) {
        const TC u = j ? up[k].y : up[k].x, v = j ? lo[k].y : lo[k].x;
        const TC old = k == 0 ? (TC)0 : Cvt<TS, TC>::ld(&sum, 0);
        Cvt<TS, TC>::st(&sum, 0, apart ? (old + u) + v : k == 0 && !J.planes ? u + v : old + (u + v));
      };
      add(0);
      if (n > 1) add(1);
      if (n > 2) {
        add(2);
        add(3);
      }
      if (l + j < a.nlanes) q[l + j] = sum;
    }
  }
}

// One system, one colour phase: one block per (column, segment, tile).
template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, int LPE, bool SH>
__global__ void FEHX_LOCAL_BOUNDS k_local(KArgs<TC> a) {
  const int w = xcd_item(blockIdx.x, gridDim.x);
  if (w >= a.ncols * a.nseg * a.ntiles) return;
  local_item<NP, NQ, VT, CPLX, TS, TC, LPE, SH>(a, w);
}

// Several systems of one class (n_p, n_q, precision, real/complex), one colour
// phase each, in one persistent launch: the blocks stride over the
// concatenated work lists (system s owns items [off[s], off[s+1])).
constexpr int LOCAL_MAXB = 8;
template <typename TC> struct BatchArgs {
  int nsys, total;
  int off[LOCAL_MAXB + 1];
  KArgs<TC> sys[LOCAL_MAXB];
};

template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, int LPE, bool SH>
__global__ void FEHX_LOCAL_BOUNDS k_local_batch(BatchArgs<TC> B) {
  for (int base = 0; base < B.total; base += gridDim.x) {
    const int w = base + xcd_item(blockIdx.x, gridDim.x);
    if (w >= B.total) return;
    int sidx = 0;
    while (sidx + 1 < B.nsys && w >= B.off[sidx + 1]) ++sidx;
    local_item<NP, NQ, VT, CPLX, TS, TC, LPE, SH>(B.sys[sidx], w - B.off[sidx]);
  }
}

// ---- host-side dispatch (templates; instantiated per precision) -------------

template <typename TC> KArgs<TC> make_args(Mesh *m, const LocalLaunch &L, int vt) {
  KArgs<TC> a{};
  a.X = L.X; a.Y = L.Y; a.ldx = L.ldx; a.ldy = L.ldy; a.nlanes = L.nlanes;
  a.N0 = m->N[0]; a.N1 = m->N[1]; a.N2 = m->N[2];
  a.M0 = m->Mn[0]; a.M1 = m->Mn[1]; a.M2 = m->Mn[2]; a.p = m->p;
  a.dmask = (m->desc.periodic[0] ? 0 : 1) | (m->desc.periodic[1] ? 0 : 2) | (m->desc.periodic[2] ? 0 : 4);
  a.offd = (m->offd && !L.mass) ? 1 : 0;
  const bool f64 = std::is_same<TC, double>::value;
  a.tab = f64 ? (const TC *)m->tab64 : (const TC *)m->tab32;
  a.wq = f64 ? (const TC *)m->wq64 : (const TC *)m->wq32;
  a.coef = f64 ? (const TC *)m->coef64 : (const TC *)m->coef32;
  a.coef_cell = (int64_t)m->ncoef * m->nq * m->nq * m->nq;
  a.ncoef = m->ncoef;
  a.gga = m->has_gga ? 1 : 0;
  if (L.mass) {
    a.tab = f64 ? (const TC *)m->tabM64 : (const TC *)m->tabM32;
    a.coef = f64 ? (const TC *)m->coefM64 : (const TC *)m->coefM32;
    a.coef_cell = m->coefM_cell;
    a.gga = 0;
  }
  a.ptab = f64 ? (const TC *)m->ptab64 : (const TC *)m->ptab32;
  const PlaneTab pt = plane_tab(m->np, m->nq);
  a.pgather = a.ptab + (L.dinv_gather ? pt.nd : pt.n);
  a.pcoef = f64 ? (const TC *)m->pcoef64 : (const TC *)m->pcoef32;
  const double ps = f64 ? 1.0 : m->pscale32;
  for (int d = 0; d < 3; ++d) a.pkap[d] = (TC)(m->pkap[d] / (ps * ps * ps));
  a.nseg = 1;
  a.dinv = L.dinv_gather;
  a.ntiles = (L.nlanes + vt - 1) / vt;
  return a;
}

// Arguments of every system with its segments, count(mesh, launch, tiles, bytes
// of side block), and its part of the side block: where the systems of a batch
// want more than one holds, each in proportion.  segments_end forms the planes
// at the cuts.
template <typename TC, typename Count>
inline void segments_begin(const LocalBatch &Bt, int vt, Count count, std::vector<KArgs<TC>> &as, SideUse &use, hipStream_t s) {
  auto seg_bytes = [&](int i) { return side_seg_bytes(Bt.ms[i], (int64_t)as[i].ntiles * vt, sizeof(TC)); };
  int64_t want = 0;
  for (int i = 0; i < Bt.n; ++i) {
    as.push_back(make_args<TC>(Bt.ms[i], Bt.Ls[i], vt));
    as[i].nseg = count(Bt.ms[i], Bt.Ls[i], as[i].ntiles, side_limit(Bt.Ls[i]));
    as[i].side = (TC *)Bt.Ls[i].side;
    as[i].side_half = Bt.Ls[i].side_bytes / 2 / (int64_t)sizeof(TC);
    if (as[i].nseg > 1 && !as[i].side) want += as[i].nseg * seg_bytes(i);
  }
  if (want == 0) return;
  int64_t half = 0;
  char *next = (char *)use.take(Bt.ms[0]->device, s, &half);
  for (int i = 0; i < Bt.n; ++i) {
    if (as[i].nseg == 1 || as[i].side) continue;
    if (next && want > SIDE_BYTES)
      as[i].nseg = count(Bt.ms[i], Bt.Ls[i], as[i].ntiles, (int64_t)((double)as[i].nseg * seg_bytes(i) / want * SIDE_BYTES));
    if (!next) as[i].nseg = 1;
    if (as[i].nseg == 1) continue;
    as[i].side = (TC *)next;
    as[i].side_half = half / (int64_t)sizeof(TC);
    next += as[i].nseg * seg_bytes(i) / 2;
  }
}
template <typename TS, typename TC>
inline fe_status segments_end(int vt, const std::vector<KArgs<TC>> &as, bool planes, hipStream_t s) {
  for (size_t i = 0; i < as.size();) {
    JoinArgs<TS, TC> J{};
    J.planes = planes;
    unsigned n = 0, mx = 0, my = 0;
    int lanes = 0;
    for (; i < as.size() && n < JOIN_MAXB; ++i) {
      const KArgs<TC> &a = as[i];
      if (a.nseg == 1) continue;
      J.sys[n++] = {(TS *)a.Y, a.side, a.side_half, a.ldy, a.M0, a.M1, a.N0, a.N1, a.N2, a.p, a.dmask, a.nseg, a.ntiles * vt, a.nlanes};
      mx = std::max(mx, (unsigned)a.M0);
      my = std::max(my, (unsigned)a.M1);
      J.segs = std::max(J.segs, a.nseg);
      lanes = std::max(lanes, a.nlanes);
      J.rp = (unsigned)((1ULL << 32) / a.p + 1);   // one degree per launch
    }
    if (n == 0) continue;
    J.rsegs = (unsigned)((1ULL << 32) / J.segs + 1);
    while (J.tl < 6 && 2 << J.tl < lanes) ++J.tl;
    const unsigned nodes = JOIN_THREADS >> J.tl;
    hipLaunchKernelGGL((k_planes_join<TS, TC>), dim3((mx + nodes - 1) / nodes, my, n * J.segs), dim3(JOIN_THREADS), 0, s, J);
    FE_HIP_TRY(hipGetLastError());
  }
  return FE_OK;
}

// LDS per workgroup on gfx950; tiles whose block cannot fit are not instantiated
constexpr size_t LDS_MAX = 160 * 1024;
template <int NP, int NQ> constexpr size_t lds_need(int vt, int bytes, bool offd = false) {
  return ((size_t)(2 * NQ * NQ * NQ + 2 * NP * NP) * vt + (offd ? NCOEF_GEN : 4) * NQ * NQ * NQ + NQ * NQ +
          (offd ? (size_t)3 * NQ * NQ * NQ * vt : 0)) * bytes;
}

// Single system: one launch per colour phase, one block per (column, tile).
// Batch (several systems of one class, or persistent=true): one persistent
// launch per colour phase over the concatenated work lists of up to
// LOCAL_MAXB systems, grid = the resident block count (rounded to 8 XCDs).
inline int max_lds(Mesh *m) {
  int maxshm = 65536;
  (void)hipDeviceGetAttribute(&maxshm, hipDeviceAttributeMaxSharedMemoryPerBlock, m->device);
  return maxshm;
}

template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, int LPE, bool SH>
inline fe_status run_local_lpe(const LocalBatch &Bt, hipStream_t s) {
  // sheared boxes add the three staged gradients to the LDS block; a launch
  // above 64 KiB raises the kernel's dynamic-LDS attribute to its size first
  bool offd = false;
  for (int i = 0; i < Bt.n; ++i) offd = offd || (Bt.ms[i]->offd && !Bt.Ls[i].mass);
  const size_t shm = lds_need<NP, NQ>(VT, sizeof(TC), offd);
  constexpr int NTB = BlockSize<NQ, VT, TC>::value;
  std::vector<KArgs<TC>> as;
  SideUse use;
  auto count = [](int per_cu) {      // blocks of this kernel on a CU
    return [per_cu](Mesh *m, const LocalLaunch &, int tiles, int64_t side_bytes) {
      return block_segment_count(m, tiles, per_cu, side_seg_bytes(m, (int64_t)tiles * VT, sizeof(TC)), side_bytes);
    };
  };
  if (Bt.n == 1 && !Bt.persistent) {
    Mesh *m = Bt.ms[0];
    auto kern = k_local<NP, NQ, VT, CPLX, TS, TC, LPE, SH>;
    static size_t attr_set = 65536;
    static int per_cu[2] = {0, 0};   // blocks without / with the staged gradients
    if (shm > attr_set) {
      FE_HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
      attr_set = shm;
    }
    if (!per_cu[offd]) FE_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu[offd], (const void *)kern, NTB, shm));
    segments_begin<TC>(Bt, VT, count(per_cu[offd]), as, use, s);
    KArgs<TC> &a = as[0];
    for (int ph = 0; ph < m->nphase; ++ph) {
      a.cols = m->cols + 2 * m->phase_off[ph];
      a.ncols = m->phase_off[ph + 1] - m->phase_off[ph];
      if (a.ncols == 0) continue;
      const int W = a.ncols * a.nseg * a.ntiles;
      const int nb = ((W + 7) / 8) * 8;
      hipLaunchKernelGGL(kern, dim3(nb), dim3(NTB), shm, s, a);
      FE_HIP_TRY(hipGetLastError());
    }
    return segments_end<TS, TC>(VT, as, false, s);
  }
  auto kern = k_local_batch<NP, NQ, VT, CPLX, TS, TC, LPE, SH>;
  static size_t battr_set = 65536;
  static int resident[2] = {0, 0};   // resident blocks without / with the staged gradients
  if (shm > battr_set) {
    FE_HIP_TRY(hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    battr_set = shm;
  }
  if (!resident[offd]) {
    int per_cu = 0;
    FE_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void *)kern, NTB, shm));
    resident[offd] = (per_cu > 0 ? per_cu : 1) * Bt.ms[0]->cus;
  }
  segments_begin<TC>(Bt, VT, count(std::max(1, resident[offd] / Bt.ms[0]->cus)), as, use, s);
  const int cap = Bt.blocks_per_cu > 0 ? Bt.blocks_per_cu * Bt.ms[0]->cus : resident[offd];
  int nphase = 0;
  for (int i = 0; i < Bt.n; ++i) nphase = nphase > Bt.ms[i]->nphase ? nphase : Bt.ms[i]->nphase;
  for (int ph = 0; ph < nphase; ++ph) {
    for (int i0 = 0; i0 < Bt.n;) {
      BatchArgs<TC> B{};
      B.nsys = 0;
      B.off[0] = 0;
      for (; i0 < Bt.n && B.nsys < LOCAL_MAXB; ++i0) {
        Mesh *m = Bt.ms[i0];
        if (ph >= m->nphase) continue;
        const int ncols = m->phase_off[ph + 1] - m->phase_off[ph];
        if (ncols == 0) continue;
        KArgs<TC> &a = as[i0];
        a.cols = m->cols + 2 * m->phase_off[ph];
        a.ncols = ncols;
        B.sys[B.nsys] = a;
        B.off[B.nsys + 1] = B.off[B.nsys] + ncols * a.nseg * a.ntiles;
        ++B.nsys;
      }
      if (B.nsys == 0) continue;
      B.total = B.off[B.nsys];
      int grid = B.total < cap ? B.total : cap;
      grid = ((grid + 7) / 8) * 8;
      hipLaunchKernelGGL(kern, dim3(grid), dim3(NTB), shm, s, B);
      FE_HIP_TRY(hipGetLastError());
    }
  }
  return segments_end<TS, TC>(VT, as, false, s);
}

// The wide (16-byte) element form when every block of every system allows it.
inline bool wide_ok(const LocalBatch &Bt, int lpe, size_t ts) {
  const uintptr_t al = (uintptr_t)lpe * ts;
  auto ok_block = [&](const void *p, int64_t ld) { return p == nullptr || ((uintptr_t)p % al == 0 && ld % lpe == 0); };
  for (int i = 0; i < Bt.n; ++i) {
    const LocalLaunch &L = Bt.Ls[i];
    if (L.nlanes % lpe != 0 || !ok_block(L.X, L.ldx) || !ok_block(L.Y, L.ldy)) return false;
  }
  return true;
}

template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC, bool SH = false>
inline fe_status run_local(const LocalBatch &Bt, hipStream_t s) {
  constexpr int W = WideLanes<TS>::value;
  if (VT % W == 0 && wide_ok(Bt, W, sizeof(TS))) return run_local_lpe<NP, NQ, VT, CPLX, TS, TC, W, SH>(Bt, s);
  return run_local_lpe<NP, NQ, VT, CPLX, TS, TC, 1, SH>(Bt, s);
}


// Vector tile per precision: the caller's (the autotuner's) choice when it is
// set and fits, else the widest default whose LDS fits.
template <int NP, int NQ, int VT, bool CPLX, typename TS, typename TC>
fe_status run_tile(bool od, const LocalBatch &B, hipStream_t s) {
  if (od) return run_local<NP, NQ, VT, CPLX, TS, TC, true>(B, s);
  // n_q = n_p with a diagonal metric comes here only past what the plane
  // kernels address: one tile
  if constexpr (NP != NQ || VT == 8) return run_local<NP, NQ, VT, CPLX, TS, TC>(B, s);
  return set_error(FE_EUNSUPPORTED, "no local-operator variant for this vector tile");
}

template <int NP, int NQ, bool CPLX>
fe_status pick_vt_f64(const LocalBatch &B, hipStream_t s) {
  const size_t mx = (size_t)max_lds(B.ms[0]);
  bool od = false;   // any system of a sheared box: the staged gradients must fit too
  for (int i = 0; i < B.n; ++i) od = od || (B.ms[i]->offd && !B.Ls[i].mass);
  int vt = NP == NQ && !od ? 8 : B.Ls[0].vt ? B.Ls[0].vt
                      : (lds_need<NP, NQ>(8, 8, od) <= mx ? 8 : (lds_need<NP, NQ>(4, 8, od) <= mx ? 4 : 2));
  if constexpr (lds_need<NP, NQ>(16, 8) <= LDS_MAX)
    if (vt == 16 && lds_need<NP, NQ>(16, 8, od) <= mx)
      return run_tile<NP, NQ, 16, CPLX, double, double>(od, B, s);
  if constexpr (NP == NQ && lds_need<NP, NQ>(10, 8) <= LDS_MAX)
    if (vt == 10 && lds_need<NP, NQ>(10, 8, od) <= mx)
      return run_tile<NP, NQ, 10, CPLX, double, double>(od, B, s);
  if constexpr (lds_need<NP, NQ>(8, 8) <= LDS_MAX)
    if (vt == 8 && lds_need<NP, NQ>(8, 8, od) <= mx)
      return run_tile<NP, NQ, 8, CPLX, double, double>(od, B, s);
  if constexpr (lds_need<NP, NQ>(4, 8) <= LDS_MAX)
    if (vt == 4 && lds_need<NP, NQ>(4, 8, od) <= mx)
      return run_tile<NP, NQ, 4, CPLX, double, double>(od, B, s);
  // two lanes (one complex vector): only where four do not fit (n_q = 12)
  if constexpr (lds_need<NP, NQ>(4, 8) > LDS_MAX && lds_need<NP, NQ>(2, 8) <= LDS_MAX)
    if (vt == 2 && lds_need<NP, NQ>(2, 8, od) <= mx)
      return run_tile<NP, NQ, 2, CPLX, double, double>(od, B, s);
  return set_error(FE_EUNSUPPORTED, "no FP64 local-operator variant for this vector tile / LDS size");
}
template <int NP, int NQ, bool CPLX>
fe_status pick_vt_f32(const LocalBatch &B, hipStream_t s) {
  const size_t mx = (size_t)max_lds(B.ms[0]);
  bool od = false;   // any system of a sheared box: the staged gradients must fit too
  for (int i = 0; i < B.n; ++i) od = od || (B.ms[i]->offd && !B.Ls[i].mass);
  int vt = NP == NQ && !od ? 8 : B.Ls[0].vt ? B.Ls[0].vt : (lds_need<NP, NQ>(16, 4, od) <= mx ? 16 : 8);
  if constexpr (lds_need<NP, NQ>(32, 4) <= LDS_MAX)
    if (vt == 32 && lds_need<NP, NQ>(32, 4, od) <= mx)
      return run_tile<NP, NQ, 32, CPLX, float, float>(od, B, s);
  if constexpr (lds_need<NP, NQ>(16, 4) <= LDS_MAX)
    if (vt == 16 && lds_need<NP, NQ>(16, 4, od) <= mx)
      return run_tile<NP, NQ, 16, CPLX, float, float>(od, B, s);
  if constexpr (lds_need<NP, NQ>(8, 4) <= LDS_MAX)
    if (vt == 8 && lds_need<NP, NQ>(8, 4, od) <= mx)
      return run_tile<NP, NQ, 8, CPLX, float, float>(od, B, s);
  return set_error(FE_EUNSUPPORTED, "no FP32 local-operator variant for this vector tile / LDS size");
}
template <int NP, int NQ, bool CPLX>
fe_status pick_vt_bf16(const LocalBatch &B, hipStream_t s) {
  const size_t mx = (size_t)max_lds(B.ms[0]);
  bool od = false;   // any system of a sheared box: the staged gradients must fit too
  for (int i = 0; i < B.n; ++i) od = od || (B.ms[i]->offd && !B.Ls[i].mass);
  int vt = NP == NQ && !od ? 8 : B.Ls[0].vt ? B.Ls[0].vt : (lds_need<NP, NQ>(32, 4, od) <= mx ? 32 : (lds_need<NP, NQ>(16, 4, od) <= mx ? 16 : 8));
  if constexpr (lds_need<NP, NQ>(32, 4) <= LDS_MAX)
    if (vt == 32 && lds_need<NP, NQ>(32, 4, od) <= mx)
      return run_tile<NP, NQ, 32, CPLX, bf16s, float>(od, B, s);
  if constexpr (lds_need<NP, NQ>(16, 4) <= LDS_MAX)
    if (vt == 16 && lds_need<NP, NQ>(16, 4, od) <= mx)
      return run_tile<NP, NQ, 16, CPLX, bf16s, float>(od, B, s);
  if constexpr (lds_need<NP, NQ>(8, 4) <= LDS_MAX)
    if (vt == 8 && lds_need<NP, NQ>(8, 4, od) <= mx)
      return run_tile<NP, NQ, 8, CPLX, bf16s, float>(od, B, s);
  return set_error(FE_EUNSUPPORTED, "no BF16 local-operator variant for this vector tile / LDS size");
}
template <int NP, int NQ> fe_status pick_cplx_f64(const LocalBatch &B, hipStream_t s) {
  return B.ms[0]->cplx ? pick_vt_f64<NP, NQ, true>(B, s) : pick_vt_f64<NP, NQ, false>(B, s);
}
template <int NP, int NQ> fe_status pick_cplx_f32(const LocalBatch &B, hipStream_t s) {
  return B.ms[0]->cplx ? pick_vt_f32<NP, NQ, true>(B, s) : pick_vt_f32<NP, NQ, false>(B, s);
}
template <int NP, int NQ> fe_status pick_cplx_bf16(const LocalBatch &B, hipStream_t s) {
  return B.ms[0]->cplx ? pick_vt_bf16<NP, NQ, true>(B, s) : pick_vt_bf16<NP, NQ, false>(B, s);
}

}  // namespace fehx
static_assert(sizeof(fehx::BatchArgs<double>) <= 4096, "batched kernel arguments exceed the 4 KB kernarg limit");
