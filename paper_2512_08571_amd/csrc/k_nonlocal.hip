// Nonlocal pseudopotential term of eqn Vnonloc / eqn AXmatrixfreenonloc,
// Y += alpha F diag(h) F^H X, with F the assembled node-level projector matrix
// (the paper's cell blocks F^(a,e) summed over cells).
//
//   k_nl_w    W_partial[chunk][s][lane] = sum over the chunk's support nodes of
//             conj(F[n][s]) X[node][lane]; one workgroup per (node chunk of one
//             atom, 256-lane tile), the chunks run in order of position, each
//             XCD taking a contiguous run of them, so that overlapping atoms'
//             chunks share cached X rows in one L2; the block's row groups
//             split the nodes and are summed in a fixed order
//   k_nl_wsum W[s][lane] = h_s sum over the atom's chunks, in chunk order
//   k_nl_yb   the rows grouped by node bricks: one workgroup per (brick, lane
//             tile) stages the W rows of the brick's projectors in LDS once,
//             then each wave updates one Y row at a time reading W from LDS
//             (W crosses the L2 once per brick instead of once per entry)
//   k_nl_ybm  the FP64 form of the brick update on the matrix cores: the
//             brick's projector values as a dense block times the brick's W
//             rows, v_mfma_f64_16x16x4 over 16-row tiles
//   k_nl_y    the rows no brick of at most NL_BPMAX projectors holds: one wave
//             per row at a time, the row's (projector, value) entries are
//             wave-uniform scalar loads taken eight at a time, W and Y are
//             read and written as 256-lane rows
// Every thread owns four adjacent lanes (one 16/32-byte vector access per
// row when the block is aligned), so a wave moves a whole 256-lane row per
// access and complex (re, im) pairs stay inside one thread.  The vector
// width of these passes is the whole block row (the paper's level-0 batch
// for the nonlocal part of Alg. 1).
#include <algorithm>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "fe_internal.h"

namespace fehx {

struct bf16n { uint16_t b; };
__device__ __forceinline__ float nl_bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t nl_f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
constexpr int NL_THREADS = 256;
constexpr int NL_TILE = 256;    // lanes per wave (4 per thread)
constexpr int NL_W_FEW = 512;   // blocks below which the reduction takes more waves per chunk (launch_nl_w_tl)

// Four adjacent lanes starting at element offset o of a row; VEC: the four
// are in range and 4-element aligned, so one vector access moves them.
// (Pair: the same for two FP64 lanes.)
template <typename TS, typename TC, bool VEC> struct Quad;
template <bool VEC> struct Quad<double, double, VEC> {
  static __device__ __forceinline__ void ld(const double *p, int64_t o, int nv, double v[4]) {
    if (VEC) {
      const double2 a = *(const double2 *)(p + o), b = *(const double2 *)(p + o + 2);
      v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = j < nv ? p[o + j] : 0.0;
    }
  }
  static __device__ __forceinline__ void st(double *p, int64_t o, int nv, const double v[4]) {
    if (VEC) {
      *(double2 *)(p + o) = make_double2(v[0], v[1]);
      *(double2 *)(p + o + 2) = make_double2(v[2], v[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (j < nv) p[o + j] = v[j];
    }
  }
};
template <bool VEC> struct Quad<float, float, VEC> {
  static __device__ __forceinline__ void ld(const float *p, int64_t o, int nv, float v[4]) {
    if (VEC) {
      const float4 a = *(const float4 *)(p + o);
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = j < nv ? p[o + j] : 0.0f;
    }
  }
  static __device__ __forceinline__ void st(float *p, int64_t o, int nv, const float v[4]) {
    if (VEC) {
      *(float4 *)(p + o) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (j < nv) p[o + j] = v[j];
    }
  }
};
template <bool VEC> struct Quad<bf16n, float, VEC> {
  static __device__ __forceinline__ void ld(const bf16n *p, int64_t o, int nv, float v[4]) {
    if (VEC) {
      const uint2 a = *(const uint2 *)(p + o);
      v[0] = __uint_as_float(a.x << 16); v[1] = __uint_as_float(a.x & 0xffff0000u);
      v[2] = __uint_as_float(a.y << 16); v[3] = __uint_as_float(a.y & 0xffff0000u);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = j < nv ? nl_bf2f(p[o + j].b) : 0.0f;
    }
  }
  static __device__ __forceinline__ void st(bf16n *p, int64_t o, int nv, const float v[4]) {
    if (VEC) {
      uint2 a;
      a.x = (uint32_t)nl_f2bf(v[0]) | ((uint32_t)nl_f2bf(v[1]) << 16);
      a.y = (uint32_t)nl_f2bf(v[2]) | ((uint32_t)nl_f2bf(v[3]) << 16);
      *(uint2 *)(p + o) = a;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (j < nv) p[o + j].b = nl_f2bf(v[j]);
    }
  }
};

template <bool VEC> struct Pair {
  static __device__ __forceinline__ void ld(const double *p, int64_t o, int nv, double v[2]) {
    if (VEC) {
      const double2 a = *(const double2 *)(p + o);
      v[0] = a.x; v[1] = a.y;
    } else {
      v[0] = nv > 0 ? p[o] : 0.0;
      v[1] = nv > 1 ? p[o + 1] : 0.0;
    }
  }
  static __device__ __forceinline__ void st(double *p, int64_t o, int nv, const double v[2]) {
    if (VEC) {
      *(double2 *)(p + o) = make_double2(v[0], v[1]);
    } else {
      if (nv > 0) p[o] = v[0];
      if (nv > 1) p[o + 1] = v[1];
    }
  }
};

// Quad load without a branch: elements past nv (>= 1) read others in range, so
// that rows in flight are not separated by conditional blocks.  FP64 in pairs
// needs an even nv only (every complex block).
template <typename TS, typename TC, bool VEC>
__device__ __forceinline__ void quad_ld_clamped(const TS *p, int64_t o, int nv, TC v[4]) {
  if constexpr (VEC && std::is_same<TS, double>::value) {
    const double2 a = *(const double2 *)(p + o), b = *(const double2 *)(p + o + (nv > 2 ? 2 : 0));
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  } else if constexpr (VEC) {
    Quad<TS, TC, true>::ld(p, o, nv, v);
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      TC t[4];
      Quad<TS, TC, false>::ld(p, o + min(j, nv - 1), 1, t);
      v[j] = t[0];
    }
  }
}

// 16 bytes of compute-type lanes per thread in the brick update
template <typename TS, typename TC, bool VEC> struct BrickIO { using T = Quad<TS, TC, VEC>; };
template <bool VEC> struct BrickIO<double, double, VEC> { using T = Pair<VEC>; };

// acc += conj(f) x (complex: lanes (re, im, re, im)) or f x (real)
template <bool CPLX, typename TC>
__device__ __forceinline__ void nl_conj_fma(TC fr, TC fi, const TC x[4], TC acc[4]) {
  if (!CPLX) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = fma(fr, x[j], acc[j]);
  } else {
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      acc[j] = fma(fr, x[j], fma(fi, x[j + 1], acc[j]));
      acc[j + 1] = fma(fr, x[j + 1], fma(-fi, x[j], acc[j + 1]));
    }
  }
}

// One system's projector term as the kernels take it.  A launch covers up to
// NL_GROUP systems (blockIdx.z), so that the small systems of a batch share the
// device: eight k-points of 74,088 DoFs x 48 lanes, reduction 8 x 35 -> 250 us,
// sums 8 x 5 -> 7, update 8 x 36 -> 191.
constexpr int NL_GROUP = 8;
template <typename TS, typename TC> struct NlSys {
  const TS *X;
  TS *Y;
  const double *dinv, *h;
  const TC *F;
  TC *part, *W;                                  // chunk partials [nchunks][NL_MAXP][ldp], W [ns][ldp]
  const int4 *chunks;
  const int *nodes, *atom_chunk0, *proj_off, *proj_atom;
  const int *b_row0, *b_p0, *b_proj, *b_rows, *kb;   // bricks as dense blocks (FP64)
  const int64_t *a_off;
  const double *A;
  int64_t ldx, ldy, ldp;
  int nlanes, nchunks, fstride, ns, nbrick;
  TC alpha;
};
template <typename TS, typename TC> struct NlGroup { NlSys<TS, TC> a[NL_GROUP]; };

// One chunk of one atom's support nodes: a row of the block is moved by TL
// threads (four lanes each), so a wave holds 64 / TL rows at a time and the
// block NW times as many; each group of TL threads takes every (NW 64 / TL)-th
// node, U of them in flight.  The groups of a wave are summed by lane
// exchanges and the waves in LDS, both in a fixed order.  PMAX bounds the
// projectors per atom: it sizes the accumulators.
// What bounds it: reading the rows.  Where the chunks do not fill the device
// the time is the latency of one chunk's chain of row reads, which the node
// indices staged in LDS, the groups and the waves shorten (times at
// launch_nl_w_tl).
template <bool CPLX, typename TS, typename TC, bool VEC, int PMAX, int TL, int NW>
__global__ void __launch_bounds__(64 * NW)
k_nl_w(NlGroup<TS, TC> grp) {
  const NlSys<TS, TC> &a = grp.a[blockIdx.z];
  const TS *__restrict__ X = a.X;
  const double *__restrict__ dinv = a.dinv;
  const int *__restrict__ nodes = a.nodes;
  const TC *__restrict__ F = a.F;
  TC *__restrict__ part = a.part;
  const int64_t ldx = a.ldx, ldp = a.ldp;
  const int nlanes = a.nlanes, fstride = a.fstride;
  constexpr int C = CPLX ? 2 : 1;
  constexpr int TILE = 4 * TL;                   // lanes per block
  constexpr int GW = 64 / TL, G = GW * NW;       // node groups per wave, per block
  constexpr int U = NW == 4 ? 2 : 4;             // nodes in flight per group
  // projectors summed per step: all of them where their sums fit 32 KiB
  constexpr int SB = (int)sizeof(TC) * PMAX * NW * TILE <= 32768 ? PMAX : 1;
  // Projector values, TE entries at a time in LDS (the space of the sums):
  // loaded row by row they were a chain of four to ten per X row and most of
  // the time (27,000 complex DoFs x 66 lanes 47 -> 25 us; eight k-points of
  // 74,088 DoFs x 48 lanes 250 -> 164 us; as scalar loads of a wave's one row,
  // 16^3 cells degree 7, nine projectors, 256 lanes 449 -> 320 us)
  constexpr int TE = PMAX <= 4 ? 512 : 256;
  constexpr int NRED = SB * NW * TILE, NF = TE * PMAX * C;
  __shared__ int snode[NL_CHUNK];
  __shared__ TC space[NRED > NF ? NRED : NF];
  auto red = reinterpret_cast<TC(*)[NW][TILE]>(space);
  // XCD-aware: block x runs on XCD x % 8, and each XCD takes a contiguous run
  // of the position-ordered chunks, so overlapping atoms' chunks share an L2
  const int item = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (item >= a.nchunks || (int)blockIdx.y * TILE >= nlanes) return;   // whole block: before any barrier
  const int4 cd = a.chunks[item];                  // partial slot, first support entry, entries, projectors
  const int ch = cd.x, n0 = cd.y, nn = cd.z, ns = cd.w;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lt = (threadIdx.x & (TL - 1)) * 4;
  const int l0 = blockIdx.y * TILE + lt;
  // lanes past the block read its first ones; they are not stored
  const int nv0 = min(4, nlanes - l0);
  const int lc = nv0 > 0 ? l0 : 0, nv = nv0 > 0 ? nv0 : min(4, nlanes);
  for (int i = threadIdx.x; i < nn; i += 64 * NW) snode[i] = nodes[n0 + i];
  __syncthreads();
  TC acc[PMAX][4];
#pragma unroll
  for (int s = 0; s < PMAX; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[s][j] = 0;
  const int g = wv * GW + (GW > 1 ? (int)((threadIdx.x & 63) / TL) : 0);
  // U rows of this group; TAIL: a group past its last node reads the chunk's
  // last row and takes it as zero, so the trip count is the block's
  int t0 = 0, t1 = 0;                            // the entries at hand
  auto rows = [&](int i0, auto tail_tag) {
    constexpr bool TAIL = decltype(tail_tag)::value;
    TC x[U][4];
    int idx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      idx[u] = i0 + u * G + g;
      if constexpr (TAIL) idx[u] = min(idx[u], t1 - 1);
      int node = snode[idx[u]];
      if constexpr (GW == 1) node = __builtin_amdgcn_readfirstlane(node);
      quad_ld_clamped<TS, TC, VEC>(X, (int64_t)node * ldx + lc, nv, x[u]);
      if (dinv) {
        const TC d = (TC)dinv[node];
#pragma unroll
        for (int j = 0; j < 4; ++j) x[u][j] *= d;
      }
      if constexpr (TAIL)
#pragma unroll
        for (int j = 0; j < 4; ++j) x[u][j] = i0 + u * G + g < t1 ? x[u][j] : (TC)0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const TC *f = space + (idx[u] - t0) * fstride * C;
#pragma unroll
      for (int s = 0; s < PMAX; ++s)
        if (s < ns) nl_conj_fma<CPLX>(f[s * C], CPLX ? f[s * C + 1] : (TC)0, x[u], acc[s]);
    }
  };
  for (; t0 < nn; t0 = t1) {
    t1 = min(nn, t0 + TE);
    if (t0 > 0) __syncthreads();
    const TC *src = F + (int64_t)(n0 + t0) * fstride * C;
    for (int e = threadIdx.x; e < (t1 - t0) * fstride * C; e += 64 * NW) space[e] = src[e];
    __syncthreads();
    int i0 = t0;
    for (; i0 + U * G <= t1; i0 += U * G) rows(i0, std::false_type{});
    if (i0 < t1) rows(i0, std::true_type{});
  }
  __syncthreads();
  // fixed-order sums, SB projectors at a time
#pragma unroll
  for (int s0 = 0; s0 < PMAX; s0 += SB) {
    if (s0 < ns) {
#pragma unroll
      for (int s = s0; s < s0 + SB; ++s) {
#pragma unroll
        for (int o = TL; o < 64; o <<= 1)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[s][j] += __shfl_xor(acc[s][j], o);
        if ((threadIdx.x & 63) < TL)
#pragma unroll
          for (int j = 0; j < 4; ++j) red[s - s0][wv][lt + j] = acc[s][j];
      }
      __syncthreads();
      for (int e = threadIdx.x; e < SB * TILE; e += 64 * NW) {
        const int s = e / TILE, l = e % TILE;
        TC sum = red[s][0][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) sum += red[s][w][l];
        const int glo = blockIdx.y * TILE + l;
        if (glo < nlanes && s0 + s < ns) part[((int64_t)ch * NL_MAXP + s0 + s) * ldp + glo] = sum;
      }
      if (SB < PMAX) __syncthreads();
    }
  }
}

template <typename TS, typename TC>
__global__ void k_nl_wsum(NlGroup<TS, TC> grp) {
  const NlSys<TS, TC> &sys = grp.a[blockIdx.z];
  const TC *__restrict__ part = sys.part;
  const int *__restrict__ atom_chunk0 = sys.atom_chunk0;
  const int nlanes = sys.nlanes;
  const int64_t ldp = sys.ldp;
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= (int64_t)sys.ns * nlanes) return;
  const int s = (int)(t / nlanes), l = (int)(t % nlanes);
  const int a = sys.proj_atom[s];
  const int sl = s - sys.proj_off[a];
  // in chunk order, eight loads in flight
  const int c1 = atom_chunk0[a + 1];
  TC sum = 0;
  for (int c0 = atom_chunk0[a]; c0 < c1; c0 += 8) {
    TC v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[((int64_t)min(c0 + u, c1 - 1) * NL_MAXP + sl) * ldp + l];
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += c0 + u < c1 ? v[u] : (TC)0;
  }
  sys.W[(int64_t)s * ldp + l] = (TC)sys.h[s] * sum;
}

template <bool CPLX, typename TS, typename TC, bool VEC>
__global__ void __launch_bounds__(NL_THREADS)
k_nl_y(TS *__restrict__ Y, int64_t ldy, int nlanes, const int *__restrict__ rows, const int *__restrict__ rowptr,
       const int *__restrict__ colidx, const TC *__restrict__ val, int64_t nrows, const TC *__restrict__ W,
       int64_t ldw, TC alpha) {
  const int l0 = blockIdx.y * NL_TILE + (threadIdx.x & 63) * 4;
  const int nv = min(4, nlanes - l0);
  const bool on = nv > 0;
  constexpr int C = CPLX ? 2 : 1;
  const int64_t wstride = (int64_t)gridDim.x * (NL_THREADS / 64);
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t r = (int64_t)blockIdx.x * (NL_THREADS / 64) + wv; r < nrows; r += wstride) {
    const int e0 = rowptr[r], e1 = rowptr[r + 1];
    const int64_t o = (int64_t)rows[r] * ldy + l0;
    TC y[4] = {0, 0, 0, 0};
    if (on) Quad<TS, TC, VEC>::ld(Y, o, nv, y);        // in flight with the W reads
    TC acc[4] = {0, 0, 0, 0};
    for (int eb = e0; eb < e1; eb += 8) {
      // eight entries at a time: independent W rows keep several loads in flight
      int sidx[8];
      TC vr[8], vi[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool in = eb + u < e1;
        const int e = in ? eb + u : e1 - 1;
        sidx[u] = colidx[e];
        vr[u] = in ? val[(int64_t)e * C] : (TC)0;
        vi[u] = (CPLX && in) ? val[(int64_t)e * C + 1] : (TC)0;
      }
      TC w[8][4];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (on) Quad<TC, TC, VEC>::ld(W, (int64_t)sidx[u] * ldw + l0, nv, w[u]);
        else w[u][0] = w[u][1] = w[u][2] = w[u][3] = 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (!CPLX) {
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = fma(vr[u], w[u][j], acc[j]);
        } else {
          // (vr + i vi)(wr + i wi): re += vr wr - vi wi, im += vr wi + vi wr
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            acc[j] = fma(vr[u], w[u][j], fma(-vi[u], w[u][j + 1], acc[j]));
            acc[j + 1] = fma(vr[u], w[u][j + 1], fma(vi[u], w[u][j], acc[j + 1]));
          }
        }
      }
    }
    if (on) {
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] += alpha * acc[j];
      Quad<TS, TC, VEC>::st(Y, o, nv, y);
    }
  }
}

constexpr int NL_BTHREADS = 1024;
constexpr int NL_YPF = 4;      // Y rows in flight per wave in the brick update

// Y[row] += alpha sum_e val_e W[proj_e] over the rows of one brick.  Each
// thread owns LPT = 16 / sizeof(TC) adjacent lanes (FP64: 2, FP32: 4), so a
// complex (re, im) pair stays in one thread and a wave covers a 64 LPT-lane
// tile; the staged block is np x tile (at most NL_BPMAX x 1 KiB).  A row's
// entries come in groups of four, two groups per step as wave-uniform scalar
// loads.  Blocks are numbered so that the lane tiles of one brick run on one
// XCD (dispatch deals consecutive blocks to the eight XCDs in turn): the
// brick's entry list is fetched from HBM once and then hit in that L2.
template <bool CPLX, typename TS, typename TC, bool VEC>
__global__ void __launch_bounds__(NL_BTHREADS)
k_nl_yb(TS *__restrict__ Y, int64_t ldy, int nlanes, int nbrick, const int *__restrict__ b_row0, const int *__restrict__ b_p0,
        const int *__restrict__ b_proj, const int *__restrict__ b_rows, const int *__restrict__ b_rowptr,
        const int4 *__restrict__ gcol, const TC *__restrict__ gval, const TC *__restrict__ W, int64_t ldw,
        TC alpha) {
  constexpr int LPT = 16 / sizeof(TC);
  constexpr int TILE = 64 * LPT;
  constexpr int C = CPLX ? 2 : 1;
  constexpr int GV = 4 * C;                          // values per group
  constexpr int NW = NL_BTHREADS / 64;
  using IO = typename BrickIO<TS, TC, VEC>::T;
  using IOW = typename BrickIO<TC, TC, VEC>::T;
  extern __shared__ __align__(16) unsigned char nl_smem[];
  TC *Wl = (TC *)nl_smem;
  const int tiles = (nlanes + TILE - 1) / TILE;
  const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3;
  const int b = (rest / tiles) * 8 + xcd, tile = rest % tiles;
  if (b >= nbrick) return;                           // whole block: before any barrier
  const int lt = (threadIdx.x & 63) * LPT;
  const int l0 = tile * TILE + lt;
  const int nv = min(LPT, nlanes - l0);
  const bool on = nv > 0;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p0 = b_p0[b], np = b_p0[b + 1] - p0;
  for (int i = wv; i < np; i += NW) {
    TC w[LPT];
    if (on) IOW::ld(W, (int64_t)b_proj[p0 + i] * ldw + l0, nv, w);
    else
#pragma unroll
      for (int j = 0; j < LPT; ++j) w[j] = 0;
#pragma unroll
    for (int j = 0; j < LPT; ++j) Wl[i * TILE + lt + j] = w[j];
  }
  __syncthreads();
  const TC *Wt = Wl + lt;
  const int r1 = b_row0[b + 1];
  // Each wave's Y rows are read NL_YPF rows ahead, one register slot per
  // row in flight (the row loop is unrolled over the slots, so a pending read
  // is never moved between registers): enough HBM reads in flight per CU to
  // cover their latency.
  // Reads are unconditional so that the waits stay counted: a lane past the
  // block reads the row's first lanes, a slot past the wave's last row reads
  // that row again; neither value is used.
  TC yq[NL_YPF][LPT];
  const int rw = b_row0[b] + wv;
  const int lc = on ? l0 : 0, nc = on ? nv : min(LPT, nlanes);
  if (rw < r1) {
#pragma unroll
    for (int k = 0; k < NL_YPF; ++k) {
      const int rk = min(rw + k * NW, r1 - 1);
      IO::ld(Y, (int64_t)b_rows[rk] * ldy + lc, nc, yq[k]);
    }
  }
  for (int r0 = rw; r0 < r1; r0 += NL_YPF * NW)
#pragma unroll
  for (int q = 0; q < NL_YPF; ++q) {
    const int r = r0 + q * NW;
    if (r >= r1) break;
    const int g0 = b_rowptr[r], g1 = b_rowptr[r + 1];
    TC acc[LPT];
#pragma unroll
    for (int j = 0; j < LPT; ++j) acc[j] = 0;
    for (int g = g0; g < g1; g += 2) {
      // two groups (eight entries) per step: one scalar-load round trip,
      // eight LDS reads in flight
      int cc[8];
      TC vc[2 * GV];
      const int4 ca = gcol[g], cb = gcol[g + 1];
      cc[0] = ca.x; cc[1] = ca.y; cc[2] = ca.z; cc[3] = ca.w;
      cc[4] = cb.x; cc[5] = cb.y; cc[6] = cb.z; cc[7] = cb.w;
#pragma unroll
      for (int k = 0; k < 2 * GV; ++k) vc[k] = gval[(int64_t)g * GV + k];
      TC w[8][LPT];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int j = 0; j < LPT; ++j) w[u][j] = Wt[cc[u] * TILE + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const TC vr = vc[u * C], vi = CPLX ? vc[u * C + 1] : (TC)0;
        if (!CPLX) {
#pragma unroll
          for (int j = 0; j < LPT; ++j) acc[j] = fma(vr, w[u][j], acc[j]);
        } else {
          // (vr + i vi)(wr + i wi): re += vr wr - vi wi, im += vr wi + vi wr
#pragma unroll
          for (int j = 0; j < LPT; j += 2) {
            acc[j] = fma(vr, w[u][j], fma(-vi, w[u][j + 1], acc[j]));
            acc[j + 1] = fma(vr, w[u][j + 1], fma(vi, w[u][j], acc[j + 1]));
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < LPT; ++j) yq[q][j] += alpha * acc[j];
    if (on) IO::st(Y, (int64_t)b_rows[r] * ldy + l0, nv, yq[q]);
    const int rn = r + NL_YPF * NW;
    IO::ld(Y, (int64_t)b_rows[rn < r1 ? rn : r] * ldy + lc, nc, yq[q]);
  }
}

// FP64 brick update on the matrix cores: Y[rows of brick b] += alpha A_b B_b.
// A_b is the brick's dense projector block (rows x K_b, columns (p, re) and
// (p, im) for complex, zero-padded to a multiple of 4); B_b (K_b x 64 lanes,
// staged in LDS) holds the W rows of the brick's projectors, the (p, im) row
// as i W_p, so that one real product yields both parts of F W:
//   re += Fr Wr + Fi (-Wi),  im += Fr Wi + Fi Wr.
// One workgroup per (brick, 64-lane tile, part of the row tiles); each wave
// takes 16-row tiles and accumulates four 16 x 16 column blocks over K with v_mfma_f64_16x16x4
// (operands: lane l holds A[l & 15][l >> 4] and B[l >> 4][l & 15]; item v of
// the result is row (l >> 4) + 4 v, column l & 15).  The K order is fixed, so
// the update is reproducible bit for bit.  The four A values of a step come
// eight steps at a time, so one load latency covers 32 columns of K.
constexpr int NL_MT = 512;   // threads of the matrix-core brick update
constexpr int NL_MN = 64;    // lanes per workgroup tile
typedef double nl_v4d __attribute__((ext_vector_type(4)));
// the staged block (at most 2 NL_BPMAX rows of 64 lanes) must stay within the
// 64 KiB of dynamic LDS a launch gets without a function attribute
static_assert(2 * NL_BPMAX * NL_MN * sizeof(double) <= 65536, "k_nl_ybm's LDS block exceeds 64 KiB");

template <bool CPLX>
__global__ void __launch_bounds__(NL_MT)
k_nl_ybm(NlGroup<double, double> grp, int parts) {
  const NlSys<double, double> &sys = grp.a[blockIdx.z];
  double *__restrict__ Y = sys.Y;
  const int *__restrict__ b_row0 = sys.b_row0, *__restrict__ b_p0 = sys.b_p0, *__restrict__ b_proj = sys.b_proj;
  const int *__restrict__ b_rows = sys.b_rows;
  const double *__restrict__ W = sys.W;
  const int64_t ldy = sys.ldy, ldw = sys.ldp;
  const int nlanes = sys.nlanes;
  const double alpha = sys.alpha;
  constexpr int NCB = NL_MN / 16;
  constexpr int NW = NL_MT / 64;
  extern __shared__ __align__(16) unsigned char nl_smem[];
  double *Bl = (double *)nl_smem;
  const int tiles = (nlanes + NL_MN - 1) / NL_MN;
  const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3;   // a brick's tiles on one XCD, as in k_nl_yb
  const int part = rest % parts, bt = rest / parts;
  const int b = (bt / tiles) * 8 + xcd, tile = bt % tiles;
  if (b >= sys.nbrick || part * 16 >= b_row0[b + 1] - b_row0[b]) return;   // whole block: before any barrier
  const int n0 = tile * NL_MN;
  const int p0 = b_p0[b], np = b_p0[b + 1] - p0, K = sys.kb[b];
  for (int e = threadIdx.x; e < K * NL_MN; e += NL_MT) {
    const int k = e / NL_MN, j = e - k * NL_MN;
    const int p = CPLX ? k >> 1 : k;
    double v = 0.0;
    if (p < np && n0 + j < nlanes) {          // complex: nlanes even, so n0 + (j | 1) < nlanes too
      const double *w = W + (int64_t)b_proj[p0 + p] * ldw + n0;
      if (!CPLX || !(k & 1)) v = w[j];
      else v = (j & 1) ? w[j - 1] : -w[j + 1];
    }
    Bl[e] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i = lane & 15, kq = lane >> 4;
  const int r0 = b_row0[b], R = b_row0[b + 1] - r0;
  const double *__restrict__ Ab = sys.A + sys.a_off[b];
  for (int mt = wv * parts + part; mt * 16 < R; mt += NW * parts) {
    // this tile's Y values (rows past the brick read its last row, columns
    // past the block its last column; neither is written back)
    double y[4][NCB];
    int64_t yo[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      yo[v] = (int64_t)b_rows[r0 + min(mt * 16 + kq + 4 * v, R - 1)] * ldy;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) y[v][cb] = Y[yo[v] + min(n0 + cb * 16 + i, nlanes - 1)];
    }
    nl_v4d acc[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) acc[cb] = (nl_v4d){0.0, 0.0, 0.0, 0.0};
    const bool arow = mt * 16 + i < R;
    const double *ap = Ab + (int64_t)min(mt * 16 + i, R - 1) * K + kq;
    for (int k0 = 0; k0 < K; k0 += 32) {
      double a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = (arow && k0 + 4 * u < K) ? ap[k0 + 4 * u] : 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (k0 + 4 * u >= K) break;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], Bl[(k0 + 4 * u + kq) * NL_MN + cb * 16 + i],
                                                         acc[cb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (mt * 16 + kq + 4 * v >= R) continue;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const int col = n0 + cb * 16 + i;
        if (col < nlanes) Y[yo[v] + col] = y[v][cb] + alpha * acc[cb][v];
      }
    }
  }
}

namespace {
// the extents a launch over a group needs
struct NlExtent {
  int n = 0, nlanes = 0, nchunks = 0, kmax = 0, form = 0;
  int64_t bricks = 0, nw = 0;   // brick groups and W entries of the largest system
};

template <bool CPLX, typename TS, typename TC, bool VEC, int PMAX, int TL, int NW>
void launch_nl_w_as(const NlGroup<TS, TC> &g, const NlExtent &e, hipStream_t s) {
  const int tiles = (e.nlanes + 4 * TL - 1) / (4 * TL);
  const unsigned gx = (unsigned)(e.nchunks + 7) / 8 * 8;   // a multiple of the 8 XCDs
  hipLaunchKernelGGL((k_nl_w<CPLX, TS, TC, VEC, PMAX, TL, NW>), dim3(gx, tiles, e.n), dim3(64 * NW), 0, s, g);
}

// The narrowest row group that holds the lanes: 32 lanes on eight threads move
// eight rows per wave access where one row per access left 56 of 64 threads
// idle (FP64, 31,500 DoFs x 32 lanes: 190 -> 15 us; eight complex atoms,
// 74,088 DoFs x 48 lanes: 213 -> 35 us).  Sixteen waves per
// chunk where the chunks do not fill the device: about 130 chunks x 128 FP64
// lanes 217 -> 79 us, 270 chunks x 192 FP32 lanes 333 -> 286 us (beside the
// local launches); with 940 chunks x 256 FP64 lanes the device is full and
// four waves are the faster (392 us; sixteen waves 11% slower), so the line
// lies at two blocks per CU.  The form fixes the summation order, so it is each
// system's own also where systems share a launch.
int nl_w_form(const Mesh *m, int nlanes) {
  const int f = nlanes <= 32 ? 0 : nlanes <= 64 ? 1 : nlanes <= 128 ? 2
                : (int64_t)m->nl_nchunks * ((nlanes + 255) / 256) < NL_W_FEW ? 3 : 4;
  return 2 * f + (m->nl_maxproj > 4 ? 1 : 0);
}

template <bool CPLX, typename TS, typename TC, bool VEC, int PMAX>
void launch_nl_w_tl(const NlGroup<TS, TC> &g, const NlExtent &e, hipStream_t s) {
  constexpr int NB = PMAX <= 4 || sizeof(TC) == 4 ? 16 : 8;   // waves of a block whose accumulators fit its registers
  switch (e.form >> 1) {
    case 0: return launch_nl_w_as<CPLX, TS, TC, VEC, PMAX, 8, NB>(g, e, s);
    case 1: return launch_nl_w_as<CPLX, TS, TC, VEC, PMAX, 16, NB>(g, e, s);
    case 2: return launch_nl_w_as<CPLX, TS, TC, VEC, PMAX, 32, NB>(g, e, s);
    case 3: return launch_nl_w_as<CPLX, TS, TC, VEC, PMAX, 64, NB>(g, e, s);
    default: return launch_nl_w_as<CPLX, TS, TC, VEC, PMAX, 64, 4>(g, e, s);
  }
}

template <bool CPLX, typename TS, typename TC, bool VEC>
void launch_nl_w(const NlGroup<TS, TC> &g, const NlExtent &e, hipStream_t s) {
  if (!(e.form & 1)) launch_nl_w_tl<CPLX, TS, TC, VEC, 4>(g, e, s);
  else launch_nl_w_tl<CPLX, TS, TC, VEC, NL_MAXP>(g, e, s);
  hipLaunchKernelGGL((k_nl_wsum<TS, TC>), dim3((unsigned)((e.nw + 255) / 256), 1, e.n), dim3(256), 0, s, g);
}

// A brick's up to 32 row tiles are four for each wave of a block; while the
// blocks do not fill the device (two per CU) they are dealt to two or four
// blocks.  27,000 complex DoFs x 66 lanes 37 -> 23 us, 31,500 real x 32 lanes
// 23 -> 12 us; 74,088 complex DoFs x 48 lanes 43 -> 36 us.
template <bool CPLX> void launch_nl_ybm(const NlGroup<double, double> &g, const NlExtent &e, hipStream_t s) {
  if (e.bricks == 0) return;
  const int64_t whole = e.bricks * 8 * ((e.nlanes + NL_MN - 1) / NL_MN);
  const int parts = whole * e.n >= 512 ? 1 : whole * e.n >= 256 ? 2 : 4;
  const size_t shm = (size_t)e.kmax * NL_MN * sizeof(double);
  hipLaunchKernelGGL((k_nl_ybm<CPLX>), dim3((unsigned)(whole * parts), 1, e.n), dim3(NL_MT), shm, s, g, parts);
}

template <bool CPLX, typename TS, typename TC, bool VEC>
void launch_nl_y(Mesh *m, TS *Y, int64_t ldy, int nlanes, const TC *val, const TC *W, int64_t ldw, TC alpha,
                 hipStream_t s) {
  if (std::is_same<TC, float>::value && m->nl_nbrick > 0) {
    const TC *bval = (const TC *)m->nl_b_val32;
    constexpr int BT = 64 * (16 / (int)sizeof(TC));
    const int64_t btiles = (nlanes + BT - 1) / BT;
    const size_t shm = (size_t)m->nl_bmaxp * BT * sizeof(TC);
    const int64_t blocks = ((int64_t)m->nl_nbrick + 7) / 8 * 8 * btiles;
    hipLaunchKernelGGL((k_nl_yb<CPLX, TS, TC, VEC>), dim3((unsigned)blocks), dim3(NL_BTHREADS), shm, s, Y,
                       ldy, nlanes, m->nl_nbrick, m->nl_b_row0, m->nl_b_p0, m->nl_b_proj, m->nl_b_rows, m->nl_b_rowptr,
                       (const int4 *)m->nl_b_lcol, bval, W, ldw, alpha);
  }
  if (m->nl_nrows > 0) {
    const int tiles = (nlanes + NL_TILE - 1) / NL_TILE;
    int64_t blocks = (m->nl_nrows + 3) / 4;
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL((k_nl_y<CPLX, TS, TC, VEC>), dim3((unsigned)blocks, tiles), dim3(NL_THREADS), 0, s, Y, ldy,
                       nlanes, m->nl_rows, m->nl_rowptr, m->nl_colidx, val, m->nl_nrows, W, ldw, alpha);
  }
}

// One system's call.  ws: the partials + W workspace (nl_workspace_bytes), or
// null for the mesh's own
struct NlCall {
  Mesh *m;
  const void *X;
  int64_t ldx;
  void *Y;
  int64_t ldy;
  int nlanes;
  const double *dinv;
  double alpha;
  void *ws;
};

// vector accesses of the reduction need every thread's lanes in range and
// aligned: pairs in FP64, all four else
template <typename TS> bool nl_w_vec(const void *X, int64_t ldx, int nlanes, int w) {
  return nlanes % w == 0 && ldx % w == 0 && (uintptr_t)X % (w * sizeof(TS)) == 0;
}

// part 1: W = diag(h) F^H (D^-1) X;  part 2: Y += alpha F W;  3: both.
// Up to NL_GROUP systems of one kind, precision and reduction form.
template <bool CPLX, typename TS, typename TC>
fe_status run_nl(const NlCall *calls, int n, int parts, hipStream_t s) {
  constexpr bool f64 = std::is_same<TC, double>::value;
  NlGroup<TS, TC> g{};
  NlExtent e;
  e.n = n;
  e.form = nl_w_form(calls[0].m, calls[0].nlanes);
  bool vec = true;
  for (int i = 0; i < n; ++i) {
    const NlCall &c = calls[i];
    Mesh *m = c.m;
    NlSys<TS, TC> &a = g.a[i];
    void *ws = c.ws;
    if (!ws) {
      fe_status st = ensure_nl_workspace(m, c.nlanes);
      if (st) return st;
      ws = m->nl_W;
    }
    // workspace: partials [nchunks][NL_MAXP][ldp] then W [ns][ldp], rows padded to 4 lanes
    a.ldp = (c.nlanes + 3) / 4 * 4;
    a.part = (TC *)ws;
    a.W = a.part + (int64_t)m->nl_nchunks * NL_MAXP * a.ldp;
    a.X = (const TS *)c.X; a.Y = (TS *)c.Y; a.ldx = c.ldx; a.ldy = c.ldy; a.nlanes = c.nlanes;
    a.dinv = c.dinv; a.h = m->nl_h; a.alpha = (TC)c.alpha;
    a.F = f64 ? (const TC *)m->nl_F64 : (const TC *)m->nl_F32;
    a.chunks = (const int4 *)m->nl_chunks; a.nchunks = m->nl_nchunks; a.nodes = m->nl_atom_nodes;
    a.fstride = m->nl_maxproj; a.ns = m->ns;
    a.atom_chunk0 = m->nl_atom_chunk0; a.proj_off = m->nl_atom_proj; a.proj_atom = m->nl_proj_atom;
    a.b_row0 = m->nl_b_row0; a.b_p0 = m->nl_b_p0; a.b_proj = m->nl_b_proj; a.b_rows = m->nl_b_rows;
    a.a_off = m->nl_b_aoff; a.kb = m->nl_b_k; a.A = m->nl_b_A64; a.nbrick = m->nl_nbrick;
    e.nlanes = std::max(e.nlanes, c.nlanes);
    e.nchunks = std::max(e.nchunks, m->nl_nchunks);
    e.kmax = std::max(e.kmax, m->nl_b_kmax);
    e.bricks = std::max<int64_t>(e.bricks, (m->nl_nbrick + 7) / 8);
    e.nw = std::max(e.nw, (int64_t)m->ns * c.nlanes);
    vec = vec && nl_w_vec<TS>(c.X, c.ldx, c.nlanes, f64 ? 2 : 4);
  }
  if (parts & 1) {
    if (vec) launch_nl_w<CPLX, TS, TC, true>(g, e, s);
    else launch_nl_w<CPLX, TS, TC, false>(g, e, s);
  }
  if (parts & 2) {
    if constexpr (f64) launch_nl_ybm<CPLX>(g, e, s);
    for (int i = 0; i < n; ++i) {
      const NlCall &c = calls[i];
      const TC *val = f64 ? (const TC *)c.m->nl_val64 : (const TC *)c.m->nl_val32;
      const bool v4 = c.nlanes % 4 == 0 && c.ldy % 4 == 0 && (uintptr_t)c.Y % (4 * sizeof(TS)) == 0;
      if (v4) launch_nl_y<CPLX, TS, TC, true>(c.m, (TS *)c.Y, c.ldy, c.nlanes, val, g.a[i].W, g.a[i].ldp, (TC)c.alpha, s);
      else launch_nl_y<CPLX, TS, TC, false>(c.m, (TS *)c.Y, c.ldy, c.nlanes, val, g.a[i].W, g.a[i].ldp, (TC)c.alpha, s);
    }
  }
  FE_HIP_TRY(hipGetLastError());
  return FE_OK;
}

fe_status dispatch_nl(Mesh *m, const void *X, int64_t ldx, void *Y, int64_t ldy, int nlanes, int prec,
                      const double *dinv, double alpha, int parts, hipStream_t s, void *ws = nullptr) {
  if (m->ns == 0) return FE_OK;
  if (m->nl_maxproj > NL_MAXP) return set_error(FE_EUNSUPPORTED, "more than 10 projectors on one atom");
  const NlCall c{m, X, ldx, Y, ldy, nlanes, dinv, alpha, ws};
  if (m->cplx) {
    if (prec == FE_F64) return run_nl<true, double, double>(&c, 1, parts, s);
    if (prec == FE_F32) return run_nl<true, float, float>(&c, 1, parts, s);
    return run_nl<true, bf16n, float>(&c, 1, parts, s);
  }
  if (prec == FE_F64) return run_nl<false, double, double>(&c, 1, parts, s);
  if (prec == FE_F32) return run_nl<false, float, float>(&c, 1, parts, s);
  return run_nl<false, bf16n, float>(&c, 1, parts, s);
}
}  // namespace

// bytes of the projector workspace for nlanes real lanes: the per-chunk
// partials [nchunks][NL_MAXP][ldp] and W [ns][ldp] (sized for FP64)
int64_t nl_workspace_bytes(const Mesh *m, int nlanes) {
  if (m->ns == 0) return 0;
  const int64_t ldp = (nlanes + 3) / 4 * 4;
  return ((int64_t)m->nl_nchunks * NL_MAXP * ldp + (int64_t)m->ns * ldp) * (int64_t)sizeof(double);
}

fe_status ensure_nl_workspace(Mesh *m, int nlanes) {
  if (m->ns == 0) return FE_OK;
  const int64_t need = nl_workspace_bytes(m, nlanes);
  if (m->nl_W != nullptr && m->nl_W_lanes >= need) return FE_OK;
  if (m->nl_W != nullptr && m->graphs > 0)
    return set_error(FE_ESTATE, "a captured filter graph holds this mesh's projector workspace; destroy it before a "
                                "call with more vectors");
  if (m->nl_W) { hipFree(m->nl_W); m->footprint -= m->nl_W_lanes; m->nl_W = nullptr; m->nl_W_lanes = 0; }
  if (hipMalloc(&m->nl_W, need) != hipSuccess) { m->nl_W = nullptr; return set_error(FE_ENOMEM, "nonlocal workspace allocation failed"); }
  m->nl_W_lanes = need;
  m->footprint += need;
  return FE_OK;
}

fe_status launch_nonlocal(Mesh *m, const void *X, int64_t ldx, void *Y, int64_t ldy, int nlanes, int prec,
                          const double *dinv, double alpha, hipStream_t s) {
  return dispatch_nl(m, X, ldx, Y, ldy, nlanes, prec, dinv, alpha, 3, s);
}

fe_status launch_nonlocal_w(Mesh *m, const void *X, int64_t ldx, int nlanes, int prec, const double *dinv,
                            hipStream_t s) {
  return dispatch_nl(m, X, ldx, nullptr, 0, nlanes, prec, dinv, 0.0, 1, s);
}

fe_status launch_nonlocal_y(Mesh *m, void *Y, int64_t ldy, int nlanes, int prec, double alpha, hipStream_t s) {
  return dispatch_nl(m, nullptr, 0, Y, ldy, nlanes, prec, nullptr, alpha, 2, s);
}

fe_status ensure_side_stream(Mesh *m) {
  if (m->side) return FE_OK;
  if (hipStreamCreateWithFlags(&m->side, hipStreamNonBlocking) != hipSuccess) {
    m->side = nullptr;
    return set_error(FE_EDEVICE, "hipStreamCreate failed");
  }
  if (hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming) != hipSuccess ||
      hipEventCreateWithFlags(&m->ev_join, hipEventDisableTiming) != hipSuccess)
    return set_error(FE_EDEVICE, "hipEventCreate failed");
  return FE_OK;
}

// An application runs the projector reduction W before the local-operator
// launches and the projector update Y += alpha F W after them.  FP64: all on
// the caller's stream.  FP32 / BF16: the reduction is forked to the mesh's
// second stream, beside the local launches (both only read X), and joined
// back before the update.  The choice is measured on the plane kernels, forked
// / in order: a filter pass in FP32 on 14^3 cells of 7 points x 192 vectors
// 12.84 / 13.01 ms, one BF16 application on 12^3 x 200 538 / 573 us, one FP32
// application on 16^3 x 256 1697 / 1682.  FP64 fills the CUs' registers and
// loses more to a co-running reduction than that takes on its own.
static bool nl_forked(int prec) { return prec != FE_F64; }

fe_status nonlocal_reduce(Mesh *m, const void *X, int64_t ldx, int nlanes, int prec, const double *dinv,
                          hipStream_t s) {
  if (m->ns == 0) return FE_OK;
  fe_status st;
  if ((st = ensure_nl_workspace(m, nlanes))) return st;
  if (!nl_forked(prec)) return launch_nonlocal_w(m, X, ldx, nlanes, prec, dinv, s);
  if ((st = ensure_side_stream(m))) return st;
  FE_HIP_TRY(hipEventRecord(m->ev_fork, s));
  FE_HIP_TRY(hipStreamWaitEvent(m->side, m->ev_fork, 0));
  if ((st = launch_nonlocal_w(m, X, ldx, nlanes, prec, dinv, m->side))) return st;
  FE_HIP_TRY(hipEventRecord(m->ev_join, m->side));
  return FE_OK;
}

fe_status nonlocal_update(Mesh *m, void *Y, int64_t ldy, int nlanes, int prec, double alpha, hipStream_t s) {
  if (m->ns == 0) return FE_OK;
  if (nl_forked(prec)) FE_HIP_TRY(hipStreamWaitEvent(s, m->ev_join, 0));
  return launch_nonlocal_y(m, Y, ldy, nlanes, prec, alpha, s);
}

// The reductions (part 1) or updates (part 2) of several distinct systems:
// FP64 NL_GROUP at a time in one launch each, where the streams are the
// caller's; the others each by itself (their reductions are forked)
fe_status nonlocal_batch(Mesh *const *ms, const LocalLaunch *Ls, int n, int part, hipStream_t s) {
  std::map<int, std::vector<NlCall>> calls;               // by kind, access width and form
  for (int i = 0; i < n; ++i) {
    const LocalLaunch &L = Ls[i];
    fe_status st = FE_OK;
    if (L.prec != FE_F64) {
      st = part == 1 ? nonlocal_reduce(ms[i], L.X, L.ldx, L.nlanes, L.prec, nullptr, s)
                     : nonlocal_update(ms[i], L.Y, L.ldy, L.nlanes, L.prec, 1.0, s);
      if (st) return st;
      continue;
    }
    if (ms[i]->ns == 0) continue;
    if (ms[i]->nl_maxproj > NL_MAXP) return set_error(FE_EUNSUPPORTED, "more than 10 projectors on one atom");
    const int vec = nl_w_vec<double>(L.X, L.ldx, L.nlanes, 2) ? 2 : 0;
    calls[4 * nl_w_form(ms[i], L.nlanes) + vec + (ms[i]->cplx ? 1 : 0)].push_back({ms[i], L.X, L.ldx, L.Y, L.ldy, L.nlanes, nullptr, 1.0, nullptr});
  }
  for (const auto &kind : calls) {
    const std::vector<NlCall> &c = kind.second;
    for (size_t i = 0; i < c.size(); i += NL_GROUP) {
      const int k = (int)std::min<size_t>(NL_GROUP, c.size() - i);
      const fe_status st = kind.first & 1 ? run_nl<true, double, double>(&c[i], k, part, s)
                                          : run_nl<false, double, double>(&c[i], k, part, s);
      if (st) return st;
    }
  }
  return FE_OK;
}

fe_status apply_with_nonlocal(Mesh *m, const LocalLaunch &L, int prec, const double *dinv, double alpha,
                              hipStream_t s) {
  fe_status st;
  if ((st = nonlocal_reduce(m, L.X, L.ldx, L.nlanes, prec, dinv, s))) return st;
  if ((st = launch_local(m, L, s))) return st;
  return nonlocal_update(m, L.Y, L.ldy, L.nlanes, prec, alpha, s);
}

// ---- the application that allocates nothing ----------------------------------
// Scratch for fe_apply_H_noalloc: the projector partials and W of one
// application, then the local operator's segment planes, in a file-scope device
// array (each device holds its own copy for the life of the process).  Host code never passes the array's name to a
// kernel: its device address comes from hipGetSymbolAddress, once per device
// with that device current, and only that address is used.
static __device__ __align__(256) unsigned char scratch[FE_NOALLOC_SCRATCH_BYTES + NOALLOC_SIDE_BYTES];

namespace {
constexpr int SCRATCH_MAXDEV = 64;
std::mutex g_scratch_mu;
void *g_scratch[SCRATCH_MAXDEV] = {};

fe_status scratch_address(int dev, void **out) {
  if (dev < 0 || dev >= SCRATCH_MAXDEV) return set_error(FE_EUNSUPPORTED, "device ordinal beyond the scratch table");
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch[dev]) {
    void *p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return set_error(FE_EDEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e));
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return FE_OK;
}
}  // namespace

}  // namespace fehx

using namespace fehx;

extern "C" fe_status fe_apply_H_noalloc(fe_mesh_t m, const void *X, int64_t ldx, void *Y, int64_t ldy, int64_t nvec,
                                        int32_t prec, void *stream) {
  if (!m) return set_error(FE_EINVAL, "NULL mesh handle");
  if (nvec < 0) return set_error(FE_EINVAL, "nvec must be >= 0");
  if (nvec == 0) return FE_OK;
  if (!X || !Y) return set_error(FE_EINVAL, "NULL vector block");
  if (ldx < nvec || ldy < nvec) return set_error(FE_EINVAL, "leading dimension smaller than nvec");
  if (prec != FE_F64 && prec != FE_F32 && prec != FE_BF16) return set_error(FE_EINVAL, "unknown precision");
  if (blocks_overlap(X, ldx, Y, ldy, m->m, nvec, block_elem_bytes(prec, m->cplx)))
    return set_error(FE_EINVAL, "X and Y must not overlap");
  const int C = m->cplx ? 2 : 1;
  if (nvec * C > (1 << 30)) return set_error(FE_EINVAL, "nvec too large");
  if (m->host_only) return set_error(FE_ESTATE, "host-only mesh (device < 0) cannot apply H");
  const int nlanes = (int)(nvec * C);
  if (nl_workspace_bytes(m, nlanes) > FE_NOALLOC_SCRATCH_BYTES)
    return set_error(FE_EINVAL, "projector workspace of " + std::to_string(nl_workspace_bytes(m, nlanes)) +
                                    " bytes exceeds the static scratch of " + std::to_string((long long)FE_NOALLOC_SCRATCH_BYTES) +
                                    " bytes; use fe_apply_H");
  if (hipSetDevice(m->device) != hipSuccess) return set_error(FE_EDEVICE, "hipSetDevice failed");
  void *ws = nullptr;
  fe_status st;
  if ((st = scratch_address(m->device, &ws))) return st;
  hipStream_t s = (hipStream_t)stream;
  LocalLaunch L;
  L.X = X; L.Y = Y; L.ldx = ldx * C; L.ldy = ldy * C; L.nlanes = nlanes; L.prec = prec;
  L.vt = m->vt_pref[prec][0];
  L.side = (unsigned char *)ws + FE_NOALLOC_SCRATCH_BYTES;
  L.side_bytes = NOALLOC_SIDE_BYTES;
  // projector reduction, local operator, projector update on the caller's
  // stream, as in fe_apply_H
  if ((st = dispatch_nl(m, X, L.ldx, nullptr, 0, nlanes, prec, nullptr, 0.0, 1, s, ws))) return st;
  if ((st = launch_local(m, L, s))) return st;
  return dispatch_nl(m, nullptr, 0, Y, L.ldy, nlanes, prec, nullptr, 1.0, 2, s, ws);
}
