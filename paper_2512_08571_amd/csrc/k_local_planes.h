// Matrix-free local operator on gfx950 for affine cells with a diagonal metric
// (Sec. 3.2, eqns ggaReal / ggaCmplx, Alg. 2): one wave per column of cells.
//
// A wave owns one column of cells along a_2 and a tile of VT real vector lanes
// and walks the column cell by cell.  Each thread holds a whole plane of the
// cell for its lanes (LPT adjacent lanes, 16-byte or narrower elements), so a
// 1D contraction along either in-plane axis runs in registers; only the change
// of plane goes through LDS, within the wave: LDS operations of one wave
// execute in order, so no barrier is needed anywhere.  Thread (plane index,
// lane) of the wave:
//   A   (x, y) plane at node z = k: gather, N along x, N along y
//   B   (x, z) plane at point y = j: N along z, the z-direction stage and the
//       potential; u goes back to (x, y) planes, the partial sum is parked
//   C   (x, y) plane at point z = k: the x- and y-direction stages completed,
//       N^T along y and x
//   D   (x, z) plane at node y = j: N^T along z, carry, scatter
// The block is exchanged in slots of one x each ([y][z][lane]): slot x serves
// the A -> B exchange, then u's return, then parks the partial sum, then the
// C -> D exchange.
//
// The weights of eqn refact are folded into the 1D tables, half on each side:
// with N' = W^1/2 N (W the 1D weights and the Jacobian's cube root), u = N' x 3 X,
// T_d = D_d u, D_d = sqrt(g_d) W^1/2 Dtilde W^-1/2 and c_d = Vtilde^G_d / sqrt(g_d),
//   r = V u + sum_d [c_d T_d + D_d^T (T_d + c_d u) - i kappa_d / sqrt(g_d) T_d],
//   Y^(e) = N'^T x 3 r,
// which is eqn refact: the weights commute with the factors at the points.
// The symmetric form needs two tables at a time, N' and one D_d, each applied
// both ways.  In filter steps D^-1 (a product of 1D factors on affine cells)
// is folded into the gather's N tables the same way.
//
// The consistent mass of affine cells is separable, M^(e) = M x 3 with
// M = N'^T N': MASS applies it along x and y in the gathered plane and along z
// after the one exchange, with no coefficients.
//
// Scatter: as in k_local_impl.h (columns coloured, one launch per colour
// phase, nodes of several columns stored by the lowest phase and
// read-modify-written by later ones; fixed summation order, no atomics; the
// planes at the cuts of a segmented column in the same order, by k_planes_join).
//
// What bounds it: with every wave slot filled, FP64 issue and the load/store
// path in about equal parts (real, 7 points, 16^3 cells x 256 vectors, one of
// four phases: 271 us of arithmetic and exchange alone, 545 us complete); with
// few columns, the length of a wave's walk.  Against one thread block per
// column with the cell in LDS and a barrier at each change of direction (one
// phase there / here): real 16^3 x 256 vectors at 6 points 583 / 386 us, at 7
// points 648 / 545, complex 8 points 1288 / 890, real 9 points 12^3 952 / 870;
// with columns cut into segments, 27,000 complex DoFs x 33 vectors 43 / 17,
// 4,096 DoFs x 8 vectors 19 / 10.
#pragma once
#include <algorithm>
#include <vector>

#include "k_local_impl.h"

namespace fehx {

// the value type of a thread's adjacent lanes
template <typename TC, int LPT> struct LaneVec;
template <> struct LaneVec<double, 1> { typedef double T; };
template <> struct LaneVec<float, 1> { typedef float T; };
template <> struct LaneVec<float, 2> { typedef float T __attribute__((ext_vector_type(2))); };

__device__ __forceinline__ double vfma(double a, double x, double y) { return fma(a, x, y); }
__device__ __forceinline__ float vfma(float a, float x, float y) { return fmaf(a, x, y); }
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f32x2 vfma(float a, f32x2 x, f32x2 y) { return (f32x2){fmaf(a, x.x, y.x), fmaf(a, x.y, y.y)}; }

// ---- 1D tables and their even-odd application --------------------------------
// y (+)= A x for a packed centro-(anti)symmetric A on lane vectors.
// FP32: table rows are wave-uniform scalar loads, as in k_local_impl.h.
// FP64: the table sits in vector registers, sixteen entries per register pair
// (the same in every row of sixteen lanes), and v_fmac_f64 reads an entry by a
// DPP row broadcast; only the first column, which a multiply takes, is scalar.
// Scalar FP64 tables need 50 SGPRs each at seven points, so that the compiler
// kept them by lane writes and reads: 2263 of them beside the 3612 FP64
// instructions of a cell.  All 64 lanes of the wave must be active here: a
// broadcast reads lane e of each row of sixteen.
template <int NIN, int NOUT> struct DppTable {
  static constexpr int CI = (NIN + 1) / 2, HI = NIN / 2, CO = (NOUT + 1) / 2;
  static constexpr int R = CI + HI - 2;                  // entries per row without the first column
  static constexpr int PT = (CO * R + 15) / 16;          // register pairs
};

// Rows of the product as one block each, all chains of a block in turn (FP64
// results may be used every other issue by the same wave):
//   DppChain  a = s x_0 + sum_i tab[E0 + i] x_{i+1}
//   DppRow    e likewise over x from E0, o over y from E0 + NE
//   DppRow2   two rows (e, o), (f, g), the second's entries after the first's
// The opening multiplies (s_nop where there is one) keep the two wait states a
// DPP read needs after a vector write of its source register.
#define FEHX_FM(ACC, T, X, E0, I) "v_fmac_f64_dpp " ACC ", " T ", " X " row_newbcast:(" E0 "+" I ")&15 row_mask:0xf bank_mask:0xf\n\t"
#define FEHX_T(K) "v"(t[(E0 + K) / 16])
template <int NC, int E0> struct DppChain;
template <int NE, int NO, int E0> struct DppRow;
template <int NE, int NO, int E0> struct DppRow2;
template <int E0> struct DppChain<1, E0> {
  static __device__ __forceinline__ void run(double &a, double s, const double *t, const double *x) {
    asm("v_mul_f64 %0, %1, %2\n\t" "s_nop 0\n\t" FEHX_FM("%0", "%4", "%3", "%5", "0")
        : "=&v"(a)
        : "s"(s), "v"(x[0]), "v"(x[1]), FEHX_T(0), "n"(E0));
  }
};
template <int E0> struct DppChain<2, E0> {
  static __device__ __forceinline__ void run(double &a, double s, const double *t, const double *x) {
    asm("v_mul_f64 %0, %1, %2\n\t" "s_nop 0\n\t" FEHX_FM("%0", "%5", "%3", "%7", "0")
        FEHX_FM("%0", "%6", "%4", "%7", "1")
        : "=&v"(a)
        : "s"(s), "v"(x[0]), "v"(x[1]), "v"(x[2]), FEHX_T(0), FEHX_T(1), "n"(E0));
  }
};
template <int E0> struct DppChain<3, E0> {
  static __device__ __forceinline__ void run(double &a, double s, const double *t, const double *x) {
    asm("v_mul_f64 %0, %1, %2\n\t" "s_nop 0\n\t" FEHX_FM("%0", "%6", "%3", "%9", "0")
        FEHX_FM("%0", "%7", "%4", "%9", "1") FEHX_FM("%0", "%8", "%5", "%9", "2")
        : "=&v"(a)
        : "s"(s), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), FEHX_T(0), FEHX_T(1), FEHX_T(2), "n"(E0));
  }
};
template <int E0> struct DppChain<4, E0> {
  static __device__ __forceinline__ void run(double &a, double s, const double *t, const double *x) {
    asm("v_mul_f64 %0, %1, %2\n\t" "s_nop 0\n\t" FEHX_FM("%0", "%7", "%3", "%11", "0")
        FEHX_FM("%0", "%8", "%4", "%11", "1") FEHX_FM("%0", "%9", "%5", "%11", "2")
        FEHX_FM("%0", "%10", "%6", "%11", "3")
        : "=&v"(a)
        : "s"(s), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), FEHX_T(0), FEHX_T(1), FEHX_T(2),
          FEHX_T(3), "n"(E0));
  }
};
template <int E0> struct DppChain<5, E0> {
  static __device__ __forceinline__ void run(double &a, double s, const double *t, const double *x) {
    asm("v_mul_f64 %0, %1, %2\n\t" "s_nop 0\n\t" FEHX_FM("%0", "%8", "%3", "%13", "0")
        FEHX_FM("%0", "%9", "%4", "%13", "1") FEHX_FM("%0", "%10", "%5", "%13", "2")
        FEHX_FM("%0", "%11", "%6", "%13", "3") FEHX_FM("%0", "%12", "%7", "%13", "4")
        : "=&v"(a)
        : "s"(s), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), FEHX_T(0), FEHX_T(1),
          FEHX_T(2), FEHX_T(3), FEHX_T(4), "n"(E0));
  }
};
template <int E0> struct DppRow<1, 0, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %6\n\t" FEHX_FM("%0", "%7", "%5", "%8", "0")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(y[0]), FEHX_T(0), "n"(E0));
  }
};
template <int E0> struct DppRow<1, 1, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %6\n\t" FEHX_FM("%0", "%8", "%5", "%10", "0")
        FEHX_FM("%1", "%9", "%7", "%10", "1")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(y[0]), "v"(y[1]), FEHX_T(0), FEHX_T(1), "n"(E0));
  }
};
template <int E0> struct DppRow<2, 1, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %7\n\t" FEHX_FM("%0", "%9", "%5", "%12", "0")
        FEHX_FM("%1", "%11", "%8", "%12", "2") FEHX_FM("%0", "%10", "%6", "%12", "1")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), FEHX_T(0), FEHX_T(1),
          FEHX_T(2), "n"(E0));
  }
};
template <int E0> struct DppRow<2, 2, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %7\n\t" FEHX_FM("%0", "%10", "%5", "%14", "0")
        FEHX_FM("%1", "%12", "%8", "%14", "2") FEHX_FM("%0", "%11", "%6", "%14", "1")
        FEHX_FM("%1", "%13", "%9", "%14", "3")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), "v"(y[2]), FEHX_T(0),
          FEHX_T(1), FEHX_T(2), FEHX_T(3), "n"(E0));
  }
};
template <int E0> struct DppRow<3, 2, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %8\n\t" FEHX_FM("%0", "%11", "%5", "%16", "0")
        FEHX_FM("%1", "%14", "%9", "%16", "3") FEHX_FM("%0", "%12", "%6", "%16", "1")
        FEHX_FM("%1", "%15", "%10", "%16", "4") FEHX_FM("%0", "%13", "%7", "%16", "2")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]), "v"(y[1]), "v"(y[2]),
          FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), "n"(E0));
  }
};
template <int E0> struct DppRow<3, 3, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %8\n\t" FEHX_FM("%0", "%12", "%5", "%18", "0")
        FEHX_FM("%1", "%15", "%9", "%18", "3") FEHX_FM("%0", "%13", "%6", "%18", "1")
        FEHX_FM("%1", "%16", "%10", "%18", "4") FEHX_FM("%0", "%14", "%7", "%18", "2")
        FEHX_FM("%1", "%17", "%11", "%18", "5")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]), "v"(y[1]), "v"(y[2]),
          "v"(y[3]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), "n"(E0));
  }
};
template <int E0> struct DppRow<4, 3, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %9\n\t" FEHX_FM("%0", "%13", "%5", "%20", "0")
        FEHX_FM("%1", "%17", "%10", "%20", "4") FEHX_FM("%0", "%14", "%6", "%20", "1")
        FEHX_FM("%1", "%18", "%11", "%20", "5") FEHX_FM("%0", "%15", "%7", "%20", "2")
        FEHX_FM("%1", "%19", "%12", "%20", "6") FEHX_FM("%0", "%16", "%8", "%20", "3")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(y[0]), "v"(y[1]),
          "v"(y[2]), "v"(y[3]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), FEHX_T(6),
          "n"(E0));
  }
};
template <int E0> struct DppRow<4, 4, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %9\n\t" FEHX_FM("%0", "%14", "%5", "%22", "0")
        FEHX_FM("%1", "%18", "%10", "%22", "4") FEHX_FM("%0", "%15", "%6", "%22", "1")
        FEHX_FM("%1", "%19", "%11", "%22", "5") FEHX_FM("%0", "%16", "%7", "%22", "2")
        FEHX_FM("%1", "%20", "%12", "%22", "6") FEHX_FM("%0", "%17", "%8", "%22", "3")
        FEHX_FM("%1", "%21", "%13", "%22", "7")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(y[0]), "v"(y[1]),
          "v"(y[2]), "v"(y[3]), "v"(y[4]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5),
          FEHX_T(6), FEHX_T(7), "n"(E0));
  }
};
template <int E0> struct DppRow<5, 4, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %10\n\t" FEHX_FM("%0", "%15", "%5", "%24", "0")
        FEHX_FM("%1", "%20", "%11", "%24", "5") FEHX_FM("%0", "%16", "%6", "%24", "1")
        FEHX_FM("%1", "%21", "%12", "%24", "6") FEHX_FM("%0", "%17", "%7", "%24", "2")
        FEHX_FM("%1", "%22", "%13", "%24", "7") FEHX_FM("%0", "%18", "%8", "%24", "3")
        FEHX_FM("%1", "%23", "%14", "%24", "8") FEHX_FM("%0", "%19", "%9", "%24", "4")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(y[0]),
          "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4),
          FEHX_T(5), FEHX_T(6), FEHX_T(7), FEHX_T(8), "n"(E0));
  }
};
template <int E0> struct DppRow<5, 5, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double se, double so, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %2, %4\n\t" "v_mul_f64 %1, %3, %10\n\t" FEHX_FM("%0", "%16", "%5", "%26", "0")
        FEHX_FM("%1", "%21", "%11", "%26", "5") FEHX_FM("%0", "%17", "%6", "%26", "1")
        FEHX_FM("%1", "%22", "%12", "%26", "6") FEHX_FM("%0", "%18", "%7", "%26", "2")
        FEHX_FM("%1", "%23", "%13", "%26", "7") FEHX_FM("%0", "%19", "%8", "%26", "3")
        FEHX_FM("%1", "%24", "%14", "%26", "8") FEHX_FM("%0", "%20", "%9", "%26", "4")
        FEHX_FM("%1", "%25", "%15", "%26", "9")
        : "=&v"(e), "=&v"(o)
        : "s"(se), "s"(so), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(x[4]), "v"(x[5]), "v"(y[0]),
          "v"(y[1]), "v"(y[2]), "v"(y[3]), "v"(y[4]), "v"(y[5]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3),
          FEHX_T(4), FEHX_T(5), FEHX_T(6), FEHX_T(7), FEHX_T(8), FEHX_T(9), "n"(E0));
  }
};
template <int E0> struct DppRow2<1, 0, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %10\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %10\n\t" FEHX_FM("%0", "%11", "%9", "%13", "0")
        FEHX_FM("%2", "%12", "%9", "%13", "1")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(y[0]), FEHX_T(0), FEHX_T(1), "n"(E0));
  }
};
template <int E0> struct DppRow2<1, 1, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %10\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %10\n\t" FEHX_FM("%0", "%12", "%9", "%16", "0")
        FEHX_FM("%2", "%14", "%9", "%16", "2") FEHX_FM("%1", "%13", "%11", "%16", "1")
        FEHX_FM("%3", "%15", "%11", "%16", "3")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(y[0]), "v"(y[1]), FEHX_T(0), FEHX_T(1),
          FEHX_T(2), FEHX_T(3), "n"(E0));
  }
};
template <int E0> struct DppRow2<2, 1, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %11\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %11\n\t" FEHX_FM("%0", "%13", "%9", "%19", "0")
        FEHX_FM("%2", "%16", "%9", "%19", "3") FEHX_FM("%1", "%15", "%12", "%19", "2")
        FEHX_FM("%3", "%18", "%12", "%19", "5") FEHX_FM("%0", "%14", "%10", "%19", "1")
        FEHX_FM("%2", "%17", "%10", "%19", "4")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), FEHX_T(0),
          FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), "n"(E0));
  }
};
template <int E0> struct DppRow2<2, 2, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %11\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %11\n\t" FEHX_FM("%0", "%14", "%9", "%22", "0")
        FEHX_FM("%2", "%18", "%9", "%22", "4") FEHX_FM("%1", "%16", "%12", "%22", "2")
        FEHX_FM("%3", "%20", "%12", "%22", "6") FEHX_FM("%0", "%15", "%10", "%22", "1")
        FEHX_FM("%2", "%19", "%10", "%22", "5") FEHX_FM("%1", "%17", "%13", "%22", "3")
        FEHX_FM("%3", "%21", "%13", "%22", "7")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(y[0]), "v"(y[1]), "v"(y[2]),
          FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), FEHX_T(6), FEHX_T(7), "n"(E0));
  }
};
template <int E0> struct DppRow2<3, 2, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %12\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %12\n\t" FEHX_FM("%0", "%15", "%9", "%25", "0")
        FEHX_FM("%2", "%20", "%9", "%25", "5") FEHX_FM("%1", "%18", "%13", "%25", "3")
        FEHX_FM("%3", "%23", "%13", "%25", "8") FEHX_FM("%0", "%16", "%10", "%25", "1")
        FEHX_FM("%2", "%21", "%10", "%25", "6") FEHX_FM("%1", "%19", "%14", "%25", "4")
        FEHX_FM("%3", "%24", "%14", "%25", "9") FEHX_FM("%0", "%17", "%11", "%25", "2")
        FEHX_FM("%2", "%22", "%11", "%25", "7")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]), "v"(y[1]),
          "v"(y[2]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), FEHX_T(6), FEHX_T(7),
          FEHX_T(8), FEHX_T(9), "n"(E0));
  }
};
template <int E0> struct DppRow2<3, 3, E0> {
  static __device__ __forceinline__ void run(double &e, double &o, double &f, double &g, double se, double so, double sf, double sg, const double *t, const double *x, const double *y) {
    asm("v_mul_f64 %0, %4, %8\n\t" "v_mul_f64 %1, %5, %12\n\t" "v_mul_f64 %2, %6, %8\n\t"
        "v_mul_f64 %3, %7, %12\n\t" FEHX_FM("%0", "%16", "%9", "%28", "0")
        FEHX_FM("%2", "%22", "%9", "%28", "6") FEHX_FM("%1", "%19", "%13", "%28", "3")
        FEHX_FM("%3", "%25", "%13", "%28", "9") FEHX_FM("%0", "%17", "%10", "%28", "1")
        FEHX_FM("%2", "%23", "%10", "%28", "7") FEHX_FM("%1", "%20", "%14", "%28", "4")
        FEHX_FM("%3", "%26", "%14", "%28", "10") FEHX_FM("%0", "%18", "%11", "%28", "2")
        FEHX_FM("%2", "%24", "%11", "%28", "8") FEHX_FM("%1", "%21", "%15", "%28", "5")
        FEHX_FM("%3", "%27", "%15", "%28", "11")
        : "=&v"(e), "=&v"(o), "=&v"(f), "=&v"(g)
        : "s"(se), "s"(so), "s"(sf), "s"(sg), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3]), "v"(y[0]), "v"(y[1]),
          "v"(y[2]), "v"(y[3]), FEHX_T(0), FEHX_T(1), FEHX_T(2), FEHX_T(3), FEHX_T(4), FEHX_T(5), FEHX_T(6),
          FEHX_T(7), FEHX_T(8), FEHX_T(9), FEHX_T(10), FEHX_T(11), "n"(E0));
  }
};
#undef FEHX_FM
#undef FEHX_T

// A table as a stage holds it: FP32 keeps the pointer, opaque once per stage so
// that the stage's lines share the loaded entries; FP64 the register pairs
// (lane l of pair k: entry 16 k + l % 16 of the broadcast copy behind the
// packed one, see PlaneTab).  TR: the transpose, applied from the table itself
// in FP32 (eo_tr), from its own packed copy in FP64.
template <int NIN, int NOUT, typename TC, bool TR = false> struct Table1D {
  cptr<TC> p;
  __device__ __forceinline__ void load(const TC *q) { p = scalar_table(q); }
  __device__ __forceinline__ void load(const Table1D<NOUT, NIN, TC, false> &t, const TC *) { p = t.p; }
  __device__ __forceinline__ void load(const TC *q, const PlaneTab &L) { p = scalar_table(q + L.n); }
};
template <int NIN, int NOUT, bool TR> struct Table1D<NIN, NOUT, double, TR> {
  cptr<double> p;
  double t[DppTable<NIN, NOUT>::PT];
  __device__ __forceinline__ void load(const double *q) {
    p = scalar_table(q);
    const auto d = p + ((NOUT + 1) / 2) * NIN + (threadIdx.x & 15);
#pragma unroll
    for (int k = 0; k < DppTable<NIN, NOUT>::PT; ++k) t[k] = d[16 * k];
  }
  template <typename T> __device__ __forceinline__ void load(const T &, const double *q) { load(q); }
  __device__ __forceinline__ void load(const double *q, const PlaneTab &L) { load(q + L.nt); }
};

// e + o and their difference into rows Q and NOUT - 1 - Q of y (+)= A x
template <int NOUT, int SYM, bool ADD, int Q, typename V>
__device__ __forceinline__ void eo_put(V e, V o, V (&y)[NOUT]) {
  const V hi = SYM > 0 ? e - o : o - e;
  y[Q] = ADD ? y[Q] + (e + o) : e + o;
  y[NOUT - 1 - Q] = ADD ? y[NOUT - 1 - Q] + hi : hi;
}

// rows Q.. of y (+)= A x from xp = x_i + x_{n-1-i}, xm = x_i - x_{n-1-i}
template <int NIN, int NOUT, int SYM, bool ADD, int Q, typename TC, bool TR, typename V>
__device__ __forceinline__ void eo_rows(const Table1D<NIN, NOUT, TC, TR> &T, const V *xp, const V *xm, V (&y)[NOUT]) {
  constexpr int CI = (NIN + 1) / 2, HI = NIN / 2, CO = (NOUT + 1) / 2, HO = NOUT / 2;
  constexpr bool mid = (NOUT & 1) && Q == HO;
  if constexpr (Q < CO) {
    cptr<TC> E = T.p + Q * NIN;
    cptr<TC> O = E + CI;
    if constexpr (std::is_same<V, double>::value) {
      constexpr int R = DppTable<NIN, NOUT>::R, E0 = Q * R;
      if constexpr (mid) {
        double v;
        if constexpr (SYM > 0) DppChain<CI - 1, E0>::run(v, E[0], T.t, xp);
        else if constexpr (HI > 1) DppChain<HI - 1, E0 + CI - 1>::run(v, O[0], T.t, xm);
        else v = O[0] * xm[0];
        y[Q] = ADD ? y[Q] + v : v;
        eo_rows<NIN, NOUT, SYM, ADD, Q + 1>(T, xp, xm, y);
      } else if constexpr (Q + 1 < HO && R <= 6) {
        double e, o, f, g;
        DppRow2<CI - 1, HI - 1, E0>::run(e, o, f, g, E[0], O[0], E[NIN], O[NIN], T.t, xp, xm);
        eo_put<NOUT, SYM, ADD, Q>(e, o, y);
        eo_put<NOUT, SYM, ADD, Q + 1>(f, g, y);
        eo_rows<NIN, NOUT, SYM, ADD, Q + 2>(T, xp, xm, y);
      } else {
        double e, o;
        DppRow<CI - 1, HI - 1, E0>::run(e, o, E[0], O[0], T.t, xp, xm);
        eo_put<NOUT, SYM, ADD, Q>(e, o, y);
        eo_rows<NIN, NOUT, SYM, ADD, Q + 1>(T, xp, xm, y);
      }
    } else {
      V e = 0, o = 0;
      if constexpr (!mid || SYM > 0) {
        e = E[0] * xp[0];
#pragma unroll
        for (int i = 1; i < CI; ++i) e = vfma(E[i], xp[i], e);
      }
      if constexpr (!mid || SYM < 0) {
        o = O[0] * xm[0];
#pragma unroll
        for (int i = 1; i < HI; ++i) o = vfma(O[i], xm[i], o);
      }
      if constexpr (mid) {
        const V v = SYM > 0 ? e : o;
        y[Q] = ADD ? y[Q] + v : v;
      } else {
        eo_put<NOUT, SYM, ADD, Q>(e, o, y);
      }
      eo_rows<NIN, NOUT, SYM, ADD, Q + 1>(T, xp, xm, y);
    }
  }
}

// y (+)= A x; T transposed: y (+)= A^T x from A's packed rows (FP32).  There the
// half of x that meets E is the one A's rows sum into E's half of y: the even
// one for a symmetric A, the odd one for an antisymmetric A.
template <int SYM, bool ADD, int NIN, int NOUT, typename TC, bool TR, typename V>
__device__ __forceinline__ void eo(const Table1D<NIN, NOUT, TC, TR> &T, const V (&x)[NIN], V (&y)[NOUT]) {
  constexpr int CI = (NIN + 1) / 2, HI = NIN / 2;
  V xp[CI], xm[HI];
#pragma unroll
  for (int i = 0; i < HI; ++i) {
    xp[i] = x[i] + x[NIN - 1 - i];
    xm[i] = x[i] - x[NIN - 1 - i];
  }
  if constexpr (NIN & 1) xp[HI] = x[HI];
  if constexpr (TR && !std::is_same<TC, double>::value) {
    constexpr int CO = (NOUT + 1) / 2, HO = NOUT / 2;    // A is NIN x NOUT: columns are y's
    constexpr int KE = SYM > 0 ? CI : HI, KO = SYM > 0 ? HI : CI;
    const V *xe = SYM > 0 ? xp : xm, *xo = SYM > 0 ? xm : xp;
#pragma unroll
    for (int i = 0; i < CO; ++i) {
      V e = T.p[i] * xe[0];
#pragma unroll
      for (int q = 1; q < KE; ++q) e = vfma(T.p[q * NOUT + i], xe[q], e);
      if (i == HO) {
        y[i] = ADD ? y[i] + e : e;
      } else {
        V o = T.p[CO + i] * xo[0];
#pragma unroll
        for (int q = 1; q < KO; ++q) o = vfma(T.p[q * NOUT + CO + i], xo[q], o);
        y[i] = ADD ? y[i] + (e + o) : e + o;
        y[NOUT - 1 - i] = ADD ? y[NOUT - 1 - i] + (e - o) : e - o;
      }
    }
  } else {
    eo_rows<NIN, NOUT, SYM, ADD, 0>(T, xp, xm, y);
  }
}

// Order this wave's LDS operations (no instruction: LDS runs a wave's
// operations in order; the compiler must not reorder them).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// FP32 (plain code, where FP64 has asm blocks): keeps the scheduler from
// interleaving lines beyond the registers
template <typename TC> __device__ __forceinline__ void line_end() {
  if constexpr (!std::is_same<TC, double>::value) __builtin_amdgcn_sched_barrier(0);
}

// FP32: a value formed here, not sunk past the next branch (a whole plane's
// inputs would stay live up to there)
template <typename TC, typename V> __device__ __forceinline__ V in_line(V x) {
  if constexpr (!std::is_same<TC, double>::value) asm volatile("" : "+v"(x));
  return x;
}

// A wave-uniform value the compiler cannot see through: products with it are
// formed where they are used instead of being hoisted out of the cell loop
// into (spilled) registers.
__device__ __forceinline__ int64_t opaque(int64_t x) {
  asm volatile("" : "+s"(x));
  return x;
}

template <typename T> __device__ __forceinline__ T *opaque(T *p) { return reinterpret_cast<T *>(opaque(reinterpret_cast<int64_t>(p))); }
template <typename T> __device__ __forceinline__ const T *scalar_ptr(const T *p) { return opaque(p); }
// A thread's lanes in global memory: gather loads by address, and the scatter's
// reads and writes through a buffer descriptor, whose bounds check turns a
// masked thread (offset BUF_OFF) into a read of zero and a dropped write.  So
// the scatter has no branches, and the compiler knows how many accesses are in
// flight at each wait (behind branches it must assume none of theirs, and
// waited for the whole next gather at the first store).
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t BufRsrc;
constexpr unsigned BUF_SPAN = (unsigned)PLANE_SPAN, BUF_OFF = 0x80000000u;
__device__ __forceinline__ BufRsrc buf_at(void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, (short)0, (int)BUF_SPAN, 0x00027000);
}
// R is an element as a load leaves it, up() its value: BF16 stays packed while
// the gather is in flight.
template <typename TS, typename V> struct LaneIO;
template <typename V> struct LaneIO64 {                  // eight bytes as they are
  typedef V R;
  static __device__ __forceinline__ V up(R v) { return v; }
  static __device__ __forceinline__ V ldb(BufRsrc r, int o) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
  }
  static __device__ __forceinline__ void stb(BufRsrc r, int o, V v) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, o, 0, 0);
  }
};
template <> struct LaneIO<double, double> : LaneIO64<double> {
  static __device__ __forceinline__ double ld(const double *p) { return *p; }
};
template <> struct LaneIO<float, f32x2> : LaneIO64<f32x2> {
  static __device__ __forceinline__ f32x2 ld(const float *p) { return *(const f32x2 *)p; }
};
template <> struct LaneIO<float, float> {
  typedef float R;
  static __device__ __forceinline__ float up(R v) { return v; }
  static __device__ __forceinline__ R ld(const float *p) { return *p; }
  static __device__ __forceinline__ R ldb(BufRsrc r, int o) {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
  }
  static __device__ __forceinline__ void stb(BufRsrc r, int o, float v) {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, o, 0, 0);
  }
};
template <> struct LaneIO<bf16s, float> {
  typedef uint16_t R;
  static __device__ __forceinline__ float up(R v) { return bf16_to_f(v); }
  static __device__ __forceinline__ R ld(const bf16s *p) { return p->b; }
  static __device__ __forceinline__ R ldb(BufRsrc r, int o) { return __builtin_amdgcn_raw_buffer_load_b16(r, o, 0, 0); }
  static __device__ __forceinline__ void stb(BufRsrc r, int o, float v) {
    __builtin_amdgcn_raw_buffer_store_b16(f_to_bf16(v), r, o, 0, 0);
  }
};
template <> struct LaneIO<bf16s, f32x2> {
  typedef uint32_t R;
  static __device__ __forceinline__ f32x2 up(R w) { return (f32x2){__uint_as_float(w << 16), __uint_as_float(w & 0xffff0000u)}; }
  static __device__ __forceinline__ R ld(const bf16s *p) { return *(const uint32_t *)p; }
  static __device__ __forceinline__ R ldb(BufRsrc r, int o) { return __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0); }
  static __device__ __forceinline__ void stb(BufRsrc r, int o, f32x2 v) {
    __builtin_amdgcn_raw_buffer_store_b32((uint32_t)f_to_bf16(v.x) | ((uint32_t)f_to_bf16(v.y) << 16), r, o, 0, 0);
  }
};

// Geometry of the wave: NQ planes of TV threads (even: complex lanes come in
// adjacent pairs, and tiles start 16-byte aligned); NS slots of one x, padded in y where a
// group of eight threads would otherwise read one bank.  At seven points only
// six of the seven slots exist, the last x parking its sum in registers: eight
// waves of 18.8 KB then share a CU's LDS instead of seven of 22 KB.
template <int NQ, bool CPLX, int LPT> struct PlaneShape {
  static constexpr int TV = plane_vt(NQ, 1);
  static constexpr int VT = TV * LPT;
  static constexpr int SZ = TV;
  static constexpr int SY = NQ * TV + ((NQ * TV * 2) % 64 == 0 ? 8 : 0);
  static constexpr int SLOT = NQ * SY;
  static constexpr int NS = NQ == 7 ? 6 : NQ;
  static constexpr int elems = NS * SLOT;      // LDS elements of LPT lanes
};

template <int NP, int NQ, bool CPLX, bool GGA, typename TS, typename TC, int LPT, bool MASS>
__device__ __forceinline__ void plane_column(const KArgs<TC> &a, const int col, const int seg, const int tile) {
  typedef typename LaneVec<TC, LPT>::T V;
  typedef PlaneShape<NQ, CPLX, LPT> S;
  typedef LaneIO<TS, V> IO;
  constexpr PlaneTab L = plane_tab(NP, NQ);
  constexpr int NQ2 = NQ * NQ, NQ3 = NQ2 * NQ;
  constexpr int RB = 2;                                  // lines of values read back in flight
  extern __shared__ __align__(16) unsigned char smem_raw[];
  V *B = reinterpret_cast<V *>(smem_raw) + (threadIdx.x >> 6) * S::elems;

  // the threads past the last plane repeat the first ones with the same values
  // to the same slots and store nothing, so that every lane of the wave is
  // active throughout
  constexpr int NT = NQ * S::TV;
  static_assert(64 - NT <= NT && (!CPLX || LPT > 1 || NT % 2 == 0), "idle threads repeat whole lane pairs");
  const int t0 = threadIdx.x & 63;
  const int tid = t0 < NT ? t0 : t0 - NT;
  const int pl = tid / S::TV, v = tid - pl * S::TV;      // plane index (z or y), lane group
  const int cx = __builtin_amdgcn_readfirstlane(a.cols[2 * col]);
  const int cy = __builtin_amdgcn_readfirstlane(a.cols[2 * col + 1]);
  const int lane = tile * S::VT + v * LPT;
  const bool on = lane < a.nlanes && t0 < NT;
  const int lane_c = lane < a.nlanes ? lane : tile * S::VT;   // lanes past the block read the tile's first
  const int p = a.p;
  const int xoff = a.dmask & 1, yoff = (a.dmask >> 1) & 1, zoff = (a.dmask >> 2) & 1;
  const int ax = colour_of(cx, a.N0), by = colour_of(cy, a.N1);
  const bool fx0 = !(ax < colour_of(cx == 0 ? a.N0 - 1 : cx - 1, a.N0));
  const bool fx1 = !(ax < colour_of(cx == a.N0 - 1 ? 0 : cx + 1, a.N0));
  const bool fy0 = !(by < colour_of(cy == 0 ? a.N1 - 1 : cy - 1, a.N1));
  const bool fy1 = !(by < colour_of(cy == a.N1 - 1 ? 0 : cy + 1, a.N1));
  const bool fy = (pl == 0 && fy0) || (pl == NP - 1 && fy1);   // this thread's node row is read-modify-written
  // Node offsets along x and y: consecutive but for the ends, which wrap on a
  // periodic axis.  A Dirichlet axis numbers its interior nodes g - 1 and has
  // no DoF on its faces: an end without one is read from its neighbour's
  // address, taken as zero and not stored.
  const int gx0 = cx * p - xoff, gy0 = cy * p - yoff;
  const bool x0 = gx0 >= 0, x1 = !xoff || gx0 + p < a.M0, y0 = gy0 >= 0, y1 = !yoff || gy0 + p < a.M1;
  const int gxl = gx0 + p < a.M0 ? gx0 + p : (xoff ? gx0 + p - 1 : 0);
  const int gyl = gy0 + p < a.M1 ? gy0 + p : (yoff ? gy0 + p - 1 : 0);
  const int gxf = x0 ? gx0 : gx0 + 1, gyf = y0 ? gy0 : gy0 + 1;
  const int64_t MM = (int64_t)a.M0 * a.M1;
  // scatter: this thread's node row (y = pl) at the column's first x
  const bool ins = on && pl < NP && (pl != 0 || y0) && (pl != NP - 1 || y1);
  const int gys = pl == 0 ? gyf : pl == NP - 1 ? gyl : gy0 + (pl < NP ? pl : 1);
  const TS *const Xl = (const TS *)a.X + lane_c;
  // byte offsets of this thread's node row: written, and read back where
  // earlier colour phases stored (first x, last x, the others)
  const unsigned yo = (unsigned)(((int64_t)gys * a.M0 * a.ldy + lane_c) * (int64_t)sizeof(TS));
  const unsigned ow = ins ? yo : BUF_OFF;
  const unsigned or0 = ins && (fy || fx0) && x0 ? yo : BUF_OFF, or1 = ins && (fy || fx1) && x1 ? yo : BUF_OFF,
                 orm = ins && fy ? yo : BUF_OFF;
  const unsigned ow0 = x0 ? ow : BUF_OFF, ow1 = x1 ? ow : BUF_OFF;
  // the planes at the cuts (layout at side_seg_bytes)
  typedef LaneIO<TC, V> SideIO;
  const int side_lanes = a.ntiles * S::VT, side_x = NP * side_lanes;
  const unsigned so = t0 < NT && pl < NP ? (unsigned)(pl * side_lanes + lane) * (unsigned)sizeof(TC) : BUF_OFF;
  auto side_at = [&](int sg, int half) {
    return a.side + half * a.side_half + ((int64_t)sg * (a.N0 * a.N1) + cx + a.N0 * cy) * (NP * NP) * side_lanes;
  };
  TC ksgn = 0;                                           // sign of the Bloch term in this lane
  if constexpr (CPLX && LPT == 1) ksgn = (lane & 1) ? (TC)-1 : (TC)1;

  // -i kappa T of a thread's lanes: the real part gets +kappa T_im, the imaginary part -kappa T_re
  auto bloch = [&](TC kap, V t, V z) -> V {
    if constexpr (LPT == 1) return vfma(kap * ksgn, swap_pair(t), z);
    else { z.x = fmaf(kap, t.y, z.x); z.y = fmaf(-kap, t.x, z.y); return z; }
  };
  // one direction's line: out += c T + D^T (T + c u) [- i kappa T], T = D u;
  // without a GGA field out += K u (real) or D^T T - i kappa T
  Table1D<NP, NQ, TC> tn;              // N' (filter steps: N' D^-1)
  Table1D<NQ, NP, TC, true> tt;        // N'^T
  Table1D<NQ, NQ, TC> td;              // the current direction's D (or K)
  Table1D<NQ, NQ, TC, true> th;        // D^T
  auto stage_tables = [&](int d) {
    td.load(a.ptab + (GGA || CPLX ? L.d : L.k) + d * L.dsz);
    if constexpr (GGA || CPLX) th.load(td, a.ptab + L.dh + d * L.dsz);
  };
  auto stage = [&](auto dtag, const V (&u)[NQ], V (&o)[NQ], const TC (&c)[NQ]) {
    constexpr int D = decltype(dtag)::value;
    if constexpr (GGA || CPLX) {
      V T[NQ];
      eo<-1, false>(td, u, T);
      line_end<TC>();
      if constexpr (CPLX) {
        const TC kap = a.pkap[D];
#pragma unroll
        for (int i = 0; i < NQ; ++i) o[i] = bloch(kap, T[i], o[i]);
      }
      if constexpr (GGA) {
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          o[i] = vfma(c[i], T[i], o[i]);
          T[i] = vfma(c[i], u[i], T[i]);
        }
      }
      line_end<TC>();
      eo<-1, true>(th, T, o);
    } else {
      eo<1, true>(td, u, o);
    }
  };

  V carry[NP];
#pragma unroll
  for (int i = 0; i < NP; ++i) carry[i] = 0;
  // Blocks narrower than the arithmetic (BF16): an uncut periodic column's
  // first plane, held for the last cell's, so that their sum rounds once as at
  // every other plane.  (Elsewhere it waits in Y, exactly.)
  constexpr bool HOLD = sizeof(TS) != sizeof(TC);
  const bool wrap = a.nseg == 1 && !zoff;
  V held[HOLD ? NP : 1];
#pragma unroll
  for (int i = 0; i < (HOLD ? NP : 1); ++i) held[i] = 0;

  V w[NQ][NQ];                                           // the plane [x][y]
  typename IO::R wr[NP][NP];                             // the next cell's, as stored
  // gather of the (x, y) plane at node z = pl of cell cz (a thread past the
  // node planes repeats the last one; its results are not used)
  auto gather = [&](int cz) {
    int gz = cz * p + (NP == NQ ? pl : min(pl, NP - 1)) - zoff;
    gz = gz >= 0 && gz < a.M2 ? gz : 0;
    const TS *const zp = Xl + gz * MM * a.ldx;
    const int64_t rs = opaque(a.M0 * a.ldx), sx = opaque(a.ldx);
    const TS *row = zp + gyf * rs;
    const TS *next = zp + (int64_t)(gy0 + 1) * rs;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      wr[0][j] = IO::ld(row + gxf * sx);
      const TS *q = row + (gx0 + 1) * sx;
#pragma unroll
      for (int i = 1; i < NP - 1; ++i, q += sx) wr[i][j] = IO::ld(q);
      wr[NP - 1][j] = IO::ld(row + gxl * sx);
      if (j == NP - 2) row = zp + gyl * rs;
      else { row = next; next += rs; }
    }
  };
  // coefficients of a stage's line, read one line ahead
  const TC *cell = nullptr;
  auto coef_z = [&](int i, TC (&vl)[NQ], TC (&c)[NQ]) {
    const auto q = reinterpret_cast<cptr<TC>>(reinterpret_cast<uint64_t>(cell + pl * (2 * NQ)));
#pragma unroll
    for (int z = 0; z < NQ; ++z) {
      vl[z] = q[i * (2 * NQ2) + 2 * z];
      if constexpr (GGA) c[z] = q[i * (2 * NQ2) + 2 * z + 1];
    }
  };
  auto coef_xy = [&](int block, int line, TC (&c)[NQ]) {
    const auto q = reinterpret_cast<cptr<TC>>(reinterpret_cast<uint64_t>(cell + block * NQ3 + pl * NQ));
    if constexpr (GGA)
#pragma unroll
      for (int i = 0; i < NQ; ++i) c[i] = q[line * NQ2 + i];
  };
  auto cell_of = [&](int cz) { return a.pcoef + (cx + (int64_t)a.N0 * (cy + (int64_t)a.N1 * cz)) * (4 * NQ3); };
  constexpr int NR = NQ - S::NS;                         // sums parked in registers
  V orr[NR > 0 ? NR : 1][NQ];

  TC cn[NQ];
  const int c0 = seg_start(seg, a.N2, a.nseg), c1 = seg_start(seg + 1, a.N2, a.nseg);
  gather(c0);
  tn.load(a.pgather);
  if constexpr (!MASS) stage_tables(2);
  for (int cz = c0; cz < c1; ++cz) {
    cell = cell_of(cz);
    if (a.dmask) {
      const int gz = cz * p + pl - zoff;
      const bool zin = !zoff || (gz >= 0 && gz < a.M2);
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const bool in = zin && (j != 0 || y0) && (j != NP - 1 || y1);
#pragma unroll
        for (int i = 0; i < NP; ++i)
          wr[i][j] = in && (i != 0 || x0) && (i != NP - 1 || x1) ? wr[i][j] : (typename IO::R)0;
      }
    }
    // A: N along x
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      V x[NP], y[NQ];
#pragma unroll
      for (int i = 0; i < NP; ++i) x[i] = IO::up(wr[i][j]);
      eo<1, false>(tn, x, y);
#pragma unroll
      for (int i = 0; i < NQ; ++i) w[i][j] = y[i];
      line_end<TC>();
    }
    if constexpr (MASS) {
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        V y[NP];
        eo<1, false>(tn, w[i], y);
#pragma unroll
        for (int j = 0; j < NP; ++j) w[i][j] = in_line<TC>(y[j]);
      }
    } else {
    // B per x (those parked in registers first, through slot 0): N along y,
    // exchange, N along z, u back to (x, y) planes, the z-direction stage and
    // the potential parked
#pragma unroll
    for (int ii = 0; ii < NQ; ++ii) {
      const int i = ii < NR ? NQ - 1 - ii : ii - NR;
      V *slot = B + (ii < NR ? 0 : i) * S::SLOT + v;
      V *sw = slot + pl * S::SZ, *sr = slot + pl * S::SY;
      TC vl[NQ], cc[NQ];
      coef_z(i, vl, cc);                                 // used after three sweeps
      if (ii == NQ - 1) coef_xy(2, 0, cn);
      {
        V x[NP], y[NQ];
#pragma unroll
        for (int j = 0; j < NP; ++j) x[j] = w[i][j];
        eo<1, false>(tn, x, y);
#pragma unroll
        for (int q = 0; q < NQ; ++q) sw[q * S::SY] = y[q];
      }
      line_end<TC>();
      wave_order();
      V x[NP], u[NQ], o[NQ];
#pragma unroll
      for (int k = 0; k < NP; ++k) x[k] = sr[k * S::SZ];
      wave_order();
      eo<1, false>(tn, x, u);
#pragma unroll
      for (int q = 0; q < NQ; ++q) sr[q * S::SZ] = u[q];
      wave_order();
#pragma unroll
      for (int q = 0; q < NQ; ++q) w[i][q] = sw[q * S::SY];
      wave_order();
#pragma unroll
      for (int q = 0; q < NQ; ++q) o[q] = vl[q] * u[q];
      stage(std::integral_constant<int, 2>{}, u, o, cc);
#pragma unroll
      for (int q = 0; q < NQ; ++q) sr[q * S::SZ] = o[q];
      if (ii < NR) {
        wave_order();
#pragma unroll
        for (int q = 0; q < NQ; ++q) orr[NQ - 1 - i][q] = sw[q * S::SY];
        wave_order();
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    stage_tables(0);
    wave_order();
    // C: the x-direction stage added to the parked sums, row by row
#pragma unroll
    for (int j = 0; j < NQ; ++j) {
      V *sw = B + v + pl * S::SZ + j * S::SY;
      V u[NQ], o[NQ];
      TC cc[NQ];
#pragma unroll
      for (int i = 0; i < NQ; ++i) cc[i] = cn[i];
      coef_xy(j + 1 < NQ ? 2 : 3, j + 1 < NQ ? j + 1 : 0, cn);
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        u[i] = w[i][j];
        o[i] = i < S::NS ? sw[i * S::SLOT] : orr[NQ - 1 - i][j];
      }
      stage(std::integral_constant<int, 0>{}, u, o, cc);
#pragma unroll
      for (int i = 0; i < NQ; ++i) {
        if (i < S::NS) sw[i * S::SLOT] = o[i];
        else orr[NQ - 1 - i][j] = o[i];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    stage_tables(1);
    tt.load(a.ptab, L);
    wave_order();
    // the y-direction stage completes the sum; N^T along y
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      const V *sw = B + v + pl * S::SZ + i * S::SLOT;
      V u[NQ], o[NQ], y[NP];
      TC cc[NQ];
#pragma unroll
      for (int j = 0; j < NQ; ++j) cc[j] = cn[j];
      if (i + 1 < NQ) coef_xy(3, i + 1, cn);
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        u[j] = w[i][j];
        o[j] = i < S::NS ? sw[j * S::SY] : orr[NQ - 1 - i][j];
      }
      stage(std::integral_constant<int, 1>{}, u, o, cc);
      eo<1, false>(tt, o, y);
#pragma unroll
      for (int j = 0; j < NP; ++j) w[i][j] = in_line<TC>(y[j]);
      __builtin_amdgcn_sched_barrier(0);
    }
    }
    wave_order();
    // The values this cell's scatter reads back, RB lines ahead of their use.  The
    // last plane of a cell is carried to the next one (after the column's last
    // cell to its first plane), so a cell stores the other NP - 1.
    const int64_t sy = opaque(a.ldy), sz = opaque(MM * a.ldy);
    const bool z0 = cz * p >= zoff;                      // the first plane holds DoFs
    TS *const Yz = (TS *)a.Y + (cz * p - zoff) * sz;
    TS *const Y0 = z0 ? Yz : Yz + sz;
    // a cut segment's first plane goes to the side block instead
    const bool cut0 = a.nseg > 1 && cz == c0;
    const bool hold0 = HOLD && wrap && cz == 0;
    TC *const side0 = side_at(seg, 0);
    const unsigned rd0 = cut0 ? BUF_OFF : or0, rd1 = cut0 ? BUF_OFF : or1, rdm = cut0 ? BUF_OFF : orm;
    typename IO::R old[NP][NP - 1];                      // [x][z]
    auto xnode = [&](int i) { return (i == 0 ? gxf : i == NP - 1 ? gxl : gx0 + i) * sy; };
    auto read_back = [&](int i) {
      const unsigned o = i == 0 ? or0 : i == NP - 1 ? or1 : orm;
      old[i][0] = IO::ldb(buf_at(opaque(Y0) + xnode(i)), (int)(i == 0 ? rd0 : i == NP - 1 ? rd1 : rdm));
      TS *q = opaque(Yz) + xnode(i);
#pragma unroll
      for (int k = 1; k < NP - 1; ++k) old[i][k] = IO::ldb(buf_at(q += sz), (int)o);
    };
    // x of the ii-th scatter line: those without a slot come after x = 0
    constexpr int NX = NP > S::NS ? NP - S::NS : 0;
    auto line = [](int ii) { return ii == 0 ? 0 : ii <= NX ? S::NS + ii - 1 : ii - NX; };
#pragma unroll
    for (int ii = 0; ii < (RB < NP ? RB : NP); ++ii) read_back(line(ii));
    // N^T along x, to (x, z) planes (an x without a slot follows in slot 0)
    V we[NP > S::NS ? NP - S::NS : 1][NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      V x[NQ], y[NP];
#pragma unroll
      for (int i = 0; i < NQ; ++i) x[i] = w[i][j];
      if constexpr (MASS) {
#pragma unroll
        for (int i = 0; i < NP; ++i) y[i] = x[i];
      } else {
        eo<1, false>(tt, x, y);
      }
      V *sw = B + v + pl * S::SZ + j * S::SY;
#pragma unroll
      for (int i = 0; i < NP; ++i) {
        if (i < S::NS) sw[i * S::SLOT] = y[i];
        else we[i - S::NS][j] = y[i];
      }
      line_end<TC>();
    }
    wave_order();
    __builtin_amdgcn_sched_barrier(0);
    // the next cell's plane, in flight from here on
    if (cz + 1 < c1) {
      gather(cz + 1);
    } else {                                             // (none of this cell's is live past here)
#pragma unroll
      for (int i = 0; i < NP * NP; ++i) wr[i / NP][i % NP] = 0;
    }
    __builtin_amdgcn_sched_barrier(0);
    // D: N^T along z, the plane shared with the next cell, scatter
#pragma unroll
    for (int ii = 0; ii < NP; ++ii) {
      const int i = line(ii);
      if (ii + RB < NP) read_back(line(ii + RB));
      if (!MASS && ii == NP - 2 && cz + 1 < c1) {
        tn.load(a.pgather);
        stage_tables(2);
      }
      const V *sr = B + v + pl * S::SY + (i < S::NS ? i : 0) * S::SLOT;
      if (i >= S::NS) {
        V *sw = B + v + pl * S::SZ;
#pragma unroll
        for (int j = 0; j < NP; ++j) sw[j * S::SY] = we[i - S::NS][j];
        wave_order();
      }
      V z[NQ], y[NP];
#pragma unroll
      for (int q = 0; q < NQ; ++q) z[q] = sr[q * S::SZ];
      if (ii <= NX) wave_order();
      if constexpr (MASS) eo<1, false>(tn, z, y);
      else eo<1, false>(tt, z, y);
      y[0] += carry[i];
      carry[i] = y[NP - 1];
      const unsigned oi = i == 0 ? ow0 : i == NP - 1 ? ow1 : ow;
      if constexpr (HOLD) {
        held[i] = hold0 ? y[0] : held[i];
        IO::stb(buf_at(opaque(Y0) + xnode(i)), (int)(z0 && !cut0 && !hold0 ? oi : BUF_OFF), IO::up(old[i][0]) + y[0]);
        SideIO::stb(buf_at(opaque(side0) + i * side_x), (int)(cut0 ? so : BUF_OFF), y[0]);
      } else {
        TS *const q0 = cut0 ? opaque(side0) + i * side_x : opaque(Y0) + xnode(i);
        IO::stb(buf_at(q0), (int)(cut0 ? so : z0 ? oi : BUF_OFF), IO::up(old[i][0]) + y[0]);
      }
      TS *q = opaque(Yz) + xnode(i);
#pragma unroll
      for (int k = 1; k < NP - 1; ++k) IO::stb(buf_at(q += sz), (int)oi, IO::up(old[i][k]) + y[k]);
      line_end<TC>();
    }
    wave_order();
  }
  // The last plane: of a segment, the cut it shares with the next one's first;
  // of a whole column on a periodic axis the column's first plane (stored by
  // this thread already and read back by all, or held).  A Dirichlet axis has
  // no DoFs there.
  if (a.nseg > 1) {
    TC *const side1 = side_at(seg + 1 < a.nseg ? seg + 1 : 0, 1);
#pragma unroll
    for (int i = 0; i < NP; ++i) SideIO::stb(buf_at(side1 + i * side_x), (int)so, carry[i]);
  } else if (wrap) {
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const BufRsrc r = buf_at((TS *)a.Y + (int64_t)(i == 0 ? gxf : i == NP - 1 ? gxl : gx0 + i) * a.ldy);
      const unsigned oi = i == 0 ? ow0 : i == NP - 1 ? ow1 : ow;
      const unsigned o = !HOLD ? oi : i == 0 ? or0 : i == NP - 1 ? or1 : orm;
      V z = carry[i];
      if constexpr (HOLD) z += held[i];
      IO::stb(r, (int)oi, IO::up(IO::ldb(r, (int)o)) + z);
    }
  }
}

// Waves are independent; they are grouped into blocks of four, which the
// device spreads over a CU's four SIMDs (single-wave blocks may share one
// while others idle).
constexpr int PLANE_WPB = 4;
#define FEHX_PLANE_WAVES (plane_waves(NQ, sizeof(TC) == 8, LPT))
#define FEHX_PLANE_BOUNDS __launch_bounds__(64 * PLANE_WPB) __attribute__((amdgpu_waves_per_eu(FEHX_PLANE_WAVES, FEHX_PLANE_WAVES)))

template <int NP, int NQ, bool CPLX, typename TS, typename TC, int LPT, bool MASS>
__device__ __forceinline__ void plane_item(const KArgs<TC> &a, int w) {
  const int cs = w / a.ntiles, tile = w - cs * a.ntiles;
  const int col = cs / a.nseg, seg = cs - col * a.nseg;
  if constexpr (MASS) {
    plane_column<NP, NQ, CPLX, false, TS, TC, LPT, true>(a, col, seg, tile);
  } else {
    if (a.gga) plane_column<NP, NQ, CPLX, true, TS, TC, LPT, false>(a, col, seg, tile);
    else plane_column<NP, NQ, CPLX, false, TS, TC, LPT, false>(a, col, seg, tile);
  }
}

template <int NP, int NQ, bool CPLX, typename TS, typename TC, int LPT, bool MASS>
__global__ void FEHX_PLANE_BOUNDS k_planes(KArgs<TC> a) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = xcd_item(blockIdx.x, gridDim.x) * PLANE_WPB + wv;
  if (w >= a.ncols * a.nseg * a.ntiles) return;
  plane_item<NP, NQ, CPLX, TS, TC, LPT, MASS>(a, w);
}

template <int NP, int NQ, bool CPLX, typename TS, typename TC, int LPT, bool MASS>
__global__ void FEHX_PLANE_BOUNDS k_planes_batch(BatchArgs<TC> Bt) {
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int w = xcd_item(blockIdx.x, gridDim.x) * PLANE_WPB + wv;
  if (w >= Bt.total) return;
  int sidx = 0;
  while (sidx + 1 < Bt.nsys && w >= Bt.off[sidx + 1]) ++sidx;
  plane_item<NP, NQ, CPLX, TS, TC, LPT, MASS>(Bt.sys[sidx], w - Bt.off[sidx]);
}

// blocks above 64 KiB raise the kernel's dynamic-LDS attribute first
inline hipError_t plane_lds(const void *kern, size_t shm) {
  return shm > 65536 ? hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm) : hipSuccess;
}
inline unsigned plane_grid(int waves) {
  const int b = (waves + PLANE_WPB - 1) / PLANE_WPB;
  return (unsigned)((b + 7) / 8 * 8);
}

template <int NP, int NQ, bool CPLX, typename TS, typename TC, int LPT, bool MASS = false>
inline fe_status run_planes(const LocalBatch &Bt, hipStream_t s) {
  typedef PlaneShape<NQ, CPLX, LPT> S;
  constexpr size_t shm = (size_t)S::elems * LPT * sizeof(TC) * PLANE_WPB;
  static_assert(shm * plane_waves(NQ, sizeof(TC) == 8, LPT) <= LDS_MAX, "the plane exchange exceeds the LDS");
  const bool single = Bt.n == 1 && !Bt.persistent;
  const void *kern = single ? (const void *)k_planes<NP, NQ, CPLX, TS, TC, LPT, MASS> : (const void *)k_planes_batch<NP, NQ, CPLX, TS, TC, LPT, MASS>;
  FE_HIP_TRY(plane_lds(kern, shm));
  std::vector<KArgs<TC>> as;
  SideUse use;
  segments_begin<TC>(Bt, S::VT, [](Mesh *m, const LocalLaunch &L, int, int64_t side_bytes) {
    return plane_segment_count(m, NQ, L.nlanes, sizeof(TC) == 8, LPT, side_bytes, nullptr);
  }, as, use, s);
  int nphase = 0;
  for (int i = 0; i < Bt.n; ++i) {
    if constexpr (MASS) as[i].pgather = as[i].ptab + plane_tab(Bt.ms[i]->np, Bt.ms[i]->nq).m;
    nphase = std::max(nphase, Bt.ms[i]->nphase);
  }
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
        KArgs<TC> &a = B.sys[B.nsys];
        a = as[i0];
        a.cols = m->cols + 2 * m->phase_off[ph];
        a.ncols = ncols;
        B.off[B.nsys + 1] = B.off[B.nsys] + ncols * a.nseg * a.ntiles;
        ++B.nsys;
      }
      if (B.nsys == 0) continue;
      B.total = B.off[B.nsys];
      const dim3 grid(plane_grid(B.total)), block(64 * PLANE_WPB);
      if (single) hipLaunchKernelGGL((k_planes<NP, NQ, CPLX, TS, TC, LPT, MASS>), grid, block, shm, s, B.sys[0]);
      else hipLaunchKernelGGL((k_planes_batch<NP, NQ, CPLX, TS, TC, LPT, MASS>), grid, block, shm, s, B);
      FE_HIP_TRY(hipGetLastError());
    }
  }
  return segments_end<TS, TC>(S::VT, as, true, s);
}

template <int NP, int NQ> fe_status pick_planes_f64(const LocalBatch &B, hipStream_t s) {
  if (B.kind != LOCAL_PLANES) return pick_cplx_f64<NP, NQ>(B, s);
  return B.ms[0]->cplx ? run_planes<NP, NQ, true, double, double, 1>(B, s)
                       : run_planes<NP, NQ, false, double, double, 1>(B, s);
}

// FP32 and BF16: threads of two adjacent lanes (a complex vector) or, real, of one
template <int NP, int NQ, typename TS> bool run_planes_f32(const LocalBatch &B, hipStream_t s, fe_status *st) {
  if (B.kind != LOCAL_PLANES && B.kind != LOCAL_PLANES_PAIRS) return false;
  const bool cplx = B.ms[0]->cplx;
  const bool pairs = B.kind == LOCAL_PLANES_PAIRS && (cplx || plane_pairs_pay(B, NQ));
  *st = cplx ? run_planes<NP, NQ, true, TS, float, 2>(B, s)
             : pairs ? run_planes<NP, NQ, false, TS, float, 2>(B, s) : run_planes<NP, NQ, false, TS, float, 1>(B, s);
  return true;
}
template <int NP, int NQ> fe_status pick_planes_f32(const LocalBatch &B, hipStream_t s) {
  fe_status st = FE_OK;
  return run_planes_f32<NP, NQ, float>(B, s, &st) ? st : pick_cplx_f32<NP, NQ>(B, s);
}
template <int NP, int NQ> fe_status pick_planes_bf16(const LocalBatch &B, hipStream_t s) {
  fe_status st = FE_OK;
  return run_planes_f32<NP, NQ, bf16s>(B, s, &st) ? st : pick_cplx_bf16<NP, NQ>(B, s);
}

}  // namespace fehx
