// Nonlocal kernel regression (Eqs. 6.5-6.6).  The operator
//   L_c[u](x) = sum over grid offsets 0 < |r| < delta of K(r) (u(x + r) - u(x)),
// K = K1(|r|) I (form 0) or K1 I + K2 e e^T, e = r / |r| (form 1), in the
// Bernstein basis B_m(|r| / delta), and the normal equations of its fit.
//
// A workgroup stages a tile of the periodic field and its halo of width R
// (the largest offset component) in LDS.  Lanes run over the A axis (x) and
// the B axis (y in 3D; in 2D the second lane index stacks runs of the C axis
// instead), and a thread owns ZV consecutive voxels along the C axis (z in
// 3D, y in 2D).  For one (dA, dB) of the horizon a thread reads the column of
// ZV + 2 R values along C once and serves all its voxels and all dC from
// registers.  A read of the LDS per offset and voxel bounded the kernels
// before: 523 of them per voxel at delta = 5.  Columns cost 69 (ZV + 8) / ZV
// there, 207 at ZV = 4 and 138 at ZV = 8.
#include <atomic>
#include <hip/hip_runtime.h>

#include <vector>

#include "fft_core.hpp"
#include "launch.hpp"
#include "lsfft_internal.hpp"

namespace lsfft {
namespace {

constexpr int NT = 256;                 // threads of every kernel here
// workgroups of the Gram kernels (two and four to a CU): fixed, so the sum
// order never depends on the device
constexpr int kSlots = 512, kSlots1 = 1024;

typedef double d4 __attribute__((ext_vector_type(4)));

// LDS entries from one C index to the next: compile-time, so that a column's
// reads are one address with immediate offsets (a runtime stride spent half
// of the vector instructions on addresses).  3D: room for both lane shapes,
// 32 x 8 and 16 x 16; 2D: the rows of 32 lanes.  (Matrix-form tiles are dense.)
template <int R, int DIM> struct Pitch {
  static constexpr int C = DIM == 3 ? (32 + 2 * R) * (8 + 2 * R) : 32 + 2 * R;
};
constexpr int pitch_c(int R, int dim) { return dim == 3 ? (32 + 2 * R) * (8 + 2 * R) : 32 + 2 * R; }

struct Geom {
  int nA, nB, nC;          // grid (2D: nB = 1)
  int dim;
  int ta, tb;              // lanes along A, second lane index
  int R;                   // halo
  int la, lb, lc;          // LDS box
  int sC;                  // LDS entries from one C index to the next
  int ntA, ntB, ntC;       // tiles
  int bv, cv;              // voxels of a tile along B and C
  int tpr;                 // threads staging one box row (power of two)
};

// tile `tile`: origin, this thread's lane coordinates and its first voxel
struct Spot {
  int a0, b0, c0;          // tile origin
  int a, b, c;             // this thread's first voxel
  int base;                // LDS index of (a, b, c - R) with the halo of A and B added
  bool in;                 // a and b inside the grid
};
__device__ __forceinline__ Spot spot(const Geom& G, int tile, int zv) {
  Spot s;
  const int tA = tile % G.ntA, rest = tile / G.ntA;
  const int tB = rest % G.ntB, tC = rest / G.ntB;
  s.a0 = tA * G.ta;
  s.b0 = tB * G.bv;
  s.c0 = tC * G.cv;
  const int al = threadIdx.x % G.ta, r2 = threadIdx.x / G.ta;
  const int l2 = r2 % G.tb, l3 = r2 / G.tb;      // l3: further runs along C (matrix-form tiles)
  s.a = s.a0 + al;
  if (G.dim == 3) {
    s.b = s.b0 + l2;
    s.c = s.c0 + l3 * zv;
    s.base = l3 * zv * G.sC + (l2 + G.R) * G.la + al + G.R;
  } else {
    s.b = 0;
    s.c = s.c0 + (l3 * G.tb + l2) * zv;
    s.base = (l3 * G.tb + l2) * zv * G.sC + al + G.R;
  }
  s.in = s.a < G.nA && s.b < G.nB;
  return s;
}
__device__ __forceinline__ long long voxel(const Geom& G, const Spot& s, int v) {
  return ((long long)(s.c + v) * G.nB + s.b) * G.nA + s.a;
}
__device__ __forceinline__ bool live(const Geom& G, const Spot& s, int v) { return s.in && s.c + v < G.nC; }

__device__ __forceinline__ int wrapped(int v, int n) {
  v %= n;
  return v < 0 ? v + n : v;
}

// Rows of the box of one tile, made once for its components: where each row
// starts in a component of the field and in the box.
constexpr int kRows = 576;               // at most (16 + 12)(8 + 12) (checked by rows_ok)
constexpr int kRowBytes = 8 * kRows;     // at the front of the LDS
__device__ __forceinline__ void row_table(const Geom& G, const Spot& s, int2* tab) {
  const int rows = G.lb * G.lc, hb = (G.dim == 3) ? G.R : 0;
  for (int row = threadIdx.x; row < rows; row += NT) {
    const int iz = row / G.lb, iy = row - iz * G.lb;
    const int gy = wrapped(s.b0 - hb + iy, G.nB), gz = wrapped(s.c0 - G.R + iz, G.nC);
    tab[row] = make_int2(gz * G.nB + gy, iz * G.sC + iy * G.la);
  }
}

// Stage one component's box (entries IL apart): tpr threads per row.  Eight
// rows' loads are in flight before the first is stored: one at a time, with
// the row's coordinates stepped along, the scalar normal equations took 468
// us instead of 327.
template <int IL, typename T>
__device__ __forceinline__ void stage(const Geom& G, const T* __restrict__ u, const Spot& s, const int2* tab, T* lds) {
  constexpr int U = 8;
  const int ix0 = threadIdx.x & (G.tpr - 1), step = NT / G.tpr;
  const int rows = G.lb * G.lc;
  const int gx = wrapped(s.a0 - G.R + ix0, G.nA);
  if (ix0 >= G.la) return;
  for (int row = threadIdx.x / G.tpr; row < rows; row += U * step) {
    T v[U];
    int at[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int2 r = tab[min(row + j * step, rows - 1)];   // past the end: the last row again
      at[j] = r.y;
      v[j] = u[(long long)r.x * G.nA + gx];
    }
#pragma unroll
    for (int j = 0; j < U; ++j) lds[(at[j] + ix0) * IL] = v[j];
  }
}

// ---------------------------------------------------------------------------
// scalar form
// ---------------------------------------------------------------------------
// Offsets folded into classes: the columns (dA, dB) of one |dA|, |dB| pair (in
// either order in 3D) share every weight, so their sum E along C is formed
// first, then E(c + dC) + E(c - dC), less u(x) as often as there are offsets in
// it: subtracted once for the whole horizon instead, the error of a field with a
// rigid offset was 2 to 24 times larger (horizons 1.5 to 6).  FP32 fields are
// rounded at 6e-8 of their offset, far above either: there the weight of r = 0 is
// minus the sum of all others (eight 64^3 fields at horizon 3: the operator in 70
// us against 81).  cls[4 k]: columns of class k (first, count), its largest dC, and
// its first weight row; `col` holds the columns' LDS offsets.  Class 0 is the column
// of r = 0.
template <typename T> constexpr bool by_class() { return sizeof(T) == 8; }
template <typename T, int R, int DIM, int ZV>
__device__ __forceinline__ void column_sums(const T* lds, int base, const int* __restrict__ col, int n,
                                            double (&E)[ZV + 2 * R]) {
#pragma unroll
  for (int w = 0; w < ZV + 2 * R; ++w) E[w] = 0.0;
  int k = 0;
  for (; k + 2 <= n; k += 2) {   // two columns' reads in flight
    const T* p = lds + base + col[k];
    const T* q = lds + base + col[k + 1];
    T x[ZV + 2 * R], y[ZV + 2 * R];
#pragma unroll
    for (int w = 0; w < ZV + 2 * R; ++w) {
      x[w] = p[w * Pitch<R, DIM>::C];
      y[w] = q[w * Pitch<R, DIM>::C];
    }
#pragma unroll
    for (int w = 0; w < ZV + 2 * R; ++w) E[w] += double(x[w]) + double(y[w]);
  }
  if (k < n) {
    const T* p = lds + base + col[k];
#pragma unroll
    for (int w = 0; w < ZV + 2 * R; ++w) E[w] += double(p[w * Pitch<R, DIM>::C]);
  }
}

// Normal equations: workgroup b walks the items (sample, tile) b, b + grid,
// ... in order and keeps the upper triangle of Phi Phi^T, Phi . Gamma and
// Gamma . Gamma per thread in FP64; the workgroup's sums go to its slot.
// Bound by FP64 issue (about 620 operations per voxel and component at
// delta = 5, degree 6) and LDS reads (207).  On eight 64^3 FP64 fields there:
// 327 us, against 1250 us with a read per offset and a triangle of nine
// features whatever the degree.
template <typename T, int R, int DIM, int NF>
__global__ __launch_bounds__(NT) void k_nl_gram(Geom G, const T* __restrict__ u, const T* __restrict__ gam, int nsample,
                                                const int* __restrict__ cls, int ncls, const int* __restrict__ col,
                                                const double* __restrict__ W, double* __restrict__ partial) {
  constexpr int ZV = 4;
  constexpr int TRI = NF * (NF + 1) / 2, NACC = TRI + NF + 1;
  extern __shared__ __align__(16) unsigned char smem[];
  int2* tab = reinterpret_cast<int2*>(smem);
  T* lds = reinterpret_cast<T*>(smem + kRowBytes);
  const long long nvox = (long long)G.nA * G.nB * G.nC;
  const int ntile = G.ntA * G.ntB * G.ntC;
  double acc[NACC];
#pragma unroll
  for (int i = 0; i < NACC; ++i) acc[i] = 0.0;
  for (long long item = blockIdx.x; item < (long long)nsample * ntile; item += gridDim.x) {
    const int k = int(item / ntile);
    const Spot s = spot(G, int(item - (long long)k * ntile), ZV);
    __syncthreads();
    row_table(G, s, tab);
    for (int a = 0; a < DIM; ++a) {
      const long long comp = ((long long)k * DIM + a) * nvox;
      __syncthreads();
      stage<1>(G, u + comp, s, tab, lds);
      __syncthreads();
      double phi[ZV][NF], u0[ZV];
#pragma unroll
      for (int v = 0; v < ZV; ++v) {
        if (by_class<T>()) u0[v] = double(lds[s.base + (v + R) * Pitch<R, DIM>::C]);
#pragma unroll
        for (int m = 0; m < NF; ++m) phi[v][m] = 0.0;
      }
      for (int q = 0; q < ncls; ++q) {
        const int c0 = cls[4 * q], cn = cls[4 * q + 1], zr = cls[4 * q + 2];
        const double* w = W + cls[4 * q + 3] * NF;
        double E[ZV + 2 * R];
        column_sums<T, R, DIM, ZV>(lds, s.base, col + c0, cn, E);
#pragma unroll
        for (int d = 0; d <= R; ++d) {
          if (d > zr) break;
          if (by_class<T>() && d == 0 && q == 0) continue;
          const double n = double(d ? 2 * cn : cn);
#pragma unroll
          for (int v = 0; v < ZV; ++v) {
            double D = d ? E[v + R + d] + E[v + R - d] : E[v + R];
            if (by_class<T>()) D = __builtin_fma(-n, u0[v], D);
#pragma unroll
            for (int m = 0; m < NF; ++m) phi[v][m] += w[d * NF + m] * D;
          }
        }
      }
#pragma unroll
      for (int v = 0; v < ZV; ++v) {
        if (!live(G, s, v)) continue;
        const double gv = double(gam[comp + voxel(G, s, v)]);
        int i = 0;
#pragma unroll
        for (int m = 0; m < NF; ++m)
#pragma unroll
          for (int n2 = m; n2 < NF; ++n2, ++i) acc[i] += phi[v][m] * phi[v][n2];
#pragma unroll
        for (int m = 0; m < NF; ++m) acc[TRI + m] += phi[v][m] * gv;
        acc[TRI + NF] += gv * gv;
      }
    }
  }
  // workgroup sum in a fixed order: waves by shuffles, then across waves
  double* red = reinterpret_cast<double*>(smem + kRowBytes);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < NACC; ++i) {
    double v = acc[i];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    if (lane == 0) red[wave * NACC + i] = v;
  }
  __syncthreads();
  if ((int)threadIdx.x < NACC) {
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += red[w * NACC + threadIdx.x];
    partial[(long long)blockIdx.x * NACC + threadIdx.x] = t;
  }
}

// The fitted scalar operator, one workgroup per (sample, tile): LDS reads
// (138 per voxel and component at delta = 5) bound it.  On eight 64^3 FP64
// fields there: 235 us, against 601 us with a read per offset.
template <typename T, int R, int DIM>
__global__ __launch_bounds__(NT) void k_nl_apply(Geom G, const T* __restrict__ u, int nsample,
                                                 const int* __restrict__ cls, int ncls, const int* __restrict__ col,
                                                 const double* __restrict__ kw, T* __restrict__ out) {
  constexpr int ZV = 8;
  extern __shared__ __align__(16) unsigned char smem[];
  int2* tab = reinterpret_cast<int2*>(smem);
  T* lds = reinterpret_cast<T*>(smem + kRowBytes);
  const long long nvox = (long long)G.nA * G.nB * G.nC;
  const int ntile = G.ntA * G.ntB * G.ntC;
  const long long item = blockIdx.x;
  if (item >= (long long)nsample * ntile) return;
  const int k = int(item / ntile);
  const Spot s = spot(G, int(item - (long long)k * ntile), ZV);
  row_table(G, s, tab);
  for (int a = 0; a < DIM; ++a) {
    const long long comp = ((long long)k * DIM + a) * nvox;
    __syncthreads();
    stage<1>(G, u + comp, s, tab, lds);
    __syncthreads();
    double r[ZV], u0[ZV];
#pragma unroll
    for (int v = 0; v < ZV; ++v) {
      r[v] = 0.0;
      if (by_class<T>()) u0[v] = double(lds[s.base + (v + R) * Pitch<R, DIM>::C]);
    }
    for (int q = 0; q < ncls; ++q) {
      const int c0 = cls[4 * q], cn = cls[4 * q + 1], zr = cls[4 * q + 2];
      const double* w = kw + cls[4 * q + 3];
      double E[ZV + 2 * R];
      column_sums<T, R, DIM, ZV>(lds, s.base, col + c0, cn, E);
#pragma unroll
      for (int d = 0; d <= R; ++d) {
        if (d > zr) break;
        if (by_class<T>() && d == 0 && q == 0) continue;
        const double n = double(d ? 2 * cn : cn);
#pragma unroll
        for (int v = 0; v < ZV; ++v) {
          double D = d ? E[v + R + d] + E[v + R - d] : E[v + R];
          if (by_class<T>()) D = __builtin_fma(-n, u0[v], D);
          r[v] += w[d] * D;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < ZV; ++v)
      if (live(G, s, v)) out[comp + voxel(G, s, v)] = T(r[v]);
  }
}

// ---------------------------------------------------------------------------
// matrix form
// ---------------------------------------------------------------------------
// The fitted matrix operator: per staged input component b and pair of offsets
// r, -r, whose coefficients are the same,
//   out_a += (K1 delta_ab + K2 e_a e_b) ((u_b(x + r) - u_b(x)) + (u_b(x - r) - u_b(x))).
// The differences are formed first, so that a constant field gives zero and a
// rigid offset costs no digits (weights times u(x + r), less their sum times u(x),
// lost 4e5 in accuracy at an offset of 1e6).  cls[4 k] holds a column (dA, dB) and
// its opposite (their LDS offsets), the largest dC and the row of dC = 0; the
// column of r = 0 is its own opposite and takes dC > 0 only.  kw has the three
// coefficients [a] per offset of the first column, one table per b.
// FP64 issue bounds it (276 operations per voxel and input component at
// delta = 3, on 21 (ZV + 4) / ZV LDS reads).  On eight 64^3 FP64 fields there:
// 107 us, against 298 us with a read per offset.
template <typename T, int R, int DIM>
__global__ __launch_bounds__(NT) void k_nl_apply1(Geom G, const T* __restrict__ u, int nsample,
                                                  const int* __restrict__ cls, int ncls,
                                                  const double* __restrict__ kw, int nkw,
                                                  T* __restrict__ out) {
  constexpr int ZV = 8;
  extern __shared__ __align__(16) unsigned char smem[];
  int2* tab = reinterpret_cast<int2*>(smem);
  T* lds = reinterpret_cast<T*>(smem + kRowBytes);
  const long long nvox = (long long)G.nA * G.nB * G.nC;
  const int ntile = G.ntA * G.ntB * G.ntC;
  const long long item = blockIdx.x;
  if (item >= (long long)nsample * ntile) return;
  const int k = int(item / ntile);
  const Spot s = spot(G, int(item - (long long)k * ntile), ZV);
  row_table(G, s, tab);
  double r[3][ZV];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int v = 0; v < ZV; ++v) r[a][v] = 0.0;
  for (int b = 0; b < DIM; ++b) {
    __syncthreads();
    stage<1>(G, u + ((long long)k * DIM + b) * nvox, s, tab, lds);
    __syncthreads();
    double u0[ZV];
#pragma unroll
    for (int v = 0; v < ZV; ++v) u0[v] = double(lds[s.base + (v + R) * Pitch<R, DIM>::C]);
    for (int q = 0; q < ncls; ++q) {
      const int o1 = cls[4 * q], o2 = cls[4 * q + 1], zr = cls[4 * q + 2];
      const T* p1 = lds + s.base + o1;
      const T* p2 = lds + s.base + o2;
      double E1[ZV + 2 * R], E2[ZV + 2 * R];
#pragma unroll
      for (int w = 0; w < ZV + 2 * R; ++w) {
        E1[w] = double(p1[w * Pitch<R, DIM>::C]);
        E2[w] = double(p2[w * Pitch<R, DIM>::C]);
      }
      const double* cf = kw + (long long)b * nkw + 3 * cls[4 * q + 3];   // the row of dC = 0
      const int lo = o1 == o2 ? 1 : -zr;
#pragma unroll
      for (int d = -R; d <= R; ++d) {
        if (d < lo || d > zr) continue;
        const double* e = cf + 3 * d;
        const double e0 = e[0], e1 = e[1], e2 = e[2];
#pragma unroll
        for (int v = 0; v < ZV; ++v) {
          const double x = (E1[v + R + d] - u0[v]) + (E2[v + R - d] - u0[v]);
          r[0][v] += e0 * x;
          r[1][v] += e1 * x;
          r[2][v] += e2 * x;
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < ZV; ++v) {
    if (!live(G, s, v)) continue;
#pragma unroll
    for (int a = 0; a < 3; ++a)
      if (a < DIM) out[((long long)k * DIM + a) * nvox + voxel(G, s, v)] = T(r[a][v]);
  }
}

// Normal equations of the matrix form, 2 NF features per component: with
// every component of the tile staged, per offset the differences
// d_b = u_b(x + r) - u_b(x), their projection e . d, and the shell sums
// S_a = sum d_a, T_a = sum e_a (e . d); then Phi1[a][m] += W[m] S_a and
// Phi2[a][m] += W[m] T_a per shell.  The products Phi Phi^T, with Gamma as one
// more feature, are contractions over the voxels: every wave passes its
// features through LDS into the operand layout of v_mfma_f64_16x16x4 (lane l:
// row l % 16, k = l / 16; the same register is both operands) and keeps the
// 16 x 16 tile (two rows of tiles from 8 features on) in its accumulators.
// Before, each of 120 threads summed one entry of the triangle over the
// tile's 256 voxels with two LDS reads per product: 1107 us on eight 64^3
// FP64 fields at delta = 3, degree 6, against 296 us.
constexpr int kHalf = 32, kFPitch = kHalf + 1;   // voxels per transposition, LDS pitch (doubles)
template <typename T, int DIM, int NF>
__global__ __launch_bounds__(NT) void k_nl_gram1(Geom G, const T* __restrict__ u, const T* __restrict__ gam,
                                                 int nsample, const int* __restrict__ offs,
                                                 const int* __restrict__ first, int nshell,
                                                 const double* __restrict__ ev, const double* __restrict__ W,
                                                 double* __restrict__ partial) {
  constexpr int ROWS = 2 * NF + 1;                 // features and Gamma
  constexpr int NTL = ROWS <= 16 ? 1 : 2;          // 16-row tiles
  constexpr int NPR = NTL * (NTL + 1) / 2;
  extern __shared__ __align__(16) unsigned char smem[];
  int2* tab = reinterpret_cast<int2*>(smem);
  T* lds = reinterpret_cast<T*>(smem + kRowBytes);
  const long long nvox = (long long)G.nA * G.nB * G.nC;
  const int ntile = G.ntA * G.ntB * G.ntC;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* tr = reinterpret_cast<double*>(smem + kRowBytes) + wave * ROWS * kFPitch;   // over the box, once it has been read
  d4 acc[NPR];
#pragma unroll
  for (int i = 0; i < NPR; ++i) acc[i] = d4{0.0, 0.0, 0.0, 0.0};
  for (long long item = blockIdx.x; item < (long long)nsample * ntile; item += gridDim.x) {
    const int k = int(item / ntile);
    const Spot s = spot(G, int(item - (long long)k * ntile), 1);
    __syncthreads();
    row_table(G, s, tab);
    __syncthreads();
    for (int b = 0; b < DIM; ++b) stage<3>(G, u + ((long long)k * DIM + b) * nvox, s, tab, lds + b);
    __syncthreads();
    const int ctr = 3 * (s.base + G.R * G.sC);
    double p1[3][NF], p2[3][NF], u0[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      u0[a] = (a < DIM) ? double(lds[ctr + a]) : 0.0;
#pragma unroll
      for (int m = 0; m < NF; ++m) {
        p1[a][m] = 0.0;
        p2[a][m] = 0.0;
      }
    }
    for (int q = 0; q < nshell; ++q) {
      const int o1 = first[q + 1];
      double S[3] = {0.0, 0.0, 0.0}, E[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
      for (int o = first[q]; o < o1; ++o) {
        const T* p = lds + ctr + offs[o];
        const double e0 = ev[3 * o], e1 = ev[3 * o + 1], e2 = ev[3 * o + 2];
        const double d0 = double(p[0]) - u0[0], d1 = double(p[1]) - u0[1];
        const double d2 = (DIM == 3) ? double(p[2]) - u0[2] : 0.0;
        const double pr = e0 * d0 + e1 * d1 + e2 * d2;
        S[0] += d0;
        S[1] += d1;
        S[2] += d2;
        E[0] += e0 * pr;
        E[1] += e1 * pr;
        E[2] += e2 * pr;
      }
#pragma unroll
      for (int m = 0; m < NF; ++m) {
        const double w = W[q * NF + m];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          p1[a][m] += w * S[a];
          p2[a][m] += w * E[a];
        }
      }
    }
    const bool ok = live(G, s, 0);
    __syncthreads();   // the box has been read: the waves' transposition tiles replace it
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      if (a >= DIM) break;
      const double gv = ok ? double(gam[((long long)k * DIM + a) * nvox + voxel(G, s, 0)]) : 0.0;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if ((lane >> 5) == h) {
          const int l = lane & 31;
#pragma unroll
          for (int m = 0; m < NF; ++m) {
            tr[m * kFPitch + l] = ok ? p1[a][m] : 0.0;
            tr[(NF + m) * kFPitch + l] = ok ? p2[a][m] : 0.0;
          }
          tr[2 * NF * kFPitch + l] = gv;
        }
        // one wave writes and reads its own tile: order the accesses, no barrier
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int i = lane & 15, kk = lane >> 4;
#pragma unroll
        for (int st = 0; st < kHalf / 4; ++st) {
          double f[NTL];
#pragma unroll
          for (int t = 0; t < NTL; ++t) {
            const int row = 16 * t + i;
            f[t] = (row < ROWS) ? tr[row * kFPitch + 4 * st + kk] : 0.0;
          }
#pragma unroll
          for (int t = 0, n = 0; t < NTL; ++t)
#pragma unroll
            for (int t2 = t; t2 < NTL; ++t2, ++n)
              acc[n] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[t], f[t2], acc[n], 0, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  // the four waves' tiles in a fixed order, then the workgroup's slot:
  // entry (i, j) of tile pair n at n 256 + i 16 + j
  double* red = reinterpret_cast<double*>(smem + kRowBytes);
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NPR; ++n)
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave * NPR * 256 + n * 256 + (4 * r + (lane >> 4)) * 16 + (lane & 15)] = acc[n][r];
  __syncthreads();
  for (int e = threadIdx.x; e < NPR * 256; e += NT) {
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += red[w * NPR * 256 + e];
    partial[(long long)blockIdx.x * (NPR * 256) + e] = t;
  }
}

// fixed-order sum of the slots, one workgroup per entry: out[i] = sum over
// slots of partial[slot stride + i] (one workgroup for all entries took 143
// to 412 us)
__global__ __launch_bounds__(NT) void k_nl_sum(const double* __restrict__ partial, int nslot, int stride,
                                               double* __restrict__ out) {
  __shared__ double red[NT / 64];
  const int i = blockIdx.x;
  double a = 0.0;
  for (int s = threadIdx.x; s < nslot; s += NT) a += partial[(long long)s * stride + i];
  for (int off = 32; off > 0; off >>= 1) a += __shfl_down(a, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < NT / 64; ++w) t += red[w];
    out[i] = t;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
// Tiles of ta x tb lanes with zv voxels each along C, and further runs along C
// when ta tb < NT.  sC 0: dense planes.
Geom geom(int dim, const int n[3], int R, int ta, int tb, int zv, int sC) {
  Geom G{};
  G.dim = dim;
  G.nA = n[0];
  G.nB = dim == 3 ? n[1] : 1;
  G.nC = dim == 3 ? n[2] : n[1];
  G.ta = ta;
  G.tb = tb;
  G.R = R;
  const int runs = NT / (ta * tb);
  G.bv = dim == 3 ? tb : 1;
  G.cv = (dim == 3 ? runs : runs * tb) * zv;
  G.la = ta + 2 * R;
  G.lb = dim == 3 ? tb + 2 * R : 1;
  G.lc = G.cv + 2 * R;
  G.sC = sC ? sC : G.la * G.lb;
  G.ntA = (G.nA + ta - 1) / ta;
  G.ntB = (G.nB + G.bv - 1) / G.bv;
  G.ntC = (G.nC + G.cv - 1) / G.cv;
  G.tpr = 16;
  while (G.tpr < G.la) G.tpr *= 2;
  return G;
}

size_t box_bytes(const Geom& G, size_t rs) { return ((size_t)G.sC * G.lc * rs + 15) / 16 * 16; }

bool rows_ok(const Geom& G) { return G.lb * G.lc <= kRows; }

// Lanes 32 x 8 fill the LDS banks with one row of FP64 values; 16 x 16 reads
// two rows at once, which meet on some banks (a third of its LDS cycles), and
// is taken where 32 lanes would run far past the end of the x axis.
Geom pick(int dim, const int n[3], int R, int zv) {
  const Geom G = geom(dim, n, R, 32, 8, zv, pitch_c(R, dim));
  if (dim == 2) return G;
  const Geom H = geom(dim, n, R, 16, 16, zv, pitch_c(R, dim));
  return 4LL * G.ntA * G.ntB * G.ntC <= 5LL * H.ntA * H.ntB * H.ntC ? G : H;
}

// compiled feature counts (degree + 1 rounded up: the padded features are
// zero) and halos
constexpr int feature_count(int nf) { return nf <= 3 ? 3 : nf <= 5 ? 5 : nf <= 7 ? 7 : 9; }

// a workgroup's partial sums in the matrix form: pairs of 16-row tiles of the features
// and Gamma
constexpr int matrix_acc(int nf) { return 2 * nf + 1 <= 16 ? 256 : 3 * 256; }

// Fixed device scratch for a call's tables and work area: allocating and freeing the
// matrix form's 2 MB took 45 us of the 517 of its two calls at 64^3 and degree 6 (472
// without; the scalar form's 0.2 MB cost nothing measurable, 576 and 575), and 6.3 MB
// 33 of the 97 us of the normal equations of a 32 x 32 grid at degree 8.  It holds every call
// that the library takes: the partial sums of the highest degree, and tables (the
// largest, of the matrix operator at horizon 7 in 3D, 51 KB).
// A device's copy belongs to one call at a time, which holds it until its stream has
// drained; a second call meanwhile allocates.
constexpr size_t kSums = sizeof(double) * (kSlots1 + 1) * matrix_acc(feature_count(kNlMaxDegree + 1));
constexpr size_t kScratch = kSums + (128u << 10);
static_assert(kSlots * 55 <= kSlots1 * matrix_acc(feature_count(kNlMaxDegree + 1)), "scalar form: 55 sums of nine features");
__device__ __align__(256) char nl_scratch[kScratch];
constexpr int kMaxDevices = 64;
std::atomic<bool> scratch_held[kMaxDevices];

struct Scratch {
  int device = -1;   // held
  char* claim(size_t bytes) {
    int d = -1;
    void* p = nullptr;
    if (bytes > kScratch || hipGetDevice(&d) != hipSuccess || d < 0 || d >= kMaxDevices) return nullptr;
    if (scratch_held[d].exchange(true, std::memory_order_acquire)) return nullptr;
    device = d;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(nl_scratch)) != hipSuccess) p = nullptr;
    if (!p) release();
    return static_cast<char*>(p);
  }
  void release() {
    if (device >= 0) scratch_held[device].store(false, std::memory_order_release);
    device = -1;
  }
};

// device copy of a call's tables (ints first, then doubles) followed by the
// work area; given back with it
struct Tables {
  char* buf = nullptr;      // allocated
  Scratch scratch;          // or held
  hipStream_t stream = nullptr;
  const int* ints = nullptr;
  const double* vals = nullptr;
  double* work = nullptr;
  ~Tables() {
    if (buf) (void)hipFree(buf);
    if (scratch.device >= 0) {
      (void)hipStreamSynchronize(stream);   // also after an error: nothing queued may use it any more
      scratch.release();
    }
  }
  hipError_t upload(const std::vector<int>& i, const std::vector<double>& v, size_t nwork, hipStream_t st) {
    const size_t b_i = (sizeof(int) * i.size() + 255) / 256 * 256, b_v = (sizeof(double) * v.size() + 255) / 256 * 256;
    host.resize(b_i + sizeof(double) * v.size());
    std::copy(i.begin(), i.end(), reinterpret_cast<int*>(host.data()));
    std::copy(v.begin(), v.end(), reinterpret_cast<double*>(host.data() + b_i));
    const size_t bytes = b_i + b_v + sizeof(double) * nwork + 256;
    stream = st;
    char* at = scratch.claim(bytes);
    if (!at) {
      if (hipMalloc(reinterpret_cast<void**>(&buf), bytes) != hipSuccess) {
        buf = nullptr;
        return hipErrorOutOfMemory;
      }
      at = buf;
    }
    ints = reinterpret_cast<const int*>(at);
    vals = reinterpret_cast<const double*>(at + b_i);
    work = reinterpret_cast<double*>(at + b_i + b_v);
    return hipMemcpyAsync(at, host.data(), host.size(), hipMemcpyHostToDevice, st);
  }
  std::vector<char> host;   // outlives the copy: every caller synchronises before this goes
};

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             kMaxDynamicLds);
}

// classes of the scalar form: row(|r|^2) -> weight row of nw doubles; the row of
// r = 0 (FP32 fields) is minus the sum of all the others over the horizon
template <typename Fn>
void scalar_classes(const Geom& G, int R, double delta, int nw, Fn&& row, std::vector<int>& ints,
                    std::vector<double>& vals, int& ncls) {
  std::vector<int> cls, col;
  std::vector<double> total(nw, 0.0);
  const bool three = G.dim == 3;
  auto inside = [&](int rr) { return std::sqrt((double)rr) < delta; };
  for (int p = 0; p <= R; ++p)
    for (int q = 0; q <= (three ? p : 0); ++q) {
      if (!inside(p * p + q * q)) continue;
      int zr = 0;
      while (zr < R && inside(p * p + q * q + (zr + 1) * (zr + 1))) ++zr;
      const int c0 = (int)col.size();
      for (int sw = 0; sw < (three && p != q ? 2 : 1); ++sw)
        for (int sa = -1; sa <= 1; sa += 2)
          for (int sb = -1; sb <= 1; sb += 2) {
            const int da = sa * (sw ? q : p), db = sb * (sw ? p : q);
            if ((da == 0 && sa > 0) || (db == 0 && sb > 0)) continue;   // one sign of zero
            col.push_back(db * G.la + da);
          }
      const int n = (int)col.size() - c0;
      cls.insert(cls.end(), {c0, n, zr, (int)(vals.size() / nw)});
      for (int d = 0; d <= zr; ++d) {
        const size_t at = vals.size();
        vals.resize(at + nw, 0.0);
        if (!p && !q && !d) continue;   // the first row, filled below
        row(p * p + q * q + d * d, &vals[at]);
        for (int m = 0; m < nw; ++m) total[m] += vals[at + m] * n * (d ? 2 : 1);
      }
    }
  for (int m = 0; m < nw; ++m) vals[m] = -total[m];
  ncls = (int)cls.size() / 4;
  ints = cls;
  ints.insert(ints.end(), col.begin(), col.end());
}

// B_{m,M}(rho / delta), m = 0..M
void bernstein(int M, double delta, int rr, double* w) {
  const double t = std::sqrt((double)rr) / delta;
  double binom = 1.0;
  for (int m = 0; m <= M; ++m) {
    if (m > 0) binom = binom * (M - m + 1) / m;
    w[m] = binom * std::pow(t, m) * std::pow(1.0 - t, M - m);
  }
}

template <typename T, int NF>
hipError_t gram_r(int R, const Geom& G, size_t lds, unsigned grid, hipStream_t st, const void* u, const void* gam,
                  int nsample, const Tables& t, int ncls) {
  switch (R) {
#define X(R_)                                                                                                  \
  case R_: {                                                                                                   \
    auto* kern = G.dim == 3 ? k_nl_gram<T, R_, 3, NF> : k_nl_gram<T, R_, 2, NF>;                               \
    const hipError_t e = allow_lds(kern, lds);                                                                 \
    if (e != hipSuccess) return e;                                                                             \
    hipLaunchKernelGGL(kern, dim3(grid), NT, lds, st, G, static_cast<const T*>(u), static_cast<const T*>(gam), \
                       nsample, t.ints, ncls, t.ints + 4 * ncls, t.vals, t.work);                              \
    return hipGetLastError();                                                                                  \
  }
    X(1) X(2) X(3) X(4) X(5) X(6)
#undef X
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t gram_scalar(int dim, const int n[3], int R, double delta, int deg, int nsample, const void* u,
                       const void* gam, double* G_, double* g_, double* gg_, hipStream_t st) {
  const int nf = deg + 1, NF = feature_count(nf);
  const Geom G = pick(dim, n, R, 4);
  if (!rows_ok(G)) return hipErrorInvalidValue;
  const int tri = NF * (NF + 1) / 2, nacc = tri + NF + 1;
  std::vector<int> ints;
  std::vector<double> vals;
  int ncls = 0;
  scalar_classes(G, R, delta, NF, [&](int rr, double* w) { bernstein(deg, delta, rr, w); }, ints, vals, ncls);
  const long long items = (long long)nsample * G.ntA * G.ntB * G.ntC;
  const unsigned grid = (unsigned)(items < kSlots ? items : kSlots);
  Tables t;
  hipError_t e = t.upload(ints, vals, ((size_t)grid + 1) * nacc, st);
  if (e != hipSuccess) return e;
  const size_t lds = kRowBytes + std::max(box_bytes(G, sizeof(T)), sizeof(double) * nacc * (NT / 64));
  switch (NF) {
    case 3: e = gram_r<T, 3>(R, G, lds, grid, st, u, gam, nsample, t, ncls); break;
    case 5: e = gram_r<T, 5>(R, G, lds, grid, st, u, gam, nsample, t, ncls); break;
    case 7: e = gram_r<T, 7>(R, G, lds, grid, st, u, gam, nsample, t, ncls); break;
    default: e = gram_r<T, 9>(R, G, lds, grid, st, u, gam, nsample, t, ncls); break;
  }
  if (e != hipSuccess) return e;
  double* out = t.work + (size_t)grid * nacc;
  hipLaunchKernelGGL(k_nl_sum, dim3((unsigned)nacc), NT, 0, st, t.work, (int)grid, nacc, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  std::vector<double> acc(nacc);
  if ((e = hipMemcpyAsync(acc.data(), out, sizeof(double) * nacc, hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  for (int m = 0; m < nf; ++m) {
    for (int k = m; k < nf; ++k) G_[m * nf + k] = G_[k * nf + m] = acc[m * NF - m * (m - 1) / 2 + (k - m)];
    g_[m] = acc[tri + m];
  }
  *gg_ = acc[tri + NF];
  return hipSuccess;
}

// offsets of the matrix-form normal equations by ascending shell
template <typename T>
hipError_t gram_matrix(int dim, const int n[3], int R, double delta, int deg, int nsample, const void* u,
                       const void* gam, double* G_, double* g_, double* gg_, hipStream_t st) {
  const int nf1 = deg + 1, NF = feature_count(nf1), nf = 2 * nf1;
  // 16 lanes along A and one voxel per thread: 16 x 4 x 4 voxels in 3D,
  // 16 x 16 in 2D (every component of the tile is staged at once)
  const Geom G = geom(dim, n, R, 16, dim == 3 ? 4 : 16, 1, 0);
  if (!rows_ok(G)) return hipErrorInvalidValue;
  std::vector<int> shell_rr;
  const int rmax = (int)std::ceil(delta * delta) + 1, rb = dim == 3 ? R : 0;
  std::vector<int> offs, first(1, 0);
  std::vector<double> ev, W;
  for (int rr = 1; rr <= rmax; ++rr) {
    if (!(std::sqrt((double)rr) < delta)) break;
    const size_t was = offs.size();
    for (int dc = -R; dc <= R; ++dc)
      for (int db = -rb; db <= rb; ++db)
        for (int da = -R; da <= R; ++da) {
          if (da * da + db * db + dc * dc != rr) continue;
          const double rho = std::sqrt((double)rr);
          offs.push_back(3 * (dc * G.sC + db * G.la + da));
          // components x first: the C axis is component dim - 1
          ev.push_back(da / rho);
          ev.push_back(dim == 3 ? db / rho : dc / rho);
          ev.push_back(dim == 3 ? dc / rho : 0.0);
        }
    if (offs.size() == was) continue;
    while (offs.size() % 4) {   // whole groups of four: r = 0 adds nothing
      offs.push_back(0);
      ev.insert(ev.end(), {0.0, 0.0, 0.0});
    }
    first.push_back((int)offs.size());
    W.resize(W.size() + NF, 0.0);
    bernstein(deg, delta, rr, &W[W.size() - NF]);
  }
  const int nshell = (int)first.size() - 1;
  if (nshell < 1) return hipErrorInvalidValue;
  std::vector<int> ints(first);
  ints.insert(ints.end(), offs.begin(), offs.end());
  std::vector<double> vals(ev);
  vals.insert(vals.end(), W.begin(), W.end());
  const int rows = 2 * NF + 1, nacc = matrix_acc(NF);
  const long long items = (long long)nsample * G.ntA * G.ntB * G.ntC;
  const unsigned grid = (unsigned)(items < kSlots1 ? items : kSlots1);
  Tables t;
  hipError_t e = t.upload(ints, vals, ((size_t)grid + 1) * nacc, st);
  if (e != hipSuccess) return e;
  size_t lds = 3 * box_bytes(G, sizeof(T));
  lds = std::max(lds, sizeof(double) * (size_t)(NT / 64) * rows * kFPitch);
  lds = std::max(lds, sizeof(double) * (size_t)(NT / 64) * nacc);
  lds += kRowBytes;
  if (lds > (size_t)kMaxDynamicLds) return hipErrorInvalidValue;
  const int* d_first = t.ints;
  const int* d_offs = t.ints + nshell + 1;
  const double* d_W = t.vals + ev.size();
  switch (NF) {
#define X(N_)                                                                                                       \
  case N_:                                                                                                          \
    {                                                                                                               \
      auto* kern = dim == 3 ? k_nl_gram1<T, 3, N_> : k_nl_gram1<T, 2, N_>;                                          \
      if ((e = allow_lds(kern, lds)) != hipSuccess) return e;                                                       \
      hipLaunchKernelGGL(kern, dim3(grid), NT, lds, st, G, static_cast<const T*>(u), static_cast<const T*>(gam),    \
                         nsample, d_offs, d_first, nshell, t.vals, d_W, t.work);                                    \
    }                                                                                                               \
    break;
    X(3) X(5) X(7) X(9)
#undef X
    default: return hipErrorInvalidValue;
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  double* out = t.work + (size_t)grid * nacc;
  hipLaunchKernelGGL(k_nl_sum, dim3((unsigned)nacc), NT, 0, st, t.work, (int)grid, nacc, out);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  std::vector<double> acc(nacc);
  if ((e = hipMemcpyAsync(acc.data(), out, sizeof(double) * nacc, hipMemcpyDeviceToHost, st)) != hipSuccess) return e;
  if ((e = hipStreamSynchronize(st)) != hipSuccess) return e;
  // entry of rows i <= j: tile pairs (0, 0)[, (0, 1), (1, 1)]
  auto entry = [&](int i, int j) {
    if (i > j) std::swap(i, j);
    const int pr = (i >= 16 ? 2 : (j >= 16 ? 1 : 0));
    return acc[pr * 256 + (i % 16) * 16 + (j % 16)];
  };
  auto row = [&](int m) { return m < nf1 ? m : NF + (m - nf1); };
  for (int m = 0; m < nf; ++m) {
    for (int k = m; k < nf; ++k) G_[m * nf + k] = G_[k * nf + m] = entry(row(m), row(k));
    g_[m] = entry(row(m), 2 * NF);
  }
  *gg_ = entry(2 * NF, 2 * NF);
  return hipSuccess;
}

template <typename T>
hipError_t apply_form(int dim, const int n[3], int R, double delta, int form, int nsample, const void* u,
                      const double* c, int deg, void* out, hipStream_t st) {
  const Geom G = pick(dim, n, R, 8);
  if (!rows_ok(G)) return hipErrorInvalidValue;
  const long long items = (long long)nsample * G.ntA * G.ntB * G.ntC;
  if (items > 0x7fffffffLL) return hipErrorInvalidValue;
  const int nf1 = deg + 1;
  std::vector<double> basis(nf1);
  auto kernel_at = [&](int rr, int f) {
    bernstein(deg, delta, rr, basis.data());
    double k = 0.0;
    for (int m = 0; m < nf1; ++m) k += c[f * nf1 + m] * basis[m];
    return k;
  };
  std::vector<int> ints;
  std::vector<double> vals;
  int ncls = 0;
  if (form == 0) {
    scalar_classes(G, R, delta, 1, [&](int rr, double* w) { *w = kernel_at(rr, 0); }, ints, vals, ncls);
  } else {
    std::vector<double> tab[3];
    const int rb = dim == 3 ? R : 0;
    auto inside = [&](int rr) { return std::sqrt((double)rr) < delta; };
    for (int db = 0; db <= rb; ++db)
      for (int da = db ? -R : 0; da <= R; ++da) {   // one column of each pair of opposites
        if (!inside(da * da + db * db)) continue;
        int zr = 0;
        while (zr < R && inside(da * da + db * db + (zr + 1) * (zr + 1))) ++zr;
        const int at = db * G.la + da;
        ints.insert(ints.end(), {at, -at, zr, (int)(tab[0].size() / 3) + zr});
        for (int dc = -zr; dc <= zr; ++dc) {
          const int rr = da * da + db * db + dc * dc;
          const double rho = rr ? std::sqrt((double)rr) : 1.0;
          const double k1 = rr ? kernel_at(rr, 0) : 0.0, k2 = rr ? kernel_at(rr, 1) : 0.0;
          const double e[3] = {da / rho, (dim == 3 ? db : dc) / rho, (dim == 3 ? dc : 0) / rho};
          for (int b = 0; b < 3; ++b)
            for (int a = 0; a < 3; ++a) tab[b].push_back(k2 * e[a] * e[b] + (a == b ? k1 : 0.0));
        }
      }
    for (int b = 0; b < 3; ++b) vals.insert(vals.end(), tab[b].begin(), tab[b].end());
    ncls = (int)ints.size() / 4;
  }
  Tables t;
  hipError_t e = t.upload(ints, vals, 0, st);
  if (e != hipSuccess) return e;
  const int nkw = (int)vals.size() / 3;
  const size_t lds = kRowBytes + box_bytes(G, sizeof(T));
  switch (R) {
#define X(R_)                                                                                                      \
  case R_:                                                                                                         \
    if (form == 0) {                                                                                               \
      auto* kern = dim == 3 ? k_nl_apply<T, R_, 3> : k_nl_apply<T, R_, 2>;                                         \
      if ((e = allow_lds(kern, lds)) != hipSuccess) return e;                                                      \
      hipLaunchKernelGGL(kern, dim3((unsigned)items), NT, lds, st, G, static_cast<const T*>(u), nsample, t.ints,   \
                         ncls, t.ints + 4 * ncls, t.vals, static_cast<T*>(out));                                   \
    } else {                                                                                                       \
      auto* kern = dim == 3 ? k_nl_apply1<T, R_, 3> : k_nl_apply1<T, R_, 2>;                                       \
      if ((e = allow_lds(kern, lds)) != hipSuccess) return e;                                                      \
      hipLaunchKernelGGL(kern, dim3((unsigned)items), NT, lds, st, G, static_cast<const T*>(u), nsample, t.ints,   \
                         ncls, t.vals, nkw, static_cast<T*>(out));                                                 \
    }                                                                                                              \
    break;
    X(1) X(2) X(3) X(4) X(5) X(6)
#undef X
    default: return hipErrorInvalidValue;
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return hipStreamSynchronize(st);
}

}  // namespace

hipError_t nl_gram(bool f64, int dim, const int n[3], int R, double delta, int deg, int form, int nsample,
                   const void* u, const void* gam, double* G, double* g, double* gg, hipStream_t st) {
  if (deg < 0 || deg > kNlMaxDegree || R < 1 || nsample < 1 || (form != 0 && form != 1)) return hipErrorInvalidValue;
  if (R > (form == 1 && dim == 3 ? kNlMaxHalo1 : kNlMaxHalo)) return hipErrorInvalidValue;
  if (form == 0)
    return f64 ? gram_scalar<double>(dim, n, R, delta, deg, nsample, u, gam, G, g, gg, st)
               : gram_scalar<float>(dim, n, R, delta, deg, nsample, u, gam, G, g, gg, st);
  return f64 ? gram_matrix<double>(dim, n, R, delta, deg, nsample, u, gam, G, g, gg, st)
             : gram_matrix<float>(dim, n, R, delta, deg, nsample, u, gam, G, g, gg, st);
}

hipError_t nl_apply(bool f64, int dim, const int n[3], int R, double delta, int deg, int form, int nsample,
                    const void* u, const double* c, void* out, hipStream_t st) {
  if (deg < 0 || deg > kNlMaxDegree || R < 1 || R > kNlMaxHalo || nsample < 1 || (form != 0 && form != 1))
    return hipErrorInvalidValue;
  return f64 ? apply_form<double>(dim, n, R, delta, form, nsample, u, c, deg, out, st)
             : apply_form<float>(dim, n, R, delta, form, nsample, u, c, deg, out, st);
}

}  // namespace lsfft
